"""GPU parity of the high-precision recent window (Sec. 5.1: the recent tokens in a second,
higher-rank ring cache) and of the overlap score (Sec. 3.2) against the oracle, through the C ABI.
Same bounds as the sparse path: selection bit-exact under the shared rule, outputs within max-abs
2e-2 (bf16) / 1e-4 (fp32) and the tighter derived bound of tests/gpu_util.py::out_tolerances;
ring rows written by the append within one unit in the last place of the storage type; overlap scores within 1e-4."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2510_24273_amd import binding, synth  # noqa: E402
from tests import gpu_util as gu  # noqa: E402

C = synth.CONFIGS
SMALL = synth.shrink(C["cfg2"], B=3, S=1000, r=128, r_hi=256, top_k=100, n_sink=4, n_recent=40, n_layers=1,
                     plant=2)


def make_win_ctx(w):
    desc = binding.make_desc(w.B, w.S, w.H, w.H_kv, w.d, w.r_hi, w.n_recent, w.dtype, r_score=min(w.r_hi, 1024),
                             rope_theta=w.theta, rope_style=w.rope_style)
    return binding.Sals(desc, gu.DEV)


def _case(oracle, w, seq_lens=None, seqs=None, label=""):
    print(f"[case] window {label or w.name} B={w.B} S={w.S} r={w.r}/{w.r_hi} k={w.n_sink}+{w.top_k}+{w.n_recent} "
          f"{w.dtype} seq_lens={seq_lens}", flush=True)
    L = synth.make_layer(w, 0, seq_lens)
    Wn = synth.make_window(w, L)
    ctx, win = gu.make_ctx(w), make_win_ctx(w)
    G = gu.upload(L, ctx)
    Gw = {k: gu.to_dev(v) for k, v in Wn.items()}
    W_hi = win.pack_weights(Gw["Uk_hi"], Gw["Uv_hi"])
    idx = torch.full((w.B, w.k_tot), -7, dtype=torch.int32, device=gu.DEV)
    n_sel = torch.full((w.B,), -7, dtype=torch.int32, device=gu.DEV)
    scores = torch.empty((w.B, w.S), dtype=torch.float32, device=gu.DEV)
    out = torch.empty((w.B, w.H, w.d), dtype=gu.out_dtype(w), device=gu.DEV)
    ctx.decode_step_window(win, G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], Gw["Kw"], Gw["Vw"], W_hi,
                           G["seq_len"], out, scores, idx, n_sel)
    # the selection call leaves the same list, entry by entry; the staged call on it, and a second whole step, must reproduce
    # the step bit for bit
    idx2, n_sel2 = torch.full_like(idx, -8), torch.full_like(n_sel, -8)
    ctx.topk_select(scores, G["seq_len"], idx2, n_sel2)
    assert torch.equal(idx, idx2) and torch.equal(n_sel, n_sel2)
    out2, out3 = torch.empty_like(out), torch.empty_like(out)
    ctx.sparse_attend_window(win, G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], Gw["Kw"], Gw["Vw"], W_hi, idx2,
                             n_sel2, out2)
    ctx.decode_step_window(win, G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], Gw["Kw"], Gw["Vw"], W_hi,
                           G["seq_len"], out3)
    torch.cuda.synchronize()
    bits = (lambda t: t.view(torch.int16)) if out.dtype == torch.bfloat16 else (lambda t: t)
    assert torch.equal(bits(out), bits(out2)) and torch.equal(bits(out), bits(out3))
    R = {"scores": scores, "idx": idx, "n_sel": n_sel, "out": out}
    wd = synth.widen
    worst = 0.0
    for b in (range(w.B) if seqs is None else seqs):
        gu.check_sequence(oracle, w, L, R, b, check_out=False)   # scores and selection as in the plain path
        S = int(L["seq_len"][b])
        n = int(n_sel[b].item())
        sel = gu.from_dev(idx[b])[:n].astype(np.int32)
        y_gpu = gu.from_dev(out[b])
        if n == 0:
            assert np.all(y_gpu == 0)
            continue
        # the recent tokens come last in the selection, in token order
        n_w = min(w.n_recent, n)
        assert sel[n - n_w:].tolist() == list(range(S - n_w, S))
        y_ref = oracle.sparse_attend_window(wd(L["q"][b]), int(L["q_pos"][b]), wd(L["Kc"][b][:S]), wd(L["Vc"][b][:S]),
                                            wd(L["Uk"]), wd(L["Uv"]), wd(Wn["Kw"][b]), wd(Wn["Vw"][b]),
                                            wd(Wn["Uk_hi"]), wd(Wn["Uv_hi"]), sel, S, w.H_kv, w.theta, w.rope_style)
        star, tight = gu.out_tolerances(w, y_ref)
        err = float(np.max(np.abs(y_gpu - y_ref)))
        worst = max(worst, err)
        assert err <= star, f"b={b}: output error {err:.3e} > {star}"
        assert err <= tight, f"b={b}: output error {err:.3e} > derived bound {tight:.3e}"
        # the window matters: the plain low-rank path over the same selection gives another answer
        y_plain = oracle.sparse_attend(wd(L["q"][b]), int(L["q_pos"][b]), wd(L["Kc"][b][:S]), wd(L["Vc"][b][:S]),
                                       wd(L["Uk"]), wd(L["Uv"]), sel, w.H_kv, w.theta, w.rope_style)
        assert np.max(np.abs(y_plain - y_ref)) > 4 * tight
    print(f"    worst output error {worst:.3e}", flush=True)
    ctx.close(); win.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_small_ragged_batch(oracle, dtype):
    # full; everything selected with some tokens outside the window; cache shorter than the window
    _case(oracle, synth.shrink(SMALL, dtype=dtype), seq_lens=[1000, 141, 23])


def test_edge_lengths(oracle):
    # empty, one token, exactly the window, one more than the window, exactly the budget, one more
    w = synth.shrink(SMALL, B=6, plant=0)
    _case(oracle, w, seq_lens=[0, 1, 40, 41, 144, 145])


def test_gqa_interleaved_rope_and_ring_wrap(oracle):
    # window of 48 over lengths that are no multiple of it (the ring is entered mid-way)
    w = synth.shrink(SMALL, B=2, S=777, H=32, H_kv=8, n_recent=48, rope_style=1, theta=500000.0)
    _case(oracle, w, seq_lens=[777, 500])


@pytest.mark.parametrize("dtype,ks", [("bf16", 1), ("bf16", 2), ("f32", 4)])
def test_windows_of_several_sequences_share_a_tile(oracle, dtype, ks, monkeypatch):
    """The window pass on tiles made of two sequences' windows (chosen by itself for batches of eight and more where it is
    estimated to be faster, as in the cfg3a case below; forced here at a small rank), unsplit and with the latent axis in
    slices: an odd batch, with empty sequences, windows that are not full and full ones."""
    monkeypatch.setenv("SALS_TUNE_LOGITS", "4")
    monkeypatch.setenv("SALS_TUNE_MULTI_KSPLIT", str(ks))
    w = synth.shrink(SMALL, B=11, plant=0, dtype=dtype)
    _case(oracle, w, seq_lens=[1000, 0, 1, 40, 41, 144, 145, 500, 23, 999, 39])


def test_shared_tiles_gqa_interleaved_rope_ring_wrap(oracle, monkeypatch):
    monkeypatch.setenv("SALS_TUNE_LOGITS", "4")
    monkeypatch.setenv("SALS_TUNE_MULTI_KSPLIT", "2")
    w = synth.shrink(SMALL, B=9, S=777, H=32, H_kv=8, n_recent=48, rope_style=1, theta=500000.0, plant=0)
    _case(oracle, w, seq_lens=[777, 500, 48, 49, 47, 0, 600, 100, 776])


@pytest.mark.parametrize("B,H,r_hi", [(8, 2, 128), (9, 4, 256), (10, 6, 704), (15, 2, 320), (16, 32, 192), (9, 3, 256), (12, 1, 128),
                                      (10, 5, 704)])
def test_wide_window_tiles(oracle, B, H, r_hi, monkeypatch):
    """The launch that a step's selection shares with the window's logits on tiles of two heads and four sequences: last tiles of
    one, two, three and four sequences, slices of two steps, of three and of uneven numbers of them; empty, partial and full
    windows.  The staged call, bit for bit, runs tiles of one head and two sequences, as the shared launch does for odd numbers of
    heads."""
    monkeypatch.setenv("SALS_TUNE_LOGITS", "4")
    w = synth.shrink(SMALL, B=B, S=600, H=H, H_kv=H, r=64, r_hi=r_hi, plant=0)
    _case(oracle, w, seq_lens=[600, 0, 1, 40, 41, 144, 145, 500, 23, 599, 39, 64, 300, 2, 139, 143][:B])


@pytest.mark.parametrize("S,B,tiles", [(4099, 3, "3"), (8192, 3, "3"), (8200, 3, "3"), (5001, 5, "4"), (8192, 3, "4")])
def test_selection_and_window_logits_in_one_launch(oracle, S, B, tiles, monkeypatch):
    """Both sides of the sequence lengths at which the selection has one more group of keys per thread (4096) and a launch of its
    own (8192), rows of the score array that start unaligned, both tile forms of the window: the step against the oracle and
    against the staged call, whose passes are launches of their own."""
    monkeypatch.setenv("SALS_TUNE_LOGITS", tiles)
    w = synth.shrink(SMALL, B=B, S=S, H=4, H_kv=4, r=64, r_hi=128, top_k=150, plant=2)
    _case(oracle, w, seq_lens=[S, S - 1, 4000, 4097, 70][:B])


@pytest.mark.parametrize("S,B,tiles,top_k", [
    (4096, 2, "3", 150), (4099, 3, "3", 150), (8192, 2, "3", 700), (5001, 5, "4", 150), (8192, 9, "4", 300),
    (700, 9, "4", 20)])     # a low-rank pass of 64 tokens, in the window's tiles
def test_selection_beside_a_window_in_slices(oracle, S, B, tiles, top_k, monkeypatch):
    """The same with the window's latent axis in four slices (64-token tiles) or two (tiles of two sequences), whose sums the
    low-rank logits kernel makes on the side, or a launch of their own where it has tiles of two sequences itself."""
    monkeypatch.setenv("SALS_TUNE_LOGITS", tiles)
    monkeypatch.setenv("SALS_TUNE_MULTI_KSPLIT", "2")
    w = synth.shrink(SMALL, B=B, S=S, H=4, H_kv=4, r=64, r_hi=512, top_k=top_k, plant=2 if top_k > 100 else 0)
    _case(oracle, w, seq_lens=[S, S - 1, S // 2 + 1, 697, 70, 0, 41, 40, 500][:B])


@pytest.mark.parametrize("dtype,B,S,r_hi,slices,forced", [
    ("f32", 1, 8192, 1024, 4, 0), ("f32", 1, 8200, 1024, 8, 0), ("f32", 1, 8192, 2048, 8, 0), ("f32", 1, 8200, 2048, 8, 0),
    ("bf16", 1, 8192, 2048, 4, 0), ("bf16", 1, 8200, 2048, 8, 0), ("bf16", 16, 4096, 2048, 3, 0), ("bf16", 16, 8200, 2048, 2, 0),
    ("bf16", 16, 4096, 2048, 1, 1), ("bf16", 16, 4096, 2048, 2, 2), ("bf16", 16, 4096, 2048, 8, 8), ("bf16", 16, 8200, 2048, 1, 1)])
def test_slices_of_the_windows_latent_axis(dtype, B, S, r_hi, slices, forced, monkeypatch):
    """A window whose logits share a launch with the selection (caches of at most 8192 rows) has other slices than one with a launch of its
    own: fewer in 64-token tiles (where halved ones do not take longer than the launch saves), as many as fit beside the selection in
    tiles of two heads and four sequences; or the number asked for.  Seen through a key channel that is 2^30 - 2^30 + 20 along the
    latent axis, 256 bytes apart (in 64-token tiles every other piece of 128 is summed apart): within a slice the sum is 20, but 0 where a
    slice begins between the first two terms (the 20 beside the second is lost)."""
    if forced:
        monkeypatch.setenv("SALS_TUNE_MULTI_KSPLIT", str(forced))
    print(f"[case] window slices {dtype} B={B} S={S} r_hi={r_hi}", flush=True)
    H, r, w = 32, 64, 64
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    ctx = binding.Sals(binding.make_desc(B, S, H, H, 128, r, 100, dtype, n_recent=w, n_sink=4), gu.DEV)
    win = binding.Sals(binding.make_desc(B, S, H, H, 128, r_hi, w, dtype, r_score=1024), gu.DEV)
    zeros = lambda *s: torch.zeros(s, dtype=dt, device=gu.DEV)
    Uk, Uv = zeros(H * 128, r_hi), zeros(H * 128, r_hi)
    Uk[0] = 1.0
    Uv[0, 0] = 1.0
    W, W_hi = ctx.pack_weights(zeros(H * 128, r), zeros(H * 128, r)), win.pack_weights(Uk, Uv)
    Vw, q = zeros(B, w, r_hi), zeros(B, H, 128)
    Vw[:, 0, 0] = 1.0
    q[:, 0, 0] = 1.0
    n = torch.full((B,), 2, dtype=torch.int32, device=gu.DEV)   # two tokens, both in the window; the second one's logit is zero
    out, out2 = zeros(B, H, 128), zeros(B, H, 128)
    idx = torch.empty((B, 168), dtype=torch.int32, device=gu.DEV)
    n_sel = torch.empty((B,), dtype=torch.int32, device=gu.DEV)
    Kc, pos = zeros(B, S, r), torch.zeros_like(n)
    step = 64 // torch.empty(0, dtype=dt).element_size()   # latent coordinates
    edges = lambda k: {r_hi // step * i // k for i in range(1, k)}
    between = lambda a, b: any(a < e <= b for e in edges(slices))   # a slice begins behind step a, at step b at the latest
    for cut in sorted(edges(2) | edges(3) | edges(4) | edges(8)):
        Kw = zeros(B, w, r_hi)
        Kw[:, 0, (cut - 4) * step], Kw[:, 0, cut * step], Kw[:, 0, (cut + 4) * step] = 2.0 ** 30, -2.0 ** 30, 20.0
        ctx.decode_step_window(win, q, pos, Kc, Kc, W, Kw, Vw, W_hi, n, out, None, idx, n_sel)
        ctx.sparse_attend_window(win, q, pos, Kc, Kc, W, Kw, Vw, W_hi, idx, n_sel, out2)
        torch.cuda.synchronize()
        logit = 0.0 if between(cut - 4, cut) and not between(cut, cut + 4) else 20.0 / 128 ** 0.5
        want = 1.0 / (1.0 + np.exp(-logit))
        assert torch.equal(out, out2)
        assert np.abs(gu.from_dev(out[:, 0, 0]) - want).max() < 2.0 ** -8, (cut, gu.from_dev(out[:, 0, 0]))
    ctx.close(); win.close()


@pytest.mark.parametrize("tiles,H,H_kv,n_recent,top_k,dtype", [
    ("1", 32, 4, 40, 100, "bf16"),    # 64 sums (a head's window tile each) for 32 waves
    ("2", 32, 4, 64, 60, "bf16"),     # 64 for 32
    ("2", 16, 4, 300, 60, "bf16"),    # 160 for 96: a window of five tiles
    ("1", 16, 4, 200, 30, "f32"),     # 128 for 32
    ("2", 32, 4, 130, 30, "f32")])    # 192 for 64
def test_more_window_sums_than_waves_of_the_low_rank_pass(oracle, tiles, H, H_kv, n_recent, top_k, dtype, monkeypatch):
    """A window in latent slices, whose sums the low-rank logits kernel makes on the side, one per wave and then the rest: more
    of them than it has waves."""
    make = make_win_ctx

    def in_64_token_tiles(w):
        monkeypatch.setenv("SALS_TUNE_LOGITS", "3")
        return make(w)
    monkeypatch.setenv("SALS_TUNE_LOGITS", tiles)
    monkeypatch.setattr(sys.modules[__name__], "make_win_ctx", in_64_token_tiles)
    w = synth.shrink(SMALL, B=2, S=1100, H=H, H_kv=H_kv, n_recent=n_recent, top_k=top_k, r_hi=512, dtype=dtype, plant=0)
    _case(oracle, w, seq_lens=[1100, n_recent + top_k // 2])


@pytest.mark.parametrize("tiles", ["1", "2"])
def test_low_rank_pass_ranks_the_threshold_bin(oracle, tiles, monkeypatch):
    """A cache long enough for the chunked selection, whose last step the low-rank logits kernel takes; one sequence is shorter
    than the selection."""
    monkeypatch.setenv("SALS_TUNE_LOGITS", tiles)
    w = synth.shrink(SMALL, B=2, S=33001, H=4, H_kv=4, r=64, r_hi=128, top_k=150, plant=2)
    _case(oracle, w, seq_lens=[32999, 100])


def test_largest_window_rank(oracle):
    w = synth.shrink(SMALL, B=2, S=600, r=640, r_hi=2048, top_k=200, n_sink=16, n_recent=128, plant=0)
    _case(oracle, w, seq_lens=[600, 345])


def test_cfg2_with_the_papers_composition(oracle):
    """Full size of the measured configuration: 16 sink + 432 critical + 64 recent tokens, window rank 2048."""
    _case(oracle, synth.lookup("cfg2_win"))


def test_cfg3a_with_the_papers_composition_sampled(oracle):
    _case(oracle, synth.lookup("cfg3a_win"), seqs=[0, 7, 15])


def test_window_append_matches_oracle_over_ring_wraps(oracle):
    """25 tokens appended to both caches with a window of 8: the ring wraps three times, rows hold the last
    eight tokens' latent images within one rounding, and the step over the result matches the oracle."""
    w = synth.shrink(SMALL, B=2, S=64, r=64, r_hi=128, top_k=6, n_sink=2, n_recent=8, plant=0, H=8, H_kv=4)
    print(f"[case] window append {w.name}", flush=True)
    L = synth.make_layer(w, 0, [0, 0])
    Wn = synth.make_window(w, L)
    ctx, win = gu.make_ctx(w), make_win_ctx(w)
    G = gu.upload(L, ctx)
    W_hi = win.pack_weights(gu.to_dev(Wn["Uk_hi"]), gu.to_dev(Wn["Uv_hi"]))
    dt = gu.out_dtype(w)
    Kc = torch.zeros((w.B, w.S, w.r), dtype=dt, device=gu.DEV)
    Vc = torch.zeros_like(Kc)
    Kw = torch.zeros((w.B, w.n_recent, w.r_hi), dtype=dt, device=gu.DEV)
    Vw = torch.zeros_like(Kw)
    seq_len = torch.tensor([0, 5], dtype=torch.int32, device=gu.DEV)   # the second sequence starts mid-ring
    rng = np.random.default_rng(4)
    n_tok = 25
    toks_k = synth.store(rng.standard_normal((n_tok, w.B, w.D_kv)), w.dtype)
    toks_v = synth.store(rng.standard_normal((n_tok, w.B, w.D_kv)), w.dtype)
    for t in range(n_tok):
        k_new, v_new = gu.to_dev(toks_k[t]), gu.to_dev(toks_v[t])
        win.window_append(k_new, v_new, W_hi, Kw, Vw, seq_len)
        ctx.compress_append(k_new, v_new, G["W"], Kc, Vc, seq_len)
    torch.cuda.synchronize()
    assert seq_len.tolist() == [25, 30]
    wd = synth.widen
    Uk_hi, Uv_hi = wd(Wn["Uk_hi"]), wd(Wn["Uv_hi"])
    ulp = 2.0 ** -7 if w.dtype == "bf16" else 2.0 ** -22   # one unit in the last place of the storage type
    for b, start in enumerate((0, 5)):
        Kw_ref, Vw_ref = np.zeros((w.n_recent, w.r_hi)), np.zeros((w.n_recent, w.r_hi))
        for t in range(n_tok):
            oracle.window_append(Kw_ref, Vw_ref, wd(toks_k[t, b]), wd(toks_v[t, b]), Uk_hi, Uv_hi, start + t)
        for got, ref in ((Kw[b], Kw_ref), (Vw[b], Vw_ref)):
            err = np.abs(gu.from_dev(got) - ref)
            assert np.all(err <= ulp * np.abs(ref) + 1e-6), f"ring rows of sequence {b}: {err.max():.3e}"
    # a decode step over the caches the appends built
    q = gu.to_dev(synth.store(rng.standard_normal((w.B, w.H, w.d)), w.dtype))
    out = torch.empty((w.B, w.H, w.d), dtype=dt, device=gu.DEV)
    idx = torch.empty((w.B, w.k_tot), dtype=torch.int32, device=gu.DEV)
    n_sel = torch.empty((w.B,), dtype=torch.int32, device=gu.DEV)
    ctx.decode_step_window(win, q, seq_len, Kc, Vc, G["W"], Kw, Vw, W_hi, seq_len, out, None, idx, n_sel)
    torch.cuda.synchronize()
    for b in range(w.B):
        S = int(seq_len[b].item())
        sel = gu.from_dev(idx[b])[: int(n_sel[b].item())].astype(np.int32)
        y_ref = oracle.sparse_attend_window(gu.from_dev(q[b]), S, gu.from_dev(Kc[b][:S]), gu.from_dev(Vc[b][:S]),
                                            wd(L["Uk"]), wd(L["Uv"]), gu.from_dev(Kw[b]), gu.from_dev(Vw[b]), Uk_hi,
                                            Uv_hi, sel, S, w.H_kv, w.theta, w.rope_style)
        star, tight = gu.out_tolerances(w, y_ref)
        assert float(np.max(np.abs(gu.from_dev(out[b]) - y_ref))) <= tight
    ctx.close(); win.close()


def test_window_argument_checks():
    w = SMALL
    ctx, win = gu.make_ctx(w), make_win_ctx(w)
    bad_w = make_win_ctx(synth.shrink(w, n_recent=w.n_recent + 8))          # ring size differs from n_recent
    bad_h = make_win_ctx(synth.shrink(w, H=16, H_kv=16))                    # another model
    t = torch.zeros(64, dtype=torch.int32, device=gu.DEV)
    for other in (bad_w, bad_h, ctx):
        with pytest.raises(binding.SalsError):
            ctx.decode_step_window(other, t, t, t, t, t, t, t, t, t, t)
    with pytest.raises(binding.SalsError):
        ctx.window_append(t, t, t, t, t, t)                                 # a context with sink / recent tokens
    for c in (ctx, win, bad_w, bad_h):
        c.close()


# ---- overlap score ---------------------------------------------------------------------

def _overlap_case(oracle, w, seq_lens, seed=0):
    print(f"[case] overlap {w.name} B={w.B} S={w.S} H={w.H}/{w.H_kv} k={w.k_tot} {w.dtype} seq_lens={seq_lens}",
          flush=True)
    L = synth.make_dense_cache(w, 0)
    sl = np.asarray(seq_lens, np.int32)
    rng = np.random.default_rng(seed)
    idx = np.zeros((w.B, w.k_tot), np.int32)
    n_sel = np.zeros(w.B, np.int32)
    for b in range(w.B):
        n_sel[b] = min(int(sl[b]), int(rng.integers(0, w.k_tot + 1)) if b else w.k_tot)
        idx[b, : n_sel[b]] = rng.choice(int(sl[b]), n_sel[b], replace=False) if n_sel[b] else []
    ctx = gu.make_ctx(w)
    os_gpu = torch.full((w.B, w.H), -1.0, dtype=torch.float32, device=gu.DEV)
    ctx.overlap_score(gu.to_dev(L["q"]), gu.to_dev(sl), gu.to_dev(L["K"]), gu.to_dev(sl), gu.to_dev(idx),
                      gu.to_dev(n_sel), os_gpu)
    torch.cuda.synchronize()
    wd = synth.widen
    for b in range(w.B):
        S = int(sl[b])
        ref = oracle.overlap_score(wd(L["q"][b]), S, wd(L["K"][b][:S]), idx[b, : n_sel[b]], w.theta, w.rope_style)
        err = np.abs(gu.from_dev(os_gpu[b]) - ref)
        assert err.max() <= 1e-4, f"b={b}: overlap score error {err.max():.3e}"
    print(f"    overlap of sequence 0: mean {float(os_gpu[0].mean()):.4f}", flush=True)
    ctx.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_overlap_small(oracle, dtype):
    w = synth.shrink(C["cfg2"], B=4, S=1000, r=128, top_k=100, n_layers=1, plant=0, dtype=dtype)
    _overlap_case(oracle, w, [1000, 333, 0, 1])


def test_overlap_gqa_and_long_cache(oracle):
    w = synth.shrink(C["cfg3b"], B=2, S=9000, r=128, top_k=1000, plant=0, rope_style=1)
    _overlap_case(oracle, w, [9000, 4097], seed=3)


def test_overlap_of_the_whole_cache_is_one(oracle):
    w = synth.shrink(C["cfg2"], B=1, S=300, r=128, top_k=300, n_layers=1, plant=0)
    L = synth.make_dense_cache(w, 0)
    ctx = gu.make_ctx(w)
    sl = torch.tensor([300], dtype=torch.int32, device=gu.DEV)
    idx = torch.arange(300, dtype=torch.int32, device=gu.DEV).reshape(1, 300)
    os_gpu = torch.empty((1, w.H), dtype=torch.float32, device=gu.DEV)
    ctx.overlap_score(gu.to_dev(L["q"]), sl, gu.to_dev(L["K"]), sl, idx, sl, os_gpu)
    torch.cuda.synchronize()
    assert float((os_gpu - 1).abs().max()) <= 1e-5
    ctx.close()


def test_overlap_of_the_sals_selection_on_the_synthetic_cache(oracle):
    """The diagnostic as Sec. 3.2 uses it: the selection that the latent, RoPE-free scores make, measured
    against dense attention over the same tokens' full-rank rotated keys (here: the keys the latent cache
    stands for, reconstructed and rotated by the oracle).  Checked against the oracle; the value itself
    describes the synthetic data only."""
    w = synth.shrink(C["cfg2"], n_layers=1)
    print(f"[case] overlap of the selection, {w.name}", flush=True)
    L = synth.make_layer(w, 0)
    wd = synth.widen
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    R = gu.run_stages(ctx, w, G)
    S = w.S
    K_full = np.zeros((w.B, S, w.H_kv, w.d), dtype=np.uint16)
    for b in range(w.B):
        rec = oracle.reconstruct(wd(L["Kc"][b]), np.arange(S, dtype=np.int32), wd(L["Uk"])).reshape(S, w.H_kv, w.d)
        K_full[b] = synth.store(oracle.rope(rec, np.arange(S, dtype=np.int32), w.theta, w.rope_style), w.dtype)
    os_gpu = torch.empty((w.B, w.H), dtype=torch.float32, device=gu.DEV)
    ctx.overlap_score(G["q"], G["q_pos"], gu.to_dev(K_full), G["seq_len"], R["idx"], R["n_sel"], os_gpu)
    torch.cuda.synchronize()
    for b in range(w.B):
        sel = gu.from_dev(R["idx"][b])[: int(R["n_sel"][b].item())]
        ref = oracle.overlap_score(wd(L["q"][b]), S, wd(K_full[b]), sel, w.theta, w.rope_style)
        assert np.abs(gu.from_dev(os_gpu[b]) - ref).max() <= 1e-4
    frac = w.k_tot / S
    print(f"    overlap score: mean {float(os_gpu.mean()):.4f}, min {float(os_gpu.min()):.4f} "
          f"(selected fraction of the cache {frac:.4f})", flush=True)
    assert 0.0 < float(os_gpu.min()) and float(os_gpu.max()) <= 1.0 + 1e-6
    ctx.close()


def test_window_graph_replays_match_eager(oracle):
    """decode_step_window captured in a HIP graph: every replay, with eager work of the same contexts and
    synchronisations in between and the inputs changed, equals the eager result bit for bit."""
    w = synth.shrink(SMALL, B=2, S=1500, top_k=300, plant=1)
    print(f"[case] window graph {w.name}", flush=True)
    ctx, win = gu.make_ctx(w), make_win_ctx(w)
    Gs = []
    for layer in range(3):
        L = synth.make_layer(w, layer)
        Wn = synth.make_window(w, L, layer)
        G = gu.upload(L, ctx)
        G["Kw"], G["Vw"] = gu.to_dev(Wn["Kw"]), gu.to_dev(Wn["Vw"])
        G["W_hi"] = win.pack_weights(gu.to_dev(Wn["Uk_hi"]), gu.to_dev(Wn["Uv_hi"]))
        Gs.append(G)
    keys = ("q", "q_pos", "Kc", "Vc", "W", "Kw", "Vw", "W_hi", "seq_len")

    def step(G, o):
        ctx.decode_step_window(win, G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], G["Kw"], G["Vw"], G["W_hi"],
                               G["seq_len"], o)

    eager = []
    for G in Gs:
        o = torch.empty((w.B, w.H, w.d), dtype=gu.out_dtype(w), device=gu.DEV)
        step(G, o)
        eager.append(o)
    torch.cuda.synchronize()
    S = {k: Gs[0][k].clone() for k in keys}
    out = torch.empty_like(eager[0])
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(S, out)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            step(S, out)
    torch.cuda.synchronize()
    for rep in (1, 2, 0, 1):
        for k in S:
            S[k].copy_(Gs[rep][k])
        out.fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), eager[rep].view(torch.int16)), f"replay on layer {rep} differs"
        tmp = torch.empty_like(out)
        step(Gs[2], tmp)
        torch.cuda.synchronize()
        assert torch.equal(tmp.view(torch.int16), eager[2].view(torch.int16))
    ctx.close(); win.close()
