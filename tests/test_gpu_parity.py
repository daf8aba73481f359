"""GPU parity: the HIP path (through the C ABI) against the fp64 oracle, element by
element, on seeded synthetic workloads.

Tolerances: selected index sets bit-exact against the oracle's rule applied to the same
fp32 scores, and against the fp64 oracle wherever its k-th/(k+1)-th score gap exceeds
1e-3 relative; outputs within max-abs 2e-2 (bf16) / 1e-4 (fp32) and within the tighter
bound derived in tests/gpu_util.py::out_tolerances.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2510_24273_amd import binding, synth  # noqa: E402
from tests import gpu_util as gu  # noqa: E402

C = synth.CONFIGS


def _run(oracle, w, layer=0, seq_lens=None, seqs=None, label=""):
    print(f"[case] {label or w.name} layer={layer} seq_lens={seq_lens}", flush=True)
    L = synth.make_layer(w, layer, seq_lens)
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    R = gu.run_stages(ctx, w, G)
    # the fused entry point must reproduce the staged calls bit for bit
    out2 = torch.empty_like(R["out"])
    idx2 = torch.empty_like(R["idx"])
    n2 = torch.empty_like(R["n_sel"])
    ctx.decode_step(G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], G["seq_len"], out2,
                    None, idx2, n2)
    torch.cuda.synchronize()
    assert torch.equal(idx2, R["idx"]) and torch.equal(n2, R["n_sel"])
    assert torch.equal(out2.view(torch.int16) if out2.dtype == torch.bfloat16 else out2,
                       R["out"].view(torch.int16) if out2.dtype == torch.bfloat16 else R["out"])
    figs = []
    for b in (range(w.B) if seqs is None else seqs):
        figs.append(gu.check_sequence(oracle, w, L, R, b))
    print("   ", figs[0], flush=True)
    ctx.close()
    return L, R, figs


# ---- configuration 1: the tiny fp32 case, whole --------------------------------------

def test_cfg1_tiny_f32(oracle):
    _run(oracle, C["cfg1"])


# ---- small cases that span several tiles and ragged tails ----------------------------

SMALL = synth.shrink(C["cfg2"], B=3, S=1000, r=192, top_k=100, n_layers=1, plant=2)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_small_ragged_batch(oracle, dtype):
    w = synth.shrink(SMALL, dtype=dtype)
    # full, odd length, shorter than k_tot
    _run(oracle, w, seq_lens=[1000, 777, 61])


def test_fp32_value_sum_in_long_ranges(oracle, monkeypatch):
    """An fp32 context on a workspace without room for value-sum ranges of 64 tokens: ranges of 128."""
    w = synth.shrink(SMALL, dtype="f32", B=2, S=700, H=8, H_kv=8, r=128, top_k=300, plant=0)
    assert binding.workspace_bytes(gu.make_ctx(w).desc) > 722688
    monkeypatch.setattr(binding, "workspace_bytes", lambda desc: 722688)
    _run(oracle, w, seq_lens=[700, 301])


def test_empty_and_single_token_sequences(oracle):
    w = synth.shrink(SMALL, B=4, plant=0)
    _run(oracle, w, seq_lens=[0, 1, 100, 101])


def test_gqa_groups(oracle):
    for H, H_kv in ((32, 8), (8, 1), (16, 16)):
        w = synth.shrink(SMALL, H=H, H_kv=H_kv, B=2, S=600)
        _run(oracle, w, seq_lens=[600, 333], label=f"gqa H={H} H_kv={H_kv}")


@pytest.mark.parametrize("rows", [16, 48, 128])
def test_capacity_above_length(oracle, rows, monkeypatch):
    """A cache allocated for more tokens than it holds: the score kernel stops loading at the sequence length
    (after the first 16-row pass of each workgroup, which is requested before the length is known) and fills the
    rest with -inf.  Lengths on both sides of every boundary of that logic: inside a workgroup's first pass, at a
    pass boundary, at a workgroup boundary, mid-range, empty, full; `rows` = cache rows per workgroup."""
    monkeypatch.setenv("SALS_TUNE_SCORE_ROWS", str(rows))
    w = synth.shrink(SMALL, B=6, S=3000, r=128, top_k=40, plant=0)
    _run(oracle, w, seq_lens=[3000, 2 * rows, 2 * rows + 1, 2 * rows + 16, 5, 1537], label=f"capacity rows={rows} a")
    _run(oracle, w, seq_lens=[0, 2999, 2 * rows - 1, 3 * rows + 17, 16, 2048], label=f"capacity rows={rows} b")


def test_odd_sizes(oracle):
    """A cache capacity that is not a multiple of 4 (score rows of later sequences start unaligned), an odd
    selection budget, an odd multiple of 8 as scoring rank."""
    w = synth.shrink(SMALL, B=3, S=997, top_k=97, n_sink=3, n_recent=5, r=192, r_score=72, plant=0)
    _run(oracle, w, seq_lens=[997, 501, 106], label="S_max=997")
    for dtype in ("bf16", "f32"):
        wq = synth.shrink(w, dtype=dtype)
        _run(oracle, wq, seq_lens=[997, 104, 105], label=f"S_max=997 {dtype}, cache barely longer than the selection")


def test_sixty_four_query_heads(oracle):
    """H_q = 64, the most the kernels take: as 64 KV heads, and as 8 groups of 8."""
    for H_kv in (64, 8):
        w = synth.shrink(SMALL, H=64, H_kv=H_kv, B=2, S=500, plant=0)
        _run(oracle, w, seq_lens=[500, 129], label=f"H=64 H_kv={H_kv}")


@pytest.mark.parametrize("dtype,H_kv,top_k", [("bf16", 32, 127), ("bf16", 8, 129), ("bf16", 3, 260), ("f32", 8, 128)])
def test_logits_tiles_of_128_tokens(oracle, dtype, H_kv, top_k, monkeypatch):
    """The logits kernel's one-head, 128-token tiles (forced here at a small shape): selections one short of a tile, just
    past one and several tiles, sequences that fill none, part and all of the last tile, an odd number of heads."""
    monkeypatch.setenv("SALS_TUNE_LOGITS", "2")
    w = synth.shrink(SMALL, B=4, S=700, H=4 * H_kv if H_kv < 16 else H_kv, H_kv=H_kv, top_k=top_k, dtype=dtype, plant=0)
    _run(oracle, w, seq_lens=[700, top_k, 128, 5], label=f"128-token tiles {dtype} H_kv={H_kv} k={top_k}")


@pytest.mark.parametrize("B,H,H_kv,ranges", [(1, 4, 4, 2), (1, 4, 4, 3), (2, 3, 3, 8), (1, 8, 2, 8), (2, 8, 2, 16), (16, 4, 4, 8),
                                             (40, 2, 2, 2), (1, 4, 4, 16)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_token_ranges_that_cancel(dtype, B, H, H_kv, ranges, monkeypatch):
    """The value sums of neighbouring token ranges are equal and opposite up to 1e-4: what is left keeps the precision of
    fp32 sums.  Uniform weights of 1/1024 (zero query) and a projector that copies latent coordinates, so that every output
    channel is one latent sum."""
    print(f"[case] cancelling ranges {dtype} B={B} H={H}/{H_kv} ranges={ranges}", flush=True)
    monkeypatch.setenv("SALS_TUNE_PV_RANGES", str(ranges))
    n, r, d = 1024, 128, 128
    dt = gu.out_dtype(synth.shrink(SMALL, dtype=dtype))
    w = synth.shrink(SMALL, B=B, S=n, H=H, H_kv=H_kv, r=r, top_k=n, dtype=dtype)
    ctx = gu.make_ctx(w)
    g = torch.Generator(device=gu.DEV)
    g.manual_seed(ranges + B)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=gu.DEV)

    tok = -(-n // (64 * ranges)) * 64          # tokens of a range (whole 64-token steps)
    of = torch.arange(n, device=gu.DEV) // tok
    sign = torch.where(of >= n // tok // 2 * 2, 0.0, 1.0 - 2.0 * (of % 2))   # +, -, +, - ...; 0 without a whole partner
    Vc = (normal(B, 1, r) * sign[None, :, None]).to(dt)
    Vc[:, ::tok] = (0.02 * normal(B, Vc[:, ::tok].shape[1], r)).to(dt)       # one token a range holds what does not cancel
    W = ctx.pack_weights(normal(H_kv * d, r).to(dt), torch.eye(d, r, device=gu.DEV).repeat(H_kv, 1).to(dt).contiguous())
    out = torch.empty(B, H, d, dtype=dt, device=gu.DEV)
    at = torch.full((B,), n, dtype=torch.int32, device=gu.DEV)
    idx = torch.arange(n, dtype=torch.int32, device=gu.DEV).repeat(B, 1).contiguous()
    ctx.sparse_attend(torch.zeros(B, H, d, dtype=dt, device=gu.DEV), at, normal(B, n, r).to(dt), Vc, W, idx, at, out)
    torch.cuda.synchronize()
    want = Vc.double().sum(dim=1)[:, None, :] / n
    mass = Vc.double().abs().sum(dim=1)[:, None, :] / n
    # one rounding of the result, and the roundings of the partial sums: products by 1/1024 are exact, and a sum passes
    # through fewer than 16 additions of partial sums whose magnitudes add up to at most `mass`
    bound = (2.0 ** -8 if dtype == "bf16" else 2.0 ** -23) * want.abs() + 2.0 ** -20 * mass
    err = (out.double() - want).abs()
    print(f"    worst error / bound {float((err / bound).max()):.3f}", flush=True)
    assert bool((err <= bound).all())
    ctx.close()


def test_truncated_scoring_rank(oracle):
    w = synth.shrink(SMALL, r=256, r_score=128, B=2)
    _run(oracle, w, seq_lens=[1000, 500])
    w = synth.shrink(SMALL, r=256, r_score=8, B=1, plant=0)
    _run(oracle, w)


def test_sink_and_recent_window(oracle):
    w = synth.shrink(SMALL, top_k=432, n_sink=16, n_recent=64, S=2048, B=2)
    L, R, _ = _run(oracle, w, seq_lens=[2048, 513])
    idx = gu.from_dev(R["idx"])
    assert idx[0, :16].tolist() == list(range(16))
    assert idx[0, -64:].tolist() == list(range(2048 - 64, 2048))


def test_interleaved_rope_and_large_theta(oracle):
    w = synth.shrink(SMALL, rope_style=1, theta=500000.0, B=1)
    _run(oracle, w)


def test_peaky_softmax_stress(oracle):
    """Caches scaled up so that logits spread over tens of units (near one-hot softmax)."""
    w = synth.shrink(SMALL, scale=30.0, B=2, plant=0)
    _run(oracle, w, seq_lens=[1000, 900])


def test_exact_ties_resolve_to_smaller_index(oracle):
    """Duplicate cache rows give bit-equal scores; the cut must keep the smaller indices."""
    w = synth.shrink(SMALL, B=1, S=512, top_k=64, plant=0)
    L = synth.make_layer(w)
    L["Kc"][0, 1::2] = L["Kc"][0, 0::2]          # rows 2m and 2m+1 identical
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    R = gu.run_stages(ctx, w, G)
    s = gu.from_dev(R["scores"][0])
    assert np.array_equal(s[0::2], s[1::2])
    gu.check_sequence(oracle, w, L, R, 0)
    # all scores equal: the first top_k tokens win
    scores = torch.zeros((1, 512), dtype=torch.float32, device=gu.DEV)
    scores[0, 100] = -0.0
    idx = torch.empty((1, 64), dtype=torch.int32, device=gu.DEV)
    n = torch.empty((1,), dtype=torch.int32, device=gu.DEV)
    ctx.topk_select(scores, G["seq_len"], idx, n)
    torch.cuda.synchronize()
    assert sorted(idx[0].tolist()) == list(range(64))
    ctx.close()


@pytest.mark.parametrize("case", ["random", "ragged", "plateaus", "constant", "short", "nonfinite"])
def test_long_sequence_selection(oracle, case):
    """S_max above 32768 takes the multi-workgroup selection; its index set must equal the
    oracle's on the same fp32 scores (the oracle's rule: larger score first, ties to the smaller
    index).  "plateaus" crowds the threshold bin and "constant" has an empty score range: both go
    through the single-workgroup kernel that the chain falls back to, as does "short" (a cache no
    longer than the selection) and a row holding infinities."""
    S, top_k, n_sink, n_recent = 40000, 300, 4, 16
    w = synth.shrink(SMALL, B=2, S=S, top_k=top_k, n_sink=n_sink, n_recent=n_recent, plant=0)
    rng = np.random.default_rng(11)
    sc = rng.standard_normal((2, S)).astype(np.float32) * 3.0
    seq = np.array([S, S], np.int32)
    if case == "ragged":
        seq = np.array([S - 7, 33001], np.int32)
    elif case == "plateaus":
        sc = np.round(sc)                      # a few dozen distinct values, thousands of ties each
    elif case == "constant":
        sc[:] = 1.25
        sc[1, 5000] = -0.0
        sc[1, :5000] = 0.0
        sc[1, 5001:] = 0.0
    elif case == "short":
        seq = np.array([top_k + n_sink + n_recent, 17], np.int32)
    elif case == "nonfinite":
        sc[0, 123] = np.inf
        sc[0, 456] = -np.inf
    ctx = gu.make_ctx(w)
    k_tot = top_k + n_sink + n_recent
    idx = torch.full((2, k_tot), -7, dtype=torch.int32, device=gu.DEV)
    n = torch.full((2,), -7, dtype=torch.int32, device=gu.DEV)
    d_sc = torch.from_numpy(sc).to(gu.DEV)
    ctx.topk_select(d_sc, torch.from_numpy(seq).to(gu.DEV), idx, n)
    torch.cuda.synchronize()
    for b in range(2):
        want = oracle.topk(sc[b, :seq[b]].astype(np.float64), top_k, n_sink, n_recent)
        got = idx[b, :int(n[b])].cpu().numpy()
        assert int(n[b]) == len(want), (case, b)
        assert np.array_equal(np.sort(got), np.sort(want)), (case, b)
    ctx.close()


def test_selection_random_shapes(oracle):
    """Seeded sweep over cache capacities up to 70000 (all four per-thread key counts of the single-workgroup
    kernel and the multi-workgroup chain), budgets, windows, ragged lengths and tie densities: the selected
    set must equal the oracle's on the same fp32 scores, bit for bit."""
    rng = np.random.default_rng(2024)
    caps = [5, 64, 1000, 4096, 4100, 8192, 9000, 16384, 20000, 32768, 33000, 70000]
    for case, S_max in enumerate(caps * 2):
        B = int(rng.integers(1, 4))
        top_k = int(rng.integers(1, max(2, min(S_max, 3000))))
        n_sink = int(rng.integers(0, 5))
        n_recent = int(rng.integers(0, 70)) if S_max > 200 else 0
        w = synth.shrink(SMALL, B=B, S=S_max, top_k=top_k, n_sink=n_sink, n_recent=n_recent, plant=0)
        sc = rng.standard_normal((B, S_max)).astype(np.float32)
        mode = case % 3
        if mode == 1:
            sc = np.round(sc * 4) / 4                      # dense ties
        elif mode == 2:
            sc = sc * np.float32(1e-3) + np.float32(7.0)   # narrow range far from zero
        seq = rng.integers(0, S_max + 1, size=B).astype(np.int32)
        seq[0] = S_max
        print(f"[case] selection S_max={S_max} B={B} top_k={top_k} sink={n_sink} recent={n_recent} mode={mode} "
              f"seq={seq.tolist()}", flush=True)
        ctx = gu.make_ctx(w)
        idx = torch.full((B, w.k_tot), -7, dtype=torch.int32, device=gu.DEV)
        n = torch.full((B,), -7, dtype=torch.int32, device=gu.DEV)
        ctx.topk_select(torch.from_numpy(sc).to(gu.DEV), torch.from_numpy(seq).to(gu.DEV), idx, n)
        torch.cuda.synchronize()
        for b in range(B):
            want = oracle.topk(sc[b, :seq[b]].astype(np.float64), top_k, n_sink, n_recent)
            got = idx[b, :int(n[b])].cpu().numpy()
            assert int(n[b]) == len(want), (S_max, b)
            assert np.array_equal(np.sort(got), np.sort(want)), (S_max, b)
            assert np.all(idx[b, int(n[b]):].cpu().numpy() == 0)
        ctx.close()


@pytest.mark.parametrize("S,n_thr", [(4093, 1024), (4096, 1024), (9001, 1024), (32768, 1024)])
@pytest.mark.parametrize("members", [1, 2, 31, 32, 33, 64, 512, 513])
def test_threshold_bin_sizes(oracle, S, n_thr, members):
    """The cut lies in a bin of `members` scores (half of them pairwise equal), at its first, a middle and its last one: the set is
    the oracle's, and above the threshold and at it the list has the order of the threads and of their groups of four."""
    rng = np.random.default_rng(members * 7 + S)
    sc = np.concatenate([rng.uniform(0.0, 0.4, S), [0.0, 1.0]])[-S:].astype(np.float32)
    at = rng.permutation(S - 2)
    n_above = 40
    sc[at[:n_above]] = rng.uniform(0.8, 0.9, n_above)
    inside = 0.6 + np.arange(members) * 1e-7   # (a bin is 2.4e-4 wide; 2460 / 4096 = 0.60059 is the nearest edge)
    inside[1::4] = inside[0::4][: len(inside[1::4])]
    sc[at[n_above:n_above + members]] = inside
    token = np.arange(S)
    place = np.argsort((token // 4 % n_thr) * S + token, kind="stable")   # thread, group, element
    rank = np.empty(S, np.int64)
    rank[place] = np.arange(S)
    for k_in in sorted({1, (members + 1) // 2, members}):
        top_k = 1 + n_above + k_in             # (the largest score is the range's end)
        w = synth.shrink(SMALL, B=1, S=S, top_k=top_k, n_sink=0, n_recent=0, plant=0)
        ctx = gu.make_ctx(w)
        idx = torch.full((1, top_k), -7, dtype=torch.int32, device=gu.DEV)
        n = torch.full((1,), -7, dtype=torch.int32, device=gu.DEV)
        ctx.topk_select(torch.from_numpy(sc[None]).to(gu.DEV), torch.tensor([S], dtype=torch.int32, device=gu.DEV), idx, n)
        torch.cuda.synchronize()
        ctx.close()
        got = idx[0].cpu().numpy()
        want = np.sort(oracle.topk(sc.astype(np.float64), top_k, 0, 0))
        assert np.array_equal(np.sort(got), want), (members, k_in)
        tau = sc[want].min()
        gt, eq = want[sc[want] > tau], want[sc[want] == tau]
        assert got.tolist() == gt[np.argsort(rank[gt])].tolist() + eq[np.argsort(rank[eq])].tolist(), (members, k_in)


def test_decode_random_shapes(oracle):
    """Seeded sweep over descriptors: ranks, head layouts, batch sizes, budgets, windows, both storage types
    and both RoPE pairings; every stage of every sequence against the oracle."""
    rng = np.random.default_rng(77)
    for case in range(14):
        H_kv = int(rng.choice([1, 2, 3, 4, 8, 16, 32]))
        G = int(rng.choice([g for g in (1, 2, 3, 4, 8) if g * H_kv <= 64]))
        B = int(rng.integers(1, 5))
        r = 64 * int(rng.integers(1, 9))
        S = int(rng.integers(40, 2500))
        top_k = int(rng.integers(1, min(S, 700)))
        w = synth.shrink(SMALL, B=B, S=S, H=H_kv * G, H_kv=H_kv, r=r, r_score=8 * int(rng.integers(1, r // 8 + 1)),
                         top_k=top_k, n_sink=int(rng.integers(0, 4)), n_recent=int(rng.integers(0, 20)),
                         dtype=str(rng.choice(["bf16", "f32"])), rope_style=int(rng.integers(0, 2)),
                         theta=float(rng.choice([1e4, 5e5])), plant=int(rng.integers(0, 3)))
        seq = rng.integers(0, S + 1, size=B).tolist()
        seq[0] = S
        _run(oracle, w, seq_lens=seq, label=f"random #{case}: B={B} S={S} H={w.H}/{H_kv} r={r}/{w.rs} k={top_k} "
                                            f"{w.dtype} style={w.rope_style}")


def test_maximum_sizes(oracle):
    """The descriptor's upper limits in one case: a 2^20-row cache (128 selection chunks, the largest
    cos/sin table), 65536 selected tokens with sinks and a recent window, at the smallest rank."""
    w = synth.shrink(SMALL, B=1, S=1 << 20, H=8, H_kv=1, r=64, top_k=65536 - 16 - 64, n_sink=16, n_recent=64,
                     plant=0)
    _run(oracle, w, label="max S_max and k_tot")


def test_maximum_rank_and_batch_columns(oracle):
    """r = r_score = 1024 (the largest scoring rank), r = 2048 (the largest rank) in both storage types, and
    B * (H_q / H_kv) = 128 (the widest projection)."""
    _run(oracle, synth.shrink(SMALL, B=2, S=700, r=1024, plant=0), seq_lens=[700, 257], label="r=1024")
    _run(oracle, synth.shrink(SMALL, B=2, S=700, r=2048, r_score=1024, plant=0), seq_lens=[700, 257], label="r=2048")
    _run(oracle, synth.shrink(SMALL, B=1, S=300, r=2048, r_score=512, top_k=70, H=16, H_kv=16, plant=0, dtype="f32"),
         label="r=2048 f32")
    _run(oracle, synth.shrink(SMALL, B=16, S=300, H=8, H_kv=1, r=128, top_k=40, plant=0), seqs=[0, 15],
         label="B*G=128")


def test_compress_append_then_decode(oracle):
    """Algorithm 1 in order: compress the new token, append, then attend with the query on
    the appended row (q_pos = seq_len - 1)."""
    w = synth.shrink(SMALL, B=2, S=400, plant=0)
    L = synth.make_layer(w, seq_lens=[399, 200])
    G = gu.upload(L)
    rng = np.random.default_rng(5)
    k_new = synth.store(rng.standard_normal((w.B, w.D_kv)), w.dtype)
    v_new = synth.store(rng.standard_normal((w.B, w.D_kv)), w.dtype)
    ctx = gu.make_ctx(w)
    G["W"] = ctx.pack_weights(G["Uk"], G["Uv"])
    for rep in range(2):           # second call: sequence 0 is full and must be left alone
        before = G["Kc"].clone()
        ctx.compress_append(gu.to_dev(k_new), gu.to_dev(v_new), G["W"], G["Kc"], G["Vc"],
                            G["seq_len"])
        torch.cuda.synchronize()
        if rep == 0:
            assert G["seq_len"].tolist() == [400, 201]
            for b, row in ((0, 399), (1, 200)):
                for new, U, cache in ((k_new, "Uk", "Kc"), (v_new, "Uv", "Vc")):
                    want = oracle.project(synth.widen(new[b]), synth.widen(L[U]))
                    got = gu.from_dev(G[cache][b, row])
                    ulp = np.maximum(np.abs(want), 1e-30) * 2.0 ** -7     # one bf16 ulp
                    assert np.all(np.abs(got - want) <= ulp + 1e-6)
        else:
            assert G["seq_len"].tolist() == [400, 202]
            assert torch.equal(before[0].view(torch.int16), G["Kc"][0].view(torch.int16))
    # decode with the query sitting on the last appended row
    L2 = dict(L)
    for kname in ("Kc", "Vc"):
        t = G[kname].cpu()
        L2[kname] = t.view(torch.int16).numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.numpy()
    L2["seq_len"] = G["seq_len"].cpu().numpy()
    L2["q_pos"] = (L2["seq_len"] - 1).astype(np.int32)
    G["q_pos"] = gu.to_dev(L2["q_pos"])
    R = gu.run_stages(ctx, w, G)
    for b in range(w.B):
        gu.check_sequence(oracle, w, L2, R, b)
    ctx.close()


@pytest.mark.parametrize("dtype,H_kv,r,B", [
    ("bf16", 32, 640, 1),    # two slices of the D axis
    ("bf16", 32, 128, 5),    # four slices
    ("bf16", 16, 64, 3),     # slices at their shortest
    ("f32", 32, 64, 2),      # eight slices
    ("f32", 12, 192, 2),     # two slices of one and a half rounds of loads
    ("bf16", 7, 64, 16)])    # no slices
def test_sliced_append_matches_oracle(oracle, dtype, H_kv, r, B):
    """Append where the D axis is cut into slices that the length-advancing launch adds up; one sequence is full and must be
    left alone, no other row may change."""
    S = 40
    w = synth.shrink(SMALL, B=B, S=S, top_k=8, H=H_kv, H_kv=H_kv, r=r, plant=0, dtype=dtype)
    lens = [S if B > 1 and b == B - 1 else (7 * b + 3) % S for b in range(B)]
    L = synth.make_layer(w, seq_lens=lens)
    G = gu.upload(L)
    rng = np.random.default_rng(11)
    k_new = synth.store(rng.standard_normal((B, w.D_kv)), dtype)
    v_new = synth.store(rng.standard_normal((B, w.D_kv)), dtype)
    ctx = gu.make_ctx(w)
    G["W"] = ctx.pack_weights(G["Uk"], G["Uv"])
    before = {c: G[c].clone() for c in ("Kc", "Vc")}
    ctx.compress_append(gu.to_dev(k_new), gu.to_dev(v_new), G["W"], G["Kc"], G["Vc"], G["seq_len"])
    torch.cuda.synchronize()
    assert G["seq_len"].tolist() == [min(n + 1, S) for n in lens]
    for new, U, c in ((k_new, "Uk", "Kc"), (v_new, "Uv", "Vc")):
        for b, row in enumerate(lens):
            if row < S:
                want = oracle.project(synth.widen(new[b]), synth.widen(L[U]))
                got = gu.from_dev(G[c][b, row])
                tol = np.abs(want) * 2.0 ** -7 + 1e-6 if dtype == "bf16" else 1e-5
                assert np.all(np.abs(got - want) <= tol), (c, b)
                before[c][b, row] = G[c][b, row]
        assert torch.equal(before[c], G[c])
    ctx.close()


@pytest.mark.parametrize("dtype,H,H_kv,r,B", [
    ("bf16", 8, 2, 128, 4),      # 16 columns of query heads: one block
    ("bf16", 8, 2, 128, 7),      # two blocks, the second one ragged
    ("bf16", 16, 2, 192, 6),     # three blocks in a round of four
    ("bf16", 4, 4, 128, 33),     # appends in rounds of four blocks
    ("bf16", 12, 12, 64, 20),    # appends of eight waves, a round of two blocks ...
    ("bf16", 12, 12, 64, 50),    # ... of eight blocks, half of them there
    ("f32", 4, 4, 64, 70),       # five blocks of a round of eight, the fifth one ragged
    ("f32", 32, 32, 1024, 70),   # the same, with two rounds of loads along the D axis
    ("bf16", 4, 4, 128, 128),    # eight whole blocks
    ("bf16", 16, 2, 192, 16)])   # the same in the projection alone
def test_projections_in_column_blocks(oracle, dtype, H, H_kv, r, B):
    """Query projection and append over one to eight blocks of 16 columns, and more of them than a round holds: scores
    and appended rows of the sequences at the blocks' edges against the oracle, one bf16 ulp for the rows as in the tests above
    (fp32: sums of at most 4096 products of unit normals and 1 / 64 in fp32, below 1e-5)."""
    S = 24
    w = synth.shrink(SMALL, B=B, S=S, top_k=8, H=H, H_kv=H_kv, r=r, plant=0, dtype=dtype)
    lens = [(5 * b + 9) % S for b in range(B)]
    L = synth.make_layer(w, seq_lens=lens)
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    scores = torch.empty((B, S), dtype=torch.float32, device="cuda")
    ctx.latent_scores(G["q"], G["W"], G["Kc"], G["seq_len"], scores)
    rng = np.random.default_rng(13)
    k_new = synth.store(rng.standard_normal((B, w.D_kv)), dtype)
    v_new = synth.store(rng.standard_normal((B, w.D_kv)), dtype)
    ctx.compress_append(gu.to_dev(k_new), gu.to_dev(v_new), G["W"], G["Kc"], G["Vc"], G["seq_len"])
    torch.cuda.synchronize()
    assert G["seq_len"].tolist() == [n + 1 for n in lens]
    for b in sorted({0, B // 2, B - 2, B - 1} | {e for e in (15, 16, 31, 32, 63, 64) if e < B}):
        n = lens[b]
        qt = oracle.project(oracle.group_sum(synth.widen(L["q"][b]), H_kv), synth.widen(L["Uk"]))
        K = synth.widen(L["Kc"][b][:n])
        got = gu.from_dev(scores[b])
        bound = 2e-5 * np.linalg.norm(qt[:w.rs]) * np.linalg.norm(K[:, :w.rs], axis=1) + 1e-6
        assert np.all(np.abs(got[:n] - oracle.scores(qt, K, w.rs)) <= bound), b
        assert np.all(np.isneginf(got[n:])), b
        for new, U, c in ((k_new, "Uk", "Kc"), (v_new, "Uv", "Vc")):
            want = oracle.project(synth.widen(new[b]), synth.widen(L[U]))
            tol = np.abs(want) * 2.0 ** -7 + 1e-6 if dtype == "bf16" else 1e-5
            assert np.all(np.abs(gu.from_dev(G[c][b, n]) - want) <= tol), (c, b)
    ctx.close()


@pytest.mark.parametrize("dtype,H,H_kv,r,top_k,lens", [
    ("bf16", 32, 32, 192, 3, [500, 2]),             # less than one group of four tokens
    ("bf16", 32, 32, 192, 64, [500]),
    ("bf16", 32, 32, 192, 65, [500, 64, 0]),        # two tiles, ranges past the selection
    ("bf16", 32, 32, 640, 129, [500]),              # two ranges, the last tile of one token
    ("bf16", 32, 32, 640, 250, [500]),              # two rounds of loads
    ("bf16", 32, 8, 256, 255, [500, 131]),          # a workgroup's limit (eight slices would pass it: added up beforehand)
    ("bf16", 64, 64, 256, 100, [300]),              # two head blocks, rounds of 64 tokens
    ("bf16", 24, 3, 128, 77, [300, 299, 5]),        # heads that do not fill a block
    ("f32", 32, 32, 192, 128, [500]),               # ranges of one step
    ("f32", 32, 32, 128, 200, [500]),
    ("f32", 64, 8, 128, 61, [300, 60])])
def test_value_sum_adds_logit_slices(oracle, dtype, H, H_kv, r, top_k, lens, monkeypatch):
    """Split logits that the value sum adds up: against the oracle, and against the unsplit logits within twice the bound that
    both keep to it."""
    w = synth.shrink(SMALL, B=len(lens), S=max(lens), r=r, H=H, H_kv=H_kv, top_k=top_k, plant=0, dtype=dtype)
    L, R, _ = _run(oracle, w, seq_lens=lens, label=f"added slices {dtype} H={H}/{H_kv} r={r} k={top_k}")
    monkeypatch.setenv("SALS_TUNE_LOGITS_KSPLIT", "0")
    _, R1, _ = _run(oracle, w, seq_lens=lens, label="unsplit")
    assert torch.equal(R["idx"], R1["idx"])
    y, y1 = gu.from_dev(R["out"]), gu.from_dev(R1["out"])
    for b in range(w.B):
        assert np.max(np.abs(y[b] - y1[b])) <= 2 * gu.out_tolerances(w, y1[b])[1]


def test_query_position_beyond_the_cache(oracle):
    """q_pos far above S_max: the query's angles are then evaluated in the kernel instead of
    being read from the per-context cos/sin table."""
    w = synth.shrink(SMALL, B=2)
    L = synth.make_layer(w)
    L["q_pos"] = np.array([w.S + 1, 1_000_003], np.int32)
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    R = gu.run_stages(ctx, w, G)
    for b in range(w.B):
        gu.check_sequence(oracle, w, L, R, b)
    ctx.close()


def test_graph_replays_match_eager(oracle):
    """decode_step captured in a HIP graph: every replay (with eager work and synchronisations of the same
    context in between, and the inputs changed between replays) equals the eager result bit for bit."""
    w = synth.shrink(SMALL, B=2, S=1500, top_k=300, plant=1)
    ctx = gu.make_ctx(w)
    Ls = [synth.make_layer(w, layer) for layer in range(3)]
    Gs = [gu.upload(L, ctx) for L in Ls]
    eager = []
    for G in Gs:
        o = torch.empty((w.B, w.H, w.d), dtype=gu.out_dtype(w), device=gu.DEV)
        ctx.decode_step(G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], G["seq_len"], o)
        eager.append(o)
    torch.cuda.synchronize()
    # static buffers the graph reads; refilled before every replay
    S = {k: Gs[0][k].clone() for k in ("q", "q_pos", "Kc", "Vc", "W", "seq_len")}
    out = torch.empty_like(eager[0])
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ctx.decode_step(S["q"], S["q_pos"], S["Kc"], S["Vc"], S["W"], S["seq_len"], out)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            ctx.decode_step(S["q"], S["q_pos"], S["Kc"], S["Vc"], S["W"], S["seq_len"], out)
    torch.cuda.synchronize()
    for rep in (1, 2, 0, 1):
        for k in S:
            S[k].copy_(Gs[rep][k])
        out.fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), eager[rep].view(torch.int16)), f"replay on layer {rep} differs"
        # eager work of the same context between the replays
        tmp = torch.empty_like(out)
        ctx.decode_step(Gs[2]["q"], Gs[2]["q_pos"], Gs[2]["Kc"], Gs[2]["Vc"], Gs[2]["W"], Gs[2]["seq_len"], tmp)
        torch.cuda.synchronize()
        assert torch.equal(tmp.view(torch.int16), eager[2].view(torch.int16))
    ctx.close()


def test_repeatable_bit_for_bit(oracle):
    w = synth.shrink(SMALL, B=2)
    L = synth.make_layer(w)
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    first = gu.run_stages(ctx, w, G)
    for _ in range(5):
        again = gu.run_stages(ctx, w, G)
        assert torch.equal(first["scores"], again["scores"])
        assert torch.equal(first["idx"], again["idx"])
        assert torch.equal(first["out"].view(torch.int16), again["out"].view(torch.int16))
    ctx.close()


# ---- the measured configurations at full size ----------------------------------------

def test_fp32_cache_large_enough_for_the_streaming_loads(oracle):
    """An fp32 cache of 32 MB and more takes the score kernel's read-once loads (the bf16 form runs at every batch
    configuration): all stages against the oracle."""
    w = synth.shrink(C["cfg1"], B=2, S=16384, r=256, top_k=64, plant=2)
    assert w.B * w.S * w.r * 4 >= 32 << 20
    _run(oracle, w, seq_lens=[16384, 9000], label="fp32, 33.5 MB cache")


def test_cfg2_full(oracle):
    L, R, _ = _run(oracle, C["cfg2"], layer=0)
    sel = set(gu.from_dev(R["idx"][0]).tolist())
    assert set(L["planted"][0].tolist()) <= sel
    _run(oracle, C["cfg2"], layer=17)


@pytest.mark.parametrize("name", ["cfg3a", "cfg3b"])
def test_cfg3_full_every_sequence(oracle, name):
    L, R, _ = _run(oracle, C[name])
    for b in range(C[name].B):
        assert set(L["planted"][b].tolist()) <= set(gu.from_dev(R["idx"][b]).tolist())


def test_cfg4_full_every_sequence(oracle):
    _run(oracle, C["cfg4"])


def test_cfg5_full(oracle):
    L, R, _ = _run(oracle, C["cfg5"])
    idx = gu.from_dev(R["idx"][0])
    S = C["cfg5"].S
    assert idx[-64:].tolist() == list(range(S - 64, S)) and len(idx) == 4160


# ---- context set-up: the cos/sin table -------------------------------------------------

def test_unprepared_context_fills_its_table_lazily_and_refuses_capture(oracle):
    """A context made through the C ABI without sals_prepare: the first attend call fills the table on its own
    stream, a call on another stream is ordered behind it, results equal a prepared context's; under graph capture
    an unprepared context is refused before anything is enqueued."""
    import ctypes
    from paper_2510_24273_amd import binding
    w = synth.shrink(SMALL, B=2, plant=0)
    L = synth.make_layer(w)
    ctx = gu.make_ctx(w)                      # prepared (the binding does it)
    G = gu.upload(L, ctx)
    want = gu.run_stages(ctx, w, G)
    lib = binding._lib

    def raw_ctx():
        ws = torch.zeros(binding.workspace_bytes(ctx.desc), dtype=torch.uint8, device=gu.DEV)
        h = ctypes.c_void_p()
        assert lib.sals_create(ctypes.byref(ctx.desc), ws.data_ptr(), ws.numel(), ctypes.byref(h)) == binding.SALS_OK
        return h, ws

    def attend(h, stream, out):
        return lib.sals_sparse_attend(h, G["q"].data_ptr(), G["q_pos"].data_ptr(), G["Kc"].data_ptr(), G["Vc"].data_ptr(),
                                      G["W"].data_ptr(), want["idx"].data_ptr(), want["n_sel"].data_ptr(), out.data_ptr(),
                                      stream.cuda_stream)

    # lazily, first on a side stream, then at once on the default stream
    h, ws = raw_ctx()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    o1, o2 = torch.empty_like(want["out"]), torch.empty_like(want["out"])
    assert attend(h, side, o1) == binding.SALS_OK
    assert attend(h, torch.cuda.current_stream(), o2) == binding.SALS_OK
    torch.cuda.synchronize()
    for o in (o1, o2):
        assert torch.equal(o.view(torch.int16), want["out"].view(torch.int16))
    lib.sals_destroy(h)
    # refused under capture while unprepared; accepted after sals_prepare
    h, ws = raw_ctx()
    o3 = torch.empty_like(want["out"])
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    codes = []
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            codes.append(attend(h, s, o3))
            if codes[0] != binding.SALS_OK:
                o3.fill_(0)              # (something to capture, so that the capture itself is well formed)
    torch.cuda.synchronize()
    assert codes[0] == binding.SALS_ERR_HIP or codes[0] == binding.SALS_ERR_INVALID_ARG
    assert lib.sals_prepare(h, torch.cuda.current_stream().cuda_stream) == binding.SALS_OK
    g2 = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g2, stream=s):
            assert attend(h, s, o3) == binding.SALS_OK
    o3.fill_(7.0)
    g2.replay()
    torch.cuda.synchronize()
    assert torch.equal(o3.view(torch.int16), want["out"].view(torch.int16))
    lib.sals_destroy(h)
    ctx.close()


@pytest.mark.parametrize("dtype,H_kv,r,S,top_k,lens", [
    ("f32", 8, 256, 1000, 100, [1000, 63]), ("f32", 32, 512, 4096, 130, [4093]), ("bf16", 8, 512, 2048, 500, [2048]),
    ("bf16", 8, 256, 4096, 1000, [4001]), ("bf16", 4, 128, 4, 3, [4, 0]),
    ("bf16", 4, 256, 4, 3, [4, 0])])
def test_selection_inside_split_logits(dtype, H_kv, r, S, top_k, lens, monkeypatch):
    """Few tiles, whose latent axis is split over workgroups that each select by themselves: list, count and output equal those of
    the step with a selection launch, bit for bit (empty tiles and sequences, one tile, a list of the largest length)."""
    print(f"[case] selection in split logits {dtype} H_kv={H_kv} r={r} S={S} k={top_k}", flush=True)
    w = synth.shrink(synth.CONFIGS["cfg2"], B=len(lens), S=S, H=32, H_kv=H_kv, r=r, top_k=top_k, n_layers=1, dtype=dtype, plant=0)
    L = synth.make_layer(w, 0, lens)
    got = []
    for fuse in ("1", "0"):
        monkeypatch.setenv("SALS_TUNE_FUSE_SELECT", fuse)
        ctx = gu.make_ctx(w)
        G = gu.upload(L, ctx)
        out = torch.empty((w.B, w.H, w.d), dtype=gu.out_dtype(w), device=gu.DEV)
        idx = torch.full((w.B, w.k_tot), -7, dtype=torch.int32, device=gu.DEV)
        n_sel = torch.full((w.B,), -7, dtype=torch.int32, device=gu.DEV)
        ctx.decode_step(G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], G["seq_len"], out, None, idx, n_sel)
        torch.cuda.synchronize()
        got.append((gu.from_dev(out), idx.cpu().numpy(), n_sel.cpu().numpy()))
        ctx.close()
    (o1, i1, n1), (o0, i0, n0) = got
    assert np.array_equal(n1, n0) and n0.tolist() == [min(s, w.k_tot) for s in lens]
    for b in range(w.B):
        assert np.array_equal(i1[b, : n1[b]], i0[b, : n0[b]])
    assert np.array_equal(o1, o0)


@pytest.mark.parametrize("B,launches", [(2, 0), (5, 1)])
def test_selection_inside_one_round_of_logits_only(B, launches):
    """64-token logits of 192 workgroups select by themselves; with 480, a second round, the selection is a launch of its own (same
    list, count and output: the test above compares the two forms)."""
    print(f"[case] selection in one round of logits B={B}", flush=True)
    w = synth.shrink(synth.CONFIGS["cfg2"], B=B, S=512, H=32, H_kv=32, r=128, top_k=130, n_layers=1, dtype="f32", plant=0)
    L = synth.make_layer(w, 0)
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    out = torch.empty((w.B, w.H, w.d), dtype=gu.out_dtype(w), device=gu.DEV)
    ctx.profile(True)
    ctx.decode_step(G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], G["seq_len"], out)
    torch.cuda.synchronize()
    assert ctx.profile_collect()["topk"][1] == launches
    ctx.close()


@pytest.mark.parametrize("pick,dtype,H_kv,r,S,top_k,n_sink,lens,copies", [
    (1, "bf16", 8, 128, 32772, 700, 4, [32772, 32001], 1),    # the shortest; ranked entries in the last of three tiles
    (1, "bf16", 2, 256, 33000, 252, 0, [33000], 1),           # entries up to a tile's end
    (2, "bf16", 8, 512, 40000, 1000, 3, [39999, 700, 0], 3),  # ties; a sequence shorter than the selection, an empty one
    (2, "f32", 4, 64, 33000, 300, 4, [33000, 371], 37),       # more ties; one token more than the selection
    (1, "f32", 4, 128, 41000, 130, 1, [41000], 1),
    (2, "bf16", 4, 128, 36000, 1, 0, [36000], 1),             # one entry
    (2, "bf16", 4, 128, 36000, 200, 4, [36000, 9000], 1000)]) # more members than are ranked: selected from scratch
def test_threshold_bin_ranked_by_the_logits_kernel(pick, dtype, H_kv, r, S, top_k, n_sink, lens, copies, monkeypatch):
    """A step on a long cache leaves the ranking of the threshold bin to its logits kernel: the list is the selection call's on the
    step's scores, and the output is, bit for bit, what the attention call gives on that list."""
    print(f"[case] ranked in logits pick={pick} {dtype} H_kv={H_kv} r={r} S={S} k={top_k} lens={lens} copies={copies}", flush=True)
    monkeypatch.setenv("SALS_TUNE_LOGITS", str(pick))
    w = synth.shrink(synth.CONFIGS["cfg2"], B=len(lens), S=S, H=8, H_kv=H_kv, r=r, top_k=top_k, n_sink=n_sink, n_recent=64,
                     n_layers=1, dtype=dtype, plant=0)
    L = synth.make_layer(w, 0, lens)
    for b in range(w.B):  # runs of equal rows: equal scores
        L["Kc"][b] = np.repeat(L["Kc"][b, ::copies], copies, axis=0)[:S]
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    out, out2 = (torch.empty((w.B, w.H, w.d), dtype=gu.out_dtype(w), device=gu.DEV) for _ in range(2))
    scores = torch.empty((w.B, w.S), dtype=torch.float32, device=gu.DEV)
    idx, idx2 = (torch.full((w.B, w.k_tot), -7, dtype=torch.int32, device=gu.DEV) for _ in range(2))
    n, n2 = (torch.full((w.B,), -7, dtype=torch.int32, device=gu.DEV) for _ in range(2))
    for rep in range(2):
        ctx.decode_step(G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], G["seq_len"], out, scores, idx, n)
        ctx.topk_select(scores, G["seq_len"], idx2, n2)
        ctx.sparse_attend(G["q"], G["q_pos"], G["Kc"], G["Vc"], G["W"], idx, n, out2)
        torch.cuda.synchronize()
        assert n.tolist() == n2.tolist() == [min(s, w.k_tot) for s in lens]
        for b in range(w.B):
            k = int(n[b])
            assert torch.equal(idx[b, :k], idx2[b, :k])
        assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
    ctx.close()
