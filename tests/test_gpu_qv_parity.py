"""GPU parity of the quantised-value path (Sec. 5.1; Algorithm 1 with the quantised cache V-hat)
against the oracle, through the C ABI.  Codes and (scale, zero) written by the quantiser must be
bit-exact (both sides decide the code in fp32 with the same operations); attention outputs within
the same bounds as the latent-value path (tests/gpu_util.py::out_tolerances)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2510_24273_amd import binding, synth  # noqa: E402
from tests import gpu_util as gu  # noqa: E402

C = synth.CONFIGS
SMALL = synth.shrink(C["cfg2"], B=3, S=1000, r=192, top_k=100, n_layers=1, plant=2)


def _meta_f64(meta):
    """storage [.., ng, 2] -> (scale, zero) float64"""
    m = synth.widen(meta)
    return m[..., 0], m[..., 1]


def _attend_case(oracle, w, bits, seq_lens=None, seqs=None, label=""):
    print(f"[case] qv attend {label or w.name} bits={bits} seq_lens={seq_lens}", flush=True)
    L = synth.make_layer(w, 0, seq_lens)
    codes_b, meta = synth.make_qv_cache(w, 0, bits)
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    Vq, Vm = torch.from_numpy(codes_b).to(gu.DEV), gu.to_dev(meta)
    scores = torch.empty((w.B, w.S), dtype=torch.float32, device=gu.DEV)
    idx = torch.full((w.B, w.k_tot), -7, dtype=torch.int32, device=gu.DEV)
    n_sel = torch.full((w.B,), -7, dtype=torch.int32, device=gu.DEV)
    out = torch.empty((w.B, w.H, w.d), dtype=gu.out_dtype(w), device=gu.DEV)
    ctx.latent_scores(G["q"], G["W"], G["Kc"], G["seq_len"], scores)
    ctx.topk_select(scores, G["seq_len"], idx, n_sel)
    ctx.sparse_attend_qv(G["q"], G["q_pos"], G["Kc"], Vq, Vm, bits, G["W"], idx, n_sel, out)
    out2 = torch.empty_like(out)
    ctx.decode_step_qv(G["q"], G["q_pos"], G["Kc"], Vq, Vm, bits, G["W"], G["seq_len"], out2)
    torch.cuda.synchronize()
    as_bits = (lambda t: t.view(torch.int16)) if out.dtype == torch.bfloat16 else (lambda t: t)
    assert torch.equal(as_bits(out), as_bits(out2)), "decode_step_qv differs from the staged calls"
    wd = synth.widen
    worst = 0.0
    for b in (range(w.B) if seqs is None else seqs):
        S = int(L["seq_len"][b])
        n = int(n_sel[b].item())
        assert n == min(S, w.k_tot)
        sel = idx[b, :n].cpu().numpy().astype(np.int32)
        y_gpu = gu.from_dev(out[b])
        if n == 0:
            assert np.all(y_gpu == 0)
            continue
        scale, zero = _meta_f64(meta[b][:S])
        y_ref = oracle.sparse_attend_qv(wd(L["q"][b]), int(L["q_pos"][b]), wd(L["Kc"][b][:S]), wd(L["Uk"]),
                                        oracle.unpack_codes(codes_b[b][:S], bits), scale, zero, sel, w.H_kv,
                                        w.theta, w.rope_style)
        star, tight = gu.out_tolerances(w, y_ref)
        err = float(np.max(np.abs(y_gpu - y_ref)))
        worst = max(worst, err)
        assert err <= star, f"b={b}: output error {err:.3e} > {star}"
        assert err <= tight, f"b={b}: output error {err:.3e} > derived bound {tight:.3e}"
    print(f"    worst output error {worst:.3e}", flush=True)
    ctx.close()


@pytest.mark.parametrize("bits", [4, 2])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_small_ragged_batch(oracle, dtype, bits):
    _attend_case(oracle, synth.shrink(SMALL, dtype=dtype), bits, seq_lens=[1000, 37, 513])


def test_empty_and_single_token_sequences(oracle):
    _attend_case(oracle, synth.shrink(SMALL, B=4, plant=0), 4, seq_lens=[0, 1, 100, 101])


@pytest.mark.parametrize("H_kv,H", [(8, 32), (4, 32), (2, 4), (1, 8), (3, 6), (12, 24), (64, 64), (8, 64)])
def test_gqa_groups(oracle, H_kv, H):
    _attend_case(oracle, synth.shrink(SMALL, B=2, S=600, H=H, H_kv=H_kv, plant=0), 4, seq_lens=[600, 333])


@pytest.mark.parametrize("dtype,H,H_kv,r,top_k,lens,bits", [
    ("bf16", 32, 32, 192, 3, [500, 2], 2),          # less than one group of four tokens
    ("bf16", 32, 32, 640, 129, [500, 128, 0], 4),   # the last tile of one token
    ("bf16", 32, 32, 640, 250, [500], 2),
    ("bf16", 32, 8, 256, 600, [900], 4),            # three rounds of loads
    ("bf16", 8, 1, 128, 1024, [1500, 1000], 2),     # the longest range that holds its logits, eight heads
    ("bf16", 8, 1, 128, 1025, [1500], 2),           # one token more: added up beforehand
    ("f32", 64, 32, 128, 61, [300, 60], 4)])
def test_split_logits_added_by_the_value_kernel(oracle, dtype, H, H_kv, r, top_k, lens, bits):
    w = synth.shrink(SMALL, B=len(lens), S=max(lens), r=r, H=H, H_kv=H_kv, top_k=top_k, plant=0, dtype=dtype)
    _attend_case(oracle, w, bits, seq_lens=lens)


def test_many_token_ranges_and_window(oracle):
    w = synth.shrink(SMALL, B=1, S=3000, top_k=700, n_sink=4, n_recent=33, plant=0)
    _attend_case(oracle, w, 2)


def test_random_shapes(oracle):
    """Seeded sweep over head layouts, budgets (one and several token ranges), windows, code widths, storage
    types and ragged lengths."""
    rng = np.random.default_rng(99)
    for case in range(12):
        H_kv = int(rng.choice([1, 2, 3, 4, 8, 16, 32]))
        G = int(rng.choice([g for g in (1, 2, 3, 4, 8) if g * H_kv <= 64]))
        B = int(rng.integers(1, 4))
        S = int(rng.integers(50, 3000))
        top_k = int(rng.integers(1, min(S, 1500)))
        w = synth.shrink(SMALL, B=B, S=S, H=H_kv * G, H_kv=H_kv, r=64 * int(rng.integers(1, 5)), top_k=top_k,
                         n_sink=int(rng.integers(0, 4)), n_recent=int(rng.integers(0, 20)),
                         dtype=str(rng.choice(["bf16", "f32"])), rope_style=int(rng.integers(0, 2)), plant=0)
        seq = rng.integers(0, S + 1, size=B).tolist()
        seq[0] = S
        _attend_case(oracle, w, int(rng.choice([2, 4])), seq_lens=seq,
                     label=f"random #{case}: B={B} S={S} H={w.H}/{H_kv} k={top_k} {w.dtype}")


def test_maximum_sizes(oracle):
    """2^20 cache rows and 65536 selected tokens (32 token ranges of 2048)."""
    w = synth.shrink(SMALL, B=1, S=1 << 20, H=8, H_kv=1, r=64, top_k=65536 - 16 - 64, n_sink=16, n_recent=64)
    _attend_case(oracle, w, 4)


def test_cfg2_full(oracle):
    _attend_case(oracle, C["cfg2"], 4)


def test_cfg3b_sampled_sequences(oracle):
    _attend_case(oracle, C["cfg3b"], 2, seqs=[0, 7, 15])


def test_cfg4_sampled_sequence(oracle):
    _attend_case(oracle, C["cfg4"], 4, seqs=[2])


def test_operator_latency_table_shapes_sampled(oracle):
    """Shapes of the paper's operator-latency table (Table 6) as bench.py times them: SALS-25 % at batch 8 and 16,
    1k tokens, and SALS-12.5 % at batch 16, 4k tokens."""
    w = synth.lookup("t6_b8_s1024_25")
    _attend_case(oracle, w, w.qv_bits, seqs=[0, 7])
    w = synth.lookup("t6_b16_s4096_12")
    _attend_case(oracle, w, w.qv_bits, seqs=[3])
    # 128 selected tokens per sequence in two-head tiles of 256 tokens (half of every tile is padding)
    w = synth.lookup("t6_b16_s1024_25")
    _attend_case(oracle, w, w.qv_bits, seqs=[0, 15])


@pytest.mark.parametrize("bits", [4, 2])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_quantise_append_bit_exact(oracle, dtype, bits):
    """compress_append_qv: the key row as the latent projection, the value row quantised; codes,
    scales and zero points bit-exact against the oracle; full sequences untouched."""
    w = synth.shrink(SMALL, B=3, S=64, dtype=dtype, plant=0)
    print(f"[case] qv append {dtype} bits={bits}", flush=True)
    L = synth.make_layer(w, seq_lens=[63, 10, 64])
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    desc = ctx.desc
    cb, mb = binding.qv_row_bytes(desc, bits)
    assert cb == w.D_kv * bits // 8 and mb == w.D_kv // 32 * 2 * w.esize
    Vq = torch.full((w.B, w.S, cb), 0xAB, dtype=torch.uint8, device=gu.DEV)
    Vm = torch.zeros((w.B, w.S, w.D_kv // 32, 2), dtype=gu.out_dtype(w), device=gu.DEV)
    rng = np.random.default_rng(9)
    k_new = synth.store(rng.standard_normal((w.B, w.D_kv)), w.dtype)
    v_new = synth.make_values(w, 0, 1)[:, 0].copy()
    v_new[1, 32:64] = v_new[1, 40]          # a constant group: scale 0
    before_q, before_k = Vq.clone(), G["Kc"].clone()
    ctx.compress_append_qv(gu.to_dev(k_new), gu.to_dev(v_new), G["W"], G["Kc"], Vq, Vm, bits, G["seq_len"])
    torch.cuda.synchronize()
    assert G["seq_len"].tolist() == [64, 11, 64]
    codes, scale, zero = oracle.quantize_values(synth.widen(v_new), bits, w.dtype)
    packed = oracle.pack_codes(codes, bits)
    for b, row in ((0, 63), (1, 10)):
        assert np.array_equal(Vq[b, row].cpu().numpy(), packed[b]), (b, "codes")
        m = gu.from_dev(Vm[b, row])
        assert np.array_equal(m[:, 0], scale[b]) and np.array_equal(m[:, 1], zero[b]), (b, "meta")
        want = oracle.project(synth.widen(k_new[b]), synth.widen(L["Uk"]))
        got = gu.from_dev(G["Kc"][b, row])
        assert np.all(np.abs(got - want) <= np.maximum(np.abs(want), 1e-30) * 2.0 ** -7 + 1e-6)
    # the full sequence and every other row are untouched
    Vq_after = Vq.clone()
    Vq_after[0, 63] = before_q[0, 63]
    Vq_after[1, 10] = before_q[1, 10]
    assert torch.equal(Vq_after, before_q)
    as_bits = (lambda t: t.view(torch.int16)) if G["Kc"].dtype == torch.bfloat16 else (lambda t: t)
    assert torch.equal(as_bits(G["Kc"][2]), as_bits(before_k[2]))
    ctx.close()
