"""Every form of the logits kernels rounds alike.  A whole step promises, bit for bit, what the staged calls leave, and the two run
different instantiations of one body: plain, selecting by themselves, ranking the threshold bin, adding up another pass's slices,
windows by length, any group size and number of steps loaded ahead.  x*c - y*s, y*c + x*s and q1*k1 + q2*k2 are one multiplication
and one fused multiply-add; which of the products is rounded first is part of the result.

The inputs make it visible: keys whose rotation cancels, so that a rotated element is nothing but the rounding error of one product
(positive or negative as the one or the other is rounded, zero if both are), times a query that turns it into a logit of a few."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2510_24273_amd import binding, synth  # noqa: E402
from tests import gpu_util as gu  # noqa: E402

F = np.float32
D = 128
SCALE = F(1.0) / np.sqrt(F(D))
# (what cancels, RoPE pair) by KV head: an element of the rotated key, the dot product of the pairs p and p + 1; or (fp32, whose
# queries can hold a cosine) an element of the rotated query
KEYS = [("k2", 3), ("k1", 9), ("dot", 16), ("k2", 28), ("k1", 37), ("dot", 44), ("k2", 55), ("k1", 62)]
QUERIES = [("q2", 3), ("q1", 9), ("q2", 16), ("q1", 28), ("q1", 37), ("q2", 44), ("q2", 55), ("q1", 62)]
Q_POS = 7                                                 # query position of QUERIES, where the angles of the low pairs are no small ones
BASE = [(g // 5) * 32 + (g % 5) * 6 for g in range(8)]   # first of a head's six latent coordinates (in one 64-byte step, see _pieces)
QA, QB = F(148 / 128 * 2 ** 16), F(231 / 128 * 2 ** 16)  # query elements of the "dot" heads: their product is half a unit from fp32


def _cos_sin(pos, p, theta=10000.0):
    a = np.asarray(pos, dtype=np.float64) * float(F(theta)) ** (-2.0 * p / D)
    return np.cos(a).astype(F), np.sin(a).astype(F)


def _pieces(y, dtype):
    """An fp32 number as the sum of three storage elements (bf16: eight bits each; their sum is exact in any order)."""
    out, rest = [], np.asarray(y, dtype=F).copy()
    for _ in range(3):
        piece = synth.widen(synth.store(rest, dtype)).astype(F)
        out.append(piece)
        rest = (rest - piece).astype(F)
    assert not np.any(rest)
    return out


def _head_keys(head, pos):
    """The two reconstructed elements of a head's keys at positions `pos`."""
    mode, p = head
    c, s = _cos_sin(pos, p)
    if mode == "k2":
        return -c, s
    if mode == "k1":
        return s, c
    first = np.where(np.asarray(pos) == 0, F(1.0), F(0.0))   # position 0 is not turned: its logit counts, the others are 0
    return {"dot": ((QB * SCALE) * first, -(QA * SCALE) * first), "q1": (first, 0 * first), "q2": (0 * first, first)}[mode]


def _lost(x, y):
    """What a product loses when it is rounded."""
    return x.astype(np.float64) * y.astype(np.float64) - (x * y).astype(F).astype(np.float64)


def _gain(head, S):
    """The power of two that makes what is lost a logit of two to four (largest position of S, or the query's)."""
    lost = np.abs(_lost(*_cos_sin(np.arange(S) if head[0][0] == "k" else [Q_POS], head[1]))).max() * float(SCALE)
    return 2.0 ** np.ceil(np.log2(2.0 / lost))


def _logits(head, pos, S):
    """k1 = fma(y1, c, -(y2 s)), k2 = fma(y1, s, y2 c), dot = fma(q_p, k_p, q_p+1 k_p+1) and of the query
    q1 = fma(x1, c, -(x2 s)), q2 = fma(x2, c, x1 s)."""
    mode, p = head
    pos = np.asarray(pos)
    if mode == "dot":
        return np.where(pos == 0, _lost(QA * SCALE, QB * SCALE), 0.0)
    lost = _lost(*_cos_sin(pos if mode[0] == "k" else [Q_POS], p)) * float(SCALE) * _gain(head, S)
    return (-lost if mode == "k2" else lost) * (1.0 if mode[0] == "k" else pos == 0)


def _rows(heads, pos, r, dtype):
    K = np.zeros((len(pos), r))
    for g in range(8):
        for e, y in enumerate(_head_keys(heads[g], pos)):
            for i, piece in enumerate(_pieces(y, dtype)):
                K[:, BASE[g] + 3 * e + i] = piece
    return synth.store(K, dtype)


def _projector(heads, r, dtype):
    U = np.zeros((8 * D, r))
    for g, (mode, p) in enumerate(heads):
        for e, dim in enumerate((p, p + 1) if mode == "dot" else (p, p + D // 2)):
            U[g * D + dim, BASE[g] + 3 * e: BASE[g] + 3 * e + 3] = 1.0
    return synth.store(U, dtype)


def _value_projector(r, dtype):
    U = np.zeros((8 * D, r))
    for g in range(8):
        U[g * D + np.arange(64), np.arange(64)] = 1.0
    return synth.store(U, dtype)


def _sign(head, m, S):
    """of query head m of a KV head (where one logit is to stand out: the sign that lets it)"""
    if head[0][0] == "k":
        return -1.0 if m % 2 else 1.0
    return np.sign(_logits(head, [0], S)[0])


def _query(heads, B, G, S, dtype):
    q = np.zeros((B, 8 * G, D), dtype=F)
    for g, head in enumerate(heads):
        mode, p = head
        c, s = (x[0] for x in _cos_sin([Q_POS], p))
        at, two = {"k1": ([p], [F(1)]), "k2": ([p + 64], [F(1)]), "dot": ([p, p + 1], [QA, QB]),
                   "q1": ([p, p + 64], [s, c]), "q2": ([p, p + 64], [-c, s])}[mode]
        for m in range(G):
            q[:, g * G + m, at] = np.asarray(two) * F(_sign(head, m, S) * (1.0 if mode == "dot" else _gain(head, S)))
    return synth.store(q, dtype)


def _case(monkeypatch, dtype, G, r, S, lens, top_k, tiles, n_sink=0, win=None, tiles_win=None, env=(), heads=KEYS):
    """win: (w, r_hi).  The staged call and the whole step, against each other bit for bit and against the logits above."""
    print(f"[case] rounding {dtype} G={G} r={r} S={S} lens={lens} k={n_sink}+{top_k} tiles={tiles} win={win} {tiles_win} {env}", flush=True)
    for k, v in env:
        monkeypatch.setenv(k, v)
    monkeypatch.setenv("SALS_TUNE_LOGITS", str(tiles))
    w = win[0] if win else 0
    B, H = len(lens), 8 * G
    ctx = binding.Sals(binding.make_desc(B, S, H, 8, D, r, top_k, dtype, n_recent=w, n_sink=n_sink), gu.DEV)
    pos = np.arange(S)
    rng = np.random.default_rng(S + r)
    V = rng.choice([-1.0, 1.0], size=(B, S, 64)) * (0.5 + rng.random((B, S, 1)))
    V = synth.widen(synth.store(V, dtype))
    Kc = np.stack([_rows(heads, pos, r, dtype)] * B)
    Vc = np.zeros((B, S, r)); Vc[:, :, :64] = V
    up = gu.to_dev
    q = up(_query(heads, B, G, S, dtype))
    q_pos = torch.full((B,), Q_POS if heads is QUERIES else 0, dtype=torch.int32, device=gu.DEV)
    seq_len = torch.tensor(lens, dtype=torch.int32, device=gu.DEV)
    W = ctx.pack_weights(up(_projector(heads, r, dtype)), up(_value_projector(r, dtype)))
    Kc, Vc = up(Kc), up(synth.store(Vc, dtype))
    idx = torch.full((B, ctx.k_tot), -7, dtype=torch.int32, device=gu.DEV)
    n_sel = torch.full((B,), -7, dtype=torch.int32, device=gu.DEV)
    odt = torch.bfloat16 if dtype == "bf16" else torch.float32
    out, out2 = (torch.empty((B, H, D), dtype=odt, device=gu.DEV) for _ in range(2))
    if win:
        monkeypatch.setenv("SALS_TUNE_LOGITS", str(tiles_win))
        r_hi = win[1]
        wc = binding.Sals(binding.make_desc(B, S, H, 8, D, r_hi, w, dtype, r_score=min(r_hi, 1024)), gu.DEV)
        Kw, Vw = np.zeros((B, w, r_hi), dtype=_rows(heads, [0], r_hi, dtype).dtype), np.zeros((B, w, r_hi))
        for b, n in enumerate(lens):
            t = np.arange(max(0, n - w), n)
            if len(t):
                Kw[b, t % w] = _rows(heads, t, r_hi, dtype)
                Vw[b, t % w, :64] = V[b, t]
        W_hi = wc.pack_weights(up(_projector(heads, r_hi, dtype)), up(_value_projector(r_hi, dtype)))
        Kw, Vw = up(Kw), up(synth.store(Vw, dtype))
        ctx.decode_step_window(wc, q, q_pos, Kc, Vc, W, Kw, Vw, W_hi, seq_len, out, None, idx, n_sel)
        ctx.sparse_attend_window(wc, q, q_pos, Kc, Vc, W, Kw, Vw, W_hi, idx, n_sel, out2)
    else:
        ctx.decode_step(q, q_pos, Kc, Vc, W, seq_len, out, None, idx, n_sel)
        ctx.sparse_attend(q, q_pos, Kc, Vc, W, idx, n_sel, out2)
    torch.cuda.synchronize()
    bits = (lambda t: t.view(torch.int16)) if dtype == "bf16" else (lambda t: t)
    same = torch.equal(bits(out), bits(out2))
    wrong = set()
    for which, o in (("step", out), ("staged", out2)):
        for b in range(B):
            t = idx[b, : int(n_sel[b])].cpu().numpy()
            for h in range(H):
                head = heads[h // G]
                x = _logits(head, t, S) * _sign(head, h % G, S)
                got = gu.from_dev(o[b, h])[:64]

                def y(x):
                    p = np.exp(x - x.max())
                    return (p / p.sum()) @ V[b, t]
                tol = 2.0 ** -7 * np.abs(y(x)).max() + 1e-4   # (bf16 weights and output)
                if head[0][0] == "k" or (t == 0).any():
                    assert min(np.abs(y(x) - y(k * x)).max() for k in (0.0, -1.0)) > 4 * tol, (head, x.min(), x.max())   # (the premise)
                if np.abs(got - y(x)).max() > tol:
                    others = [name for name, k in (("opposite", -1.0), ("both", 0.0)) if np.abs(got - y(k * x)).max() <= tol]
                    wrong.add((which, head, *others))
    ctx.close()
    if win:
        wc.close()
    assert not wrong, sorted(wrong)
    assert same


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("tiles", [1, 2])
def test_tiles_of_256_and_128_tokens(monkeypatch, tiles, G, dtype):
    _case(monkeypatch, dtype, G, 64, 300, [300], 300, tiles)


@pytest.mark.parametrize("dtype,r", [("bf16", 64 * n) for n in range(1, 11)] +
                         [("f32", r) for r in (64, 128, 192, 256, 320, 448, 576)])
def test_tiles_of_64_tokens_any_number_of_steps_ahead(monkeypatch, dtype, r):
    _case(monkeypatch, dtype, 2, r, 100, [100], 100, 3, env=[("SALS_TUNE_LOGITS_KSPLIT", "0")])


@pytest.mark.parametrize("dtype,r", [("f32", 192), ("f32", 320), ("f32", 704), ("bf16", 640), ("bf16", 1024)])
def test_tiles_of_64_tokens_with_a_split_latent_axis(monkeypatch, dtype, r):
    _case(monkeypatch, dtype, 4, r, 100, [100], 100, 3)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("G,slices", [(1, 1), (4, 1), (8, 1), (2, 1), (4, 2)])
def test_tiles_of_several_sequences(monkeypatch, G, slices, dtype):
    _case(monkeypatch, dtype, G, 128, 60, [60, 59, 40], 60, 4, env=[("SALS_TUNE_MULTI_KSPLIT", str(slices))])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tiles,G", [(1, 1), (1, 2), (1, 4), (1, 8), (2, 1), (2, 2), (2, 4), (2, 8)])
def test_ranking_the_threshold_bin(monkeypatch, tiles, G, dtype):
    _case(monkeypatch, dtype, G, 64, 33000, [33000], 200, tiles, n_sink=4)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tiles,r,G", [(1, 64, 1), (1, 64, 2), (1, 64, 4), (1, 64, 8), (2, 64, 1), (2, 64, 2), (2, 64, 4), (2, 64, 8)] +
                         [(3, 64 * n, 2) for n in range(1, 11)])
def test_beside_a_window_in_slices(monkeypatch, tiles, r, G, dtype):
    """The low-rank tiles add up the slices of a window in 64-token tiles, whose launch also selects."""
    _case(monkeypatch, dtype, G, r, 150, [150], 100, tiles, n_sink=4, win=(40, 1024), tiles_win=3)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("G,slices", [(1, 1), (2, 1), (4, 1), (8, 1), (4, 2)])
def test_beside_a_window_in_tiles_of_several_sequences(monkeypatch, G, slices, dtype):
    _case(monkeypatch, dtype, G, 64, 150, [150, 149, 120], 100, 2, n_sink=4, win=(40, 256), tiles_win=4,
          env=[("SALS_TUNE_MULTI_KSPLIT", str(slices))])


@pytest.mark.parametrize("r_hi", [64 * n for n in range(2, 11)])
def test_window_in_64_token_tiles_any_number_of_steps_ahead(monkeypatch, r_hi):
    _case(monkeypatch, "bf16", 2, 64, 150, [150], 100, 2, n_sink=4, win=(40, r_hi), tiles_win=3, env=[("SALS_TUNE_LOGITS_KSPLIT", "0")])


@pytest.mark.parametrize("tiles,win", [(1, False), (2, False), (3, False), (4, False), (2, True)])
def test_rotated_queries(monkeypatch, tiles, win):
    _case(monkeypatch, "f32", 4, 128, 150 if win else 60, [150 if win else 60], 60, tiles, n_sink=4 if win else 0,
          win=(40, 256) if win else None, tiles_win=3, heads=QUERIES)
