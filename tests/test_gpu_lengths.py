"""Lengths advanced by the last workgroup of an append or a prompt compression: rows, codes and lengths against a context that was
never prepared, whose lengths a second launch advances, bit for bit, call after call and in replays of a captured graph.  Shapes: batches at the edges of a
wave's lanes, full caches, sequences without new tokens, grids with workgroups that have nothing to do.  (Batches of 64 and 128 sequences have no room for
a count of arrivals: there a second launch advances the lengths of either context.)"""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2510_24273_amd import binding  # noqa: E402

DEV = "cuda:0"


def _unprepared(desc):
    c = binding.Sals.__new__(binding.Sals)
    c.desc, c.device = desc, torch.device(DEV)
    nbytes = binding.workspace_bytes(desc)
    c.workspace = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device=DEV)
    c._h = ctypes.c_void_p()
    assert binding._lib.sals_create(ctypes.byref(desc), c.workspace.data_ptr(), nbytes, ctypes.byref(c._h)) == 0
    c._destroy = binding._lib.sals_destroy
    return c


def _contexts(*a, **kw):
    return [binding.Sals(binding.make_desc(*a, **kw), DEV), _unprepared(binding.make_desc(*a, **kw))]


def _rand(gen, dtype, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).to(dtype)


@pytest.mark.parametrize("dtype,B,bits", [("bf16", 1, 0), ("bf16", 64, 0), ("bf16", 65, 4), ("bf16", 128, 0), ("bf16", 12, 2),
                                          ("f32", 17, 0), ("f32", 128, 4), ("bf16", 63, 0), ("bf16", 127, 2), ("f32", 127, 4), ("f32", 63, 0)])
def test_append(dtype, B, bits):
    print(f"[case] append {dtype} B={B} bits={bits}", flush=True)
    S, H_kv, r = 9, 4, 128
    D, dt = H_kv * 128, torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=DEV).manual_seed(B)
    Uk, Uv = _rand(g, dt, D, r), _rand(g, dt, D, r)
    new = [(_rand(g, dt, B, D), _rand(g, dt, B, D)) for _ in range(4)]
    start = torch.tensor([(3 * b + 5) % (S + 1) for b in range(B)], dtype=torch.int32, device=DEV)  # (some are full)
    results = []
    for ctx in _contexts(B, S, H_kv, H_kv, 128, r, 4, dtype):
        W = ctx.pack_weights(Uk, Uv)
        state = [torch.zeros((B, S, r), dtype=dt, device=DEV), start.clone()]
        if bits:
            state += [torch.zeros((B, S, D * bits // 8), dtype=torch.uint8, device=DEV), torch.zeros((B, S, D // 32, 2), dtype=dt, device=DEV)]
        else:
            state.append(torch.zeros((B, S, r), dtype=dt, device=DEV))
        for k, v in new:
            if bits:
                ctx.compress_append_qv(k, v, W, state[0], state[2], state[3], bits, state[1])
            else:
                ctx.compress_append(k, v, W, state[0], state[2], state[1])
        torch.cuda.synchronize()
        results.append(state)
    assert torch.equal(results[0][1], torch.clamp(start + len(new), max=S))
    for x, y in zip(*results):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,B,n_tok,r,counts", [
    ("bf16", 3, 130, 192, [130, 0, 77]), ("bf16", 2, 64, 64, None), ("bf16", 65, 40, 64, [(7 * b) % 41 for b in range(65)]),
    ("bf16", 6, 1001, 640, [1001, 900, 0, 513, 256, 1]), ("bf16", 4, 2600, 640, None), ("f32", 3, 300, 128, [300, 0, 129]),
    ("bf16", 63, 40, 64, [(7 * b) % 41 for b in range(63)]), ("bf16", 127, 33, 64, [(5 * b) % 34 for b in range(127)]),
    ("f32", 127, 20, 64, [(3 * b) % 21 for b in range(127)])])
def test_prompt(dtype, B, n_tok, r, counts):
    print(f"[case] prompt {dtype} B={B} n_tok={n_tok} r={r} counts={counts}", flush=True)
    H_kv = 4
    D, S, dt = H_kv * 128, 2 * n_tok - 3, torch.bfloat16 if dtype == "bf16" else torch.float32   # (the second call overruns)
    g = torch.Generator(device=DEV).manual_seed(n_tok)
    Uk, Uv, k, v = _rand(g, dt, D, r), _rand(g, dt, D, r), _rand(g, dt, B, n_tok, D), _rand(g, dt, B, n_tok, D)
    n_new = None if counts is None else torch.tensor(counts, dtype=torch.int32, device=DEV)
    results = []
    for ctx in _contexts(B, S, H_kv, H_kv, 128, r, 4, dtype):
        W = ctx.pack_weights(Uk, Uv)
        Kc, Vc = torch.zeros((B, S, r), dtype=dt, device=DEV), torch.zeros((B, S, r), dtype=dt, device=DEV)
        seq_len = torch.zeros(B, dtype=torch.int32, device=DEV)
        for _ in range(2):
            ctx.compress_prefill(k, v, W, Kc, Vc, seq_len, n_tok, n_new)
        torch.cuda.synchronize()
        results.append([Kc, Vc, seq_len])
    want = [min(2 * (n_tok if counts is None else counts[b]), S) for b in range(B)]
    assert results[0][2].tolist() == want
    for x, y in zip(*results):
        assert torch.equal(x, y)


def test_captured():
    B, S, H_kv, r, n_tok = 5, 400, 4, 64, 37
    D = H_kv * 128
    print(f"[case] captured prompt and append B={B}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(7)
    dt = torch.bfloat16
    ctx = binding.Sals(binding.make_desc(B, S, H_kv, H_kv, 128, r, 4, "bf16"), DEV)
    W = ctx.pack_weights(_rand(g, dt, D, r), _rand(g, dt, D, r))
    k, v = _rand(g, dt, B, n_tok, D), _rand(g, dt, B, n_tok, D)
    k1, v1 = k[:, 0].contiguous(), v[:, 0].contiguous()
    n_new = torch.tensor([37, 0, 20, 1, 36], dtype=torch.int32, device=DEV)

    def step(Kc, Vc, seq_len):
        ctx.compress_prefill(k, v, W, Kc, Vc, seq_len, n_tok, n_new)
        ctx.compress_append(k1, v1, W, Kc, Vc, seq_len)

    def buffers():
        return [torch.zeros((B, S, r), dtype=dt, device=DEV), torch.zeros((B, S, r), dtype=dt, device=DEV),
                torch.zeros(B, dtype=torch.int32, device=DEV)]

    eager, played = buffers(), buffers()
    step(*buffers())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(*played)
    for t in played:
        t.zero_()
    for i in range(4):
        step(*eager)
        graph.replay()
        torch.cuda.synchronize()
        assert played[2].tolist() == [(i + 1) * (int(n) + 1) for n in n_new]
        for x, y in zip(eager, played):
            assert torch.equal(x, y), i
