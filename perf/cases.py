"""Calls a serving or calibration program makes into this package, with their inputs.

Kinds of cases:
  decode   one decode step of one or more layers: optionally the append of the new token, then the sparse attention over
           the latent key cache, with latent or quantised values and with or without the high-precision recent window
  dense    dense decode attention (the layers that are left uncompressed, and the baseline)
  prefill  the prompt compressed into the latent caches
  cov      calibration: one batch of keys added to the covariance
  eig      calibration: the leading eigenvectors of a covariance

Caches hold N(0, 1) entries under the spectrum (c+1)^-1/2 of the latent coordinate, scaled so that the attention logits
have unit variance, with a few tokens per sequence aligned with the query; projectors have near-orthonormal columns.
"""
from __future__ import annotations

import math

import torch

from paper_2510_24273_amd import binding

DEV = "cuda:0"
HEAD = 128
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _decode(name=None, **kw):
    c = dict(kind="decode", dtype="bf16", B=1, S=4096, len=4096, ragged=False, H=32, H_kv=32, r=640, rs=640, top_k=512, sink=0,
             recent=0, bits=0, r_hi=0, style=0, theta=10000.0, append=False, layers=1)
    c.update(kw)
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # a short single sequence in full precision: latency and launches are all there is
        _decode("decode_f32_b1_1k", dtype="f32", S=1024, len=1024, r=512, rs=512, top_k=128),
        # interactive use: one sequence of a 7B-class multi-head model; several layers, as a model walks them
        _decode("decode_b1_4k_layers8", layers=8),
        # batch serving of the same model
        _decode("decode_b16_4k", B=16),
        # batch serving of a grouped-query model: sequences of different lengths in caches with room, token appended first
        _decode("step_b12_gqa_ragged", B=12, S=6002, len=5500, ragged=True, H_kv=8, top_k=432, sink=16, recent=64, append=True),
        # long contexts, multi-head
        _decode("decode_b4_32k", B=4, S=32768, len=32768, top_k=2048),
        # one very long context, grouped-query
        _decode("decode_b1_128k_gqa", S=131072, len=131072, H_kv=8, r=512, rs=512, top_k=4096, recent=64, theta=500000.0),
        # the whole mixed-precision setting: low-rank keys scored on their leading half, 2-bit values, the recent tokens at
        # higher rank and 8 bits; token appended first
        _decode("step_qv2_window_b16_4k", B=16, S=4224, len=4096, r=512, rs=256, top_k=432, sink=16, recent=64, bits=2, r_hi=2048,
                append=True),
        # the recent window over latent values, one sequence
        _decode("decode_window_b1_4k", top_k=432, sink=16, recent=64, r_hi=2048),
        # a layer that stays dense
        dict(name="dense_b8_2k", kind="dense", dtype="bf16", B=8, S=2048, len=2048, ragged=False, H=32, H_kv=32, style=0,
             theta=10000.0),
        # a batch of prompts of different lengths
        dict(name="prefill_b6_gqa_4k", kind="prefill", dtype="bf16", B=6, n_tok=4001, ragged=True, H_kv=8, r=640),
        # calibration: eight sequences of keys, then a model's eigenvectors
        dict(name="calib_covariance_d4096", kind="cov", dtype="bf16", D=4096, n_tok=32768),
        dict(name="calib_eigenvectors_d1024", kind="eig", dtype="bf16", D=1024, r=640),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 8 + ["dense", "prefill", "cov", "eig"])
    if kind == "eig":
        D = 256 * rng.randint(1, 4)
        return dict(kind="eig", dtype=rng.choice(["bf16", "f32"]), D=D, r=max(64, min(640, rng.randint(1, D // 64) * 64)))
    if kind == "cov":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        return dict(kind="cov", dtype=dtype, D=128 * rng.randint(2, 32 if dtype == "bf16" else 8), n_tok=_log_int(rng, 500, 32768))
    H_kv = rng.choice([32, 32, 8])
    if kind == "prefill":
        B = rng.randint(1, 6)
        return dict(kind="prefill", dtype="bf16", B=B, n_tok=_log_int(rng, 64, 24000 // B if H_kv == 8 else 6000 // B),
                    ragged=rng.random() < 0.5, H_kv=H_kv, r=64 * rng.randint(4, 16))
    B = _log_int(rng, 1, 16)
    if kind == "dense":
        S = _log_int(rng, 256, 65536 // B)
        return dict(kind="dense", dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), B=B, S=S, len=S, ragged=rng.random() < 0.5, H=32,
                    H_kv=8 if S * B > 16384 else H_kv, style=rng.randint(0, 1), theta=10000.0)
    dtype = rng.choice(["bf16"] * 7 + ["f32"])
    S = _log_int(rng, 512, 131072 // B if dtype == "bf16" else 16384 // B)
    r = 64 * rng.randint(4, 10) if rng.random() < 0.8 else 1024
    if r == 1024:
        S = min(S, 65536 // B)
    append = rng.random() < 0.5
    longest = S - 1 if append else S
    if rng.random() < 0.4:
        longest = max(1, int(longest * rng.uniform(0.5, 1.0)))
    # one token in 8 to one in 32 attended, within what the largest batch reconstructs
    budget = (16 * 512 * 640 if dtype == "bf16" else 512 * 640) // (B * r)
    recent = rng.choice([0, 64, 64])
    sink = 16 if recent else 0
    top_k = max(48, min(longest // rng.choice([8, 16, 32]), 4096, budget) - recent - sink)
    bits = rng.choice([0, 0, 4, 2])
    return _decode(dtype=dtype, B=B, S=S, len=longest, ragged=B > 1 and rng.random() < 0.5, H_kv=H_kv, r=r,
                   rs=rng.choice([r, r // 2]), top_k=top_k, sink=sink, recent=recent, bits=bits,
                   r_hi=HEAD * H_kv // 2 if recent and r < HEAD * H_kv // 2 and rng.random() < 0.4 else 0,
                   style=rng.randint(0, 1), theta=rng.choice([10000.0, 500000.0]), append=append)


def _lengths(c):
    """Sequence b of a ragged batch is shorter by b / (2 B) of the longest one."""
    return [c["len"] - (b * c["len"] // (2 * c["B"]) if c["ragged"] else 0) for b in range(c["B"])]


class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, *shape, dtype=torch.float32):
        return torch.randn(shape, generator=self.g, device=DEV, dtype=dtype)

    def codes(self, *shape):
        return torch.randint(0, 256, shape, generator=self.g, device=DEV, dtype=torch.uint8)

    def projector(self, D, r, dt):
        return (self.normal(D, r) * D ** -0.5).to(dt)


def _spectrum(r, D):
    s = torch.arange(1, r + 1, device=DEV, dtype=torch.float32) ** -0.5
    return s * math.sqrt(D / float((s * s).sum()))


def _cache(R, B, S, r, D, dt):
    """[B, S, r] latent rows."""
    out = torch.empty((B, S, r), dtype=dt, device=DEV)
    s = _spectrum(r, D)
    for b in range(B):
        out[b] = R.normal(S, r).mul_(s).to(dt)
    return out


def _meta(R, B, S, D, bits, dt):
    """(scale, zero) of the value groups, the ranges unit-variance groups of 32 channels have."""
    scale = (R.normal(B, S, D // 32).abs_() + 0.05) * (4.0 / ((1 << bits) - 1))
    zero = R.normal(B, S, D // 32) * 0.5 - 2.0
    return torch.stack([scale, zero], dim=-1).to(dt)


def _prepare_decode(c, R):
    dt, B, S, D, r = DTYPES[c["dtype"]], c["B"], c["S"], c["H_kv"] * HEAD, c["r"]
    lens = torch.tensor(_lengths(c), dtype=torch.int32)
    ctx = binding.Sals(binding.make_desc(B, S, c["H"], c["H_kv"], HEAD, r, c["top_k"], c["dtype"], r_score=c["rs"],
                                         n_recent=c["recent"], n_sink=c["sink"], rope_theta=c["theta"], rope_style=c["style"]), DEV)
    win = None
    if c["r_hi"]:
        win = binding.Sals(binding.make_desc(B, S, c["H"], c["H_kv"], HEAD, c["r_hi"], c["recent"], c["dtype"],
                                             r_score=min(c["r_hi"], 1024), rope_theta=c["theta"], rope_style=c["style"]), DEV)
    layers = []
    for _ in range(c["layers"]):
        L = {"q": R.normal(B, c["H"], HEAD).to(dt), "Kc": _cache(R, B, S, r, D, dt)}
        Uk = R.projector(D, r, dt)
        # three tokens of each sequence lie along the query's latent image, far above the other scores
        qt = L["q"].float().view(B, c["H_kv"], -1, HEAD).sum(dim=2).view(B, D) @ Uk.float()
        spread = (qt * _spectrum(r, D)).norm(dim=1, keepdim=True)
        aligned = (10.0 * spread / (qt * qt).sum(dim=1, keepdim=True) * qt).to(dt)
        for b in range(B):
            at = torch.randint(0, int(lens[b]), (3,), generator=R.g, device=DEV)
            L["Kc"][b, at] += aligned[b]
        L["W"] = ctx.pack_weights(Uk, R.projector(D, r, dt))
        if c["bits"]:
            L["Vq"], L["Vmeta"] = R.codes(B, S, D * c["bits"] // 8), _meta(R, B, S, D, c["bits"], dt)
        else:
            L["Vc"] = _cache(R, B, S, r, D, dt)
        if win is not None:
            L["W_hi"] = win.pack_weights(R.projector(D, c["r_hi"], dt), R.projector(D, c["r_hi"], dt))
            L["Kw"] = _cache(R, B, c["recent"], c["r_hi"], D, dt)
            if c["bits"]:
                L["Vqw"], L["Vmeta_w"] = R.codes(B, c["recent"], D), _meta(R, B, c["recent"], D, 8, dt)
            else:
                L["Vw"] = _cache(R, B, c["recent"], c["r_hi"], D, dt)
        if c["append"]:
            L["k_new"], L["v_new"] = R.normal(B, D).to(dt), R.normal(B, D).to(dt)
        L["seq_len"] = lens.to(DEV)
        L["out"] = torch.empty((B, c["H"], HEAD), dtype=dt, device=DEV)
        layers.append(L)
    lens = lens.to(DEV)
    return {"case": c, "ctx": ctx, "win": win, "layers": layers, "len0": lens, "q_pos": lens.clone()}


def _run_decode(s):
    c, ctx, win, q_pos, outs = s["case"], s["ctx"], s["win"], s["q_pos"], []
    bits = c["bits"]
    for L in s["layers"]:
        kept = {}
        if c["append"]:
            # (the previous pass's token is taken back, as after a rejected draft of speculative decoding)
            L["seq_len"].copy_(s["len0"])
            if bits:
                if win is not None:
                    win.window_append_qv(L["k_new"], L["v_new"], L["W_hi"], L["Kw"], L["Vqw"], L["Vmeta_w"], L["seq_len"])
                    kept.update(Kw=L["Kw"], Vqw=L["Vqw"], Vmeta_w=L["Vmeta_w"])
                ctx.compress_append_qv(L["k_new"], L["v_new"], L["W"], L["Kc"], L["Vq"], L["Vmeta"], bits, L["seq_len"])
                kept.update(Kc=L["Kc"], Vq=L["Vq"], Vmeta=L["Vmeta"], seq_len=L["seq_len"])
            else:
                if win is not None:
                    win.window_append(L["k_new"], L["v_new"], L["W_hi"], L["Kw"], L["Vw"], L["seq_len"])
                    kept.update(Kw=L["Kw"], Vw=L["Vw"])
                ctx.compress_append(L["k_new"], L["v_new"], L["W"], L["Kc"], L["Vc"], L["seq_len"])
                kept.update(Kc=L["Kc"], Vc=L["Vc"], seq_len=L["seq_len"])
        if bits and win is not None:
            ctx.decode_step_qv_window(win, L["q"], q_pos, L["Kc"], L["Vq"], L["Vmeta"], bits, L["W"], L["Kw"], L["Vqw"],
                                      L["Vmeta_w"], L["W_hi"], L["seq_len"], L["out"])
        elif bits:
            ctx.decode_step_qv(L["q"], q_pos, L["Kc"], L["Vq"], L["Vmeta"], bits, L["W"], L["seq_len"], L["out"])
        elif win is not None:
            ctx.decode_step_window(win, L["q"], q_pos, L["Kc"], L["Vc"], L["W"], L["Kw"], L["Vw"], L["W_hi"], L["seq_len"], L["out"])
        else:
            ctx.decode_step(L["q"], q_pos, L["Kc"], L["Vc"], L["W"], L["seq_len"], L["out"])
        outs.append(dict(out=L["out"], **kept))
    return outs


def _prepare_dense(c, R):
    dt, B, S = DTYPES[c["dtype"]], c["B"], c["S"]
    ctx = binding.Sals(binding.make_desc(B, S, c["H"], c["H_kv"], HEAD, 512, 512, c["dtype"], rope_theta=c["theta"],
                                         rope_style=c["style"]), DEV)
    lens = torch.tensor(_lengths(c), dtype=torch.int32, device=DEV)
    return {"case": c, "ctx": ctx, "q": R.normal(B, c["H"], HEAD).to(dt), "K": R.normal(B, S, c["H_kv"], HEAD, dtype=dt),
            "V": R.normal(B, S, c["H_kv"], HEAD, dtype=dt), "len": lens, "out": torch.empty((B, c["H"], HEAD), dtype=dt, device=DEV)}


def _run_dense(s):
    s["ctx"].dense_attend(s["q"], s["len"], s["K"], s["V"], s["len"], s["out"])
    return s["out"]


def _prompt_lengths(c):
    return [c["n_tok"] - (b * c["n_tok"] // (2 * c["B"]) if c["ragged"] else 0) for b in range(c["B"])]


def _prepare_prefill(c, R):
    dt, B, D, r, n = DTYPES[c["dtype"]], c["B"], c["H_kv"] * HEAD, c["r"], c["n_tok"]
    ctx = binding.Sals(binding.make_desc(B, n, 32, c["H_kv"], HEAD, r, 512, c["dtype"]), DEV)
    s = {"case": c, "ctx": ctx, "W": ctx.pack_weights(R.projector(D, r, dt), R.projector(D, r, dt)),
         "k": R.normal(B, n, D, dtype=dt), "v": R.normal(B, n, D, dtype=dt), "Kc": torch.zeros((B, n, r), dtype=dt, device=DEV),
         "Vc": torch.zeros((B, n, r), dtype=dt, device=DEV), "seq_len": torch.zeros(B, dtype=torch.int32, device=DEV), "n_new": None}
    if c["ragged"]:
        s["n_new"] = torch.tensor(_prompt_lengths(c), dtype=torch.int32, device=DEV)
    return s


def _run_prefill(s):
    s["seq_len"].zero_()
    s["ctx"].compress_prefill(s["k"], s["v"], s["W"], s["Kc"], s["Vc"], s["seq_len"], s["case"]["n_tok"], s["n_new"])
    return {"Kc": s["Kc"], "Vc": s["Vc"], "seq_len": s["seq_len"]}


def _keys(R, n, D, dt):
    """Keys with a decaying spectrum along directions that mix all channels."""
    sigma = torch.arange(1, D + 1, device=DEV, dtype=dt) ** -0.5
    return (R.normal(n, D, dtype=dt) * sigma) @ (R.normal(D, D, dtype=dt) * D ** -0.5)


def _prepare_cov(c, R):
    return {"case": c, "keys": _keys(R, c["n_tok"], c["D"], torch.float32).to(DTYPES[c["dtype"]]),
            "C": torch.zeros((c["D"], c["D"]), dtype=torch.float64, device=DEV)}


def _run_cov(s):
    # (batch after batch is added to the same matrix)
    s["workspace"] = binding.calib_accumulate(s["keys"], s["C"])
    return s["C"]


def _prepare_eig(c, R):
    X = _keys(R, 4 * c["D"], c["D"], torch.float64)
    C = X.T.contiguous() @ X
    return {"case": c, "C": (C + C.T) * 0.5}


def _run_eig(s):
    c = s["case"]
    # (the call overwrites its matrix, which the calibration keeps for the captured energy)
    eigval, U, _ = binding.calib_eigenvectors(s["C"].clone(), c["r"], DTYPES[c["dtype"]])
    return {"eigval": eigval[: c["r"]], "U": U}  # (the values past the r-th are rough estimates by definition)


_PREPARE = {"decode": _prepare_decode, "dense": _prepare_dense, "prefill": _prepare_prefill, "cov": _prepare_cov, "eig": _prepare_eig}
_RUN = {"decode": _run_decode, "dense": _run_dense, "prefill": _run_prefill, "cov": _run_cov, "eig": _run_eig}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, _Rand(seed))


def run(state):
    return _RUN[state["case"]["kind"]](state)


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "eig":  # reduction to tridiagonal form and the r vectors carried back
        D, r = c["D"], c["r"]
        return {"bytes": D * D * 8 + D * r * e + r * 8, "flops": 4 * D ** 3 // 3 + 2 * D * D * r}
    if c["kind"] == "cov":  # the upper triangle
        D, n = c["D"], c["n_tok"]
        return {"bytes": n * D * e + 2 * D * D * 8, "flops": n * D * (D + 1)}
    D = c["H_kv"] * HEAD
    if c["kind"] == "prefill":
        n, r = sum(_prompt_lengths(c)), c["r"]
        return {"bytes": 2 * (n * (D + r) + D * r) * e, "flops": 4 * n * D * r}
    B, H, lens = c["B"], c["H"], _lengths(c)
    if c["kind"] == "dense":
        return {"bytes": (2 * sum(lens) * D + 2 * B * H * HEAD) * e, "flops": 4 * H * HEAD * sum(lens)}
    r, rs, r_hi = c["r"], c["rs"], c["r_hi"]
    new = 1 if c["append"] else 0
    k_tot = c["top_k"] + c["sink"] + c["recent"]
    n_sel = sum(min(n + new, k_tot) for n in lens)
    n_hi = sum(min(n + new, c["recent"]) for n in lens) if r_hi else 0
    n_lo = n_sel - n_hi
    val = r * e if not c["bits"] else D * c["bits"] // 8 + D // 32 * 2 * e       # a value row
    val_hi = r_hi * e if not c["bits"] else D + D // 32 * 2 * e
    proj = 1 if c["bits"] else 2                                                 # projectors that are read
    byts = 2 * B * H * HEAD * e + sum(lens) * rs * e + n_lo * (r * e + val) + n_hi * (r_hi * e + val_hi) + proj * D * (r + r_hi) * e
    # query projection, scores, keys of the selection, logits, values
    flops = 2 * B * D * r + 2 * sum(lens) * rs + 2 * D * (n_lo * r + n_hi * r_hi) + 2 * H * HEAD * n_sel
    flops += 2 * H * HEAD * n_sel if c["bits"] else 2 * H * (n_lo * r + n_hi * r_hi) + 2 * B * H * HEAD * (r + r_hi)
    if new:
        byts += 2 * B * D * e + B * (r * e + val + (r_hi * e + val_hi if r_hi else 0))
        flops += 2 * proj * B * D * (r + r_hi)
    return {"bytes": c["layers"] * byts, "flops": c["layers"] * flops}


def tolerance(case):
    """bf16 results: one rounding of an fp32 sum whose order is free; fp32 results: that order."""
    if case["kind"] == "cov":
        return {"rel": 1e-5, "max": 1e-4}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    return {"rel": 5e-3, "max": 3e-2}
