"""GPU parity of the offline calibration (Sec. 4.2) through the C ABI: the covariance against the fp64 oracle element
by element, the eigen-decomposition against the oracle's on the same matrix (eigenvalues, eigenvectors up to sign,
orthonormality, the defining equation), the cases where eigenvectors are not unique through what is, and the whole
step through the captured energy of Lemma 1."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2510_24273_amd import binding, synth
from tests import gpu_util as gu
from oracle import calibration_oracle as cal

pytestmark = pytest.mark.gpu


def _cov_gpu(X_store, split=None):
    n, D = X_store.shape
    C = torch.zeros(D, D, dtype=torch.float64, device=gu.DEV)
    X = gu.to_dev(X_store)
    keep = []
    parts = [(0, n)] if split is None else [(0, split), (split, n)]
    for a, b in parts:
        keep.append(binding.calib_accumulate(X[a:b].contiguous(), C))
    torch.cuda.synchronize()
    return C


def _check_cov(C_gpu, X_store, chunk_tokens=4096):
    Xd = synth.widen(X_store)
    C_ref = cal.covariance(Xd)
    got = C_gpu.cpu().numpy()
    dg = np.sqrt(np.diag(C_ref))
    # products of stored values are exact in fp32; a chunk's sum of at most 4096 of them carries at most
    # 4096 * 2^-24 relative to sum |x_i x_j| <= sqrt(C_ii C_jj); typical error is the square root of that count
    bound = 2e-5 * np.outer(dg, dg) + 1e-30
    err = np.abs(got - C_ref)
    assert np.all(err <= bound), float(np.max(err / bound))
    assert np.array_equal(got, got.T) or np.max(np.abs(got - got.T)) <= 1e-6 * np.max(dg) ** 2
    return C_ref


@pytest.mark.parametrize("dtype,D,n", [("bf16", 256, 1000), ("bf16", 512, 9001), ("f32", 256, 4200),
                                        ("bf16", 1024, 5000), ("bf16", 2048, 300), ("bf16", 128, 64), ("f32", 384, 1)])
def test_covariance_matches_the_oracle(dtype, D, n):
    print(f"[case] covariance {dtype} D={D} n={n}", flush=True)
    X = synth.make_calibration_keys(100 + D + n, n, D, dtype, decay=0.98)
    C = _cov_gpu(X)
    _check_cov(C, X)


@pytest.mark.parametrize("D,n", [(384, 33), (128, 4097), (1152, 31), (8192, 8250)])
def test_covariance_tile_and_slice_remainders(D, n):
    """Widths that are no whole number of tiles, token counts one past a step or a slice, more tokens than one launch
    takes; against fp64 products on the device."""
    print(f"[case] covariance remainders D={D} n={n}", flush=True)
    g = torch.Generator(device=gu.DEV)
    g.manual_seed(D + n)
    X = torch.randn(n, D, generator=g, device=gu.DEV, dtype=torch.bfloat16)
    C = torch.randn(D, D, generator=g, device=gu.DEV, dtype=torch.float64)
    want = torch.triu(C)
    want = want + torch.triu(want, 1).T + X.double().T.contiguous() @ X.double()
    ws = binding.calib_accumulate(X, C)
    torch.cuda.synchronize()
    dg = want.diagonal().abs().sqrt()
    assert bool(((C - want).abs() <= 2e-5 * torch.outer(dg, dg) + 1e-9).all())
    assert torch.equal(C, C.T)


@pytest.mark.parametrize("D,n", [(4096, 4096), (3968, 12001), (4096, 9000)])
def test_covariance_with_additions_beside_the_last_round(D, n):
    """Batches whose tiles take whole rounds of the chip and a part: the part's launch also adds up the others."""
    test_covariance_tile_and_slice_remainders(D, n)


def test_covariance_accumulates_over_calls():
    print("[case] covariance in two calls", flush=True)
    X = synth.make_calibration_keys(7, 6000, 256, "bf16", decay=0.95)
    C = _cov_gpu(X, split=1777)
    _check_cov(C, X)


def _same_up_to_sign(a, b, tol):
    worst = 0.0
    for i in range(a.shape[1]):
        worst = max(worst, min(np.max(np.abs(a[:, i] - b[:, i])), np.max(np.abs(a[:, i] + b[:, i]))))
    assert worst <= tol, worst


def _eig_gpu(C_np, r, dtype=torch.float32, max_sweeps=80):
    C = torch.from_numpy(np.ascontiguousarray(C_np)).to(gu.DEV)
    lam, U, sweeps = binding.calib_eigenvectors(C, r, dtype, max_sweeps)
    torch.cuda.synchronize()
    return lam.cpu().numpy(), gu.from_dev(U), sweeps


@pytest.mark.parametrize("D,r,decay", [(256, 64, 0.9), (512, 128, 0.95), (256, 256, 0.97)])
def test_eigenvectors_match_the_oracle_on_a_separated_spectrum(D, r, decay):
    print(f"[case] eigenvectors D={D} r={r}", flush=True)
    X = synth.widen(synth.make_calibration_keys(11 + D, 4 * D, D, "f32", decay=decay))
    C = cal.covariance(X)
    lam_ref, U_ref = cal.leading_eigenvectors(C, r)
    lam, U, sweeps = _eig_gpu(C, r)
    assert 0 < sweeps <= 60, sweeps
    print('    sweeps', sweeps, flush=True)
    np.testing.assert_allclose(lam[:r], lam_ref[:r], rtol=0, atol=1e-11 * lam_ref[0])
    np.testing.assert_allclose(lam, lam_ref, rtol=0, atol=1e-3 * lam_ref[0])
    np.testing.assert_allclose(lam[:r], lam_ref[:r], rtol=1e-8)
    # eigenvectors: fp64 on both sides, stored as fp32 by the GPU: half an ulp of fp32 plus the conditioning
    # (1e-16 * lambda_0 / gap, gaps of at least a few percent of lambda_i)
    _same_up_to_sign(U, U_ref, 2e-7)
    np.testing.assert_allclose(U.T @ U, np.eye(r), atol=5e-7)
    resid = C @ U - U * lam[:r]
    assert np.max(np.abs(resid)) <= 5e-7 * lam_ref[0]
    # sign convention: the largest component of every column is positive
    big = U[np.argmax(np.abs(U), axis=0), np.arange(r)]
    assert np.all(big > 0)


@pytest.mark.parametrize("D,r", [(256, 256), (768, 300), (1280, 200)])
def test_eigenvectors_at_widths_of_uneven_column_slices(D, r):
    """Widths whose 32-row blocks make an uneven number of pairs and whose column slices are not powers of two, with a spectrum
    that several sweeps work on."""
    print(f"[case] eigenvectors D={D} r={r}, slow decay", flush=True)
    rng = np.random.default_rng(D)
    Q, _ = np.linalg.qr(rng.standard_normal((D, D)))
    lam_true = 1.0 / np.arange(1, D + 1)
    C = (Q * lam_true) @ Q.T
    C = 0.5 * (C + C.T)
    lam_ref, U_ref = cal.leading_eigenvectors(C, r)
    lam, U, sweeps = _eig_gpu(C, r)
    assert 0 < sweeps <= 30, sweeps
    np.testing.assert_allclose(lam[:r], lam_ref[:r], rtol=0, atol=1e-11 * lam_ref[0])
    # vectors: half an ulp of fp32, plus 1e-15 lambda_0 over the smallest gap (1 / r^2)
    _same_up_to_sign(U, U_ref, 2e-7)
    np.testing.assert_allclose(U.T @ U, np.eye(r), atol=5e-7)


@pytest.mark.parametrize("D,r,decay", [(256, 256, 0.5), (512, 200, 1.0), (768, 768, 0.25)])
def test_rows_left_behind_are_orthogonal_in_fp64(D, r, decay):
    """What the call leaves in C, eigenvalue times eigenvector by row, before the vectors are rounded to their storage type:
    orthogonal and solving the defining equation to fp64, also where the last rotations are made all at once (flat spectra, whose
    smallest gaps keep the angles large for long)."""
    print(f"[case] eigenvector rows in fp64, D={D} r={r}", flush=True)
    rng = np.random.default_rng(2 * D)
    X = rng.standard_normal((4 * D, D)) * np.arange(1, D + 1) ** -decay
    C = X.T @ X
    C = 0.5 * (C + C.T)
    Cg = gu.to_dev(C)
    lam, U, sweeps = binding.calib_eigenvectors(Cg, r, torch.float32)
    torch.cuda.synchronize()
    assert 0 < sweeps <= 30, sweeps
    rows = Cg.cpu().numpy()
    norm = np.linalg.norm(rows, axis=1)
    lead = np.argsort(-norm)[:r]
    V = rows[lead] / norm[lead, None]
    # sums of D products: a few 1e-16 sqrt(D), and the angles the call may leave (1e-11)
    assert np.max(np.abs(V @ V.T - np.eye(r))) <= 2e-11
    assert np.max(np.linalg.norm(V @ C - norm[lead, None] * V, axis=1)) <= 2e-11 * norm[lead[0]]
    np.testing.assert_allclose(norm[lead], lam.cpu().numpy()[:r], rtol=1e-13)


@pytest.mark.parametrize("D,r,kind", [(256, 256, "flat"), (512, 512, "repeated"), (512, 300, "shuffled"), (768, 100, "steep"),
                                      (1280, 700, "slow"), (1536, 1536, "flat"), (2304, 128, "slow"), (3072, 64, "slow"), (3584, 1000, "flat")])
def test_transformations_of_all_rows_at_once(D, r, kind):
    """Spectra on which the call transforms all rows at once, from the first sweep on and (D above 2048) later, and such on which the
    transformations gain little and sweeps take turns with them: eigenvalues that repeat, rows of very different norms in no order."""
    print(f"[case] transformations of all rows, D={D} r={r} {kind}", flush=True)
    rng = np.random.default_rng(7 * D + r)
    if kind == "repeated":
        Q, _ = np.linalg.qr(rng.standard_normal((D, D)))
        C = (Q * np.repeat(1.0 / np.arange(1, D // 16 + 1), 16)) @ Q.T
    else:
        X = rng.standard_normal((4 * D, D))
        if kind == "shuffled":
            X = (X @ (np.eye(D) + 0.3 / np.sqrt(D) * rng.standard_normal((D, D))) * 10.0 ** -np.linspace(0.0, 5.0, D))[:, rng.permutation(D)]
        else:
            X = X * np.arange(1, D + 1) ** -{"flat": 0.25, "slow": 0.5, "steep": 1.5}[kind] @ rng.standard_normal((D, D)) / np.sqrt(D)
        C = X.T @ X
    C = 0.5 * (C + C.T)
    lam_ref = np.linalg.eigvalsh(C)[::-1]
    Cg = gu.to_dev(C)
    lam, U, sweeps = binding.calib_eigenvectors(Cg, r, torch.float32)
    torch.cuda.synchronize()
    assert 0 < sweeps <= 40, sweeps
    rows = Cg.cpu().numpy()
    norm = np.linalg.norm(rows, axis=1)
    lead = np.argsort(-norm)[:r]
    V = rows[lead] / norm[lead, None]
    assert np.max(np.abs(V @ V.T - np.eye(r))) <= 2e-11     # (the angles the call may leave, and rounding)
    # at most 20 transformations of three fp64 products each, sums of D terms: sqrt(D) 2^-53 of a row each time.  What fp32 leaves
    # of the transformation's orthogonality is 1e-6, its square 1e-12: either of them left in would show.  The eigensolver is off by as
    # much, and a factor of four covers that and the sweeps.
    eps = 4 * 60 * np.sqrt(D) * 2.0 ** -53
    np.testing.assert_allclose(lam.cpu().numpy()[:r], lam_ref[:r], rtol=0, atol=eps * lam_ref[0])
    assert np.max(np.linalg.norm(V @ C - norm[lead, None] * V, axis=1)) <= (2e-11 + eps) * norm[lead[0]]


@pytest.mark.parametrize("D,r,kind", [(256, 256, "wide"), (512, 300, "geometric"), (768, 768, "close"), (256, 64, "half zero"),
                                      (1024, 640, "steps"), (2560, 64, "wide")])
def test_the_way_in_floats_leaves_no_trace(D, r, kind):
    """Spectra whose rows go most of the way in floats, or are left to doubles (eigenvalues within 1e-3), or come out of it with
    angles that floats do not tell apart (eigenvalues in steps): the eigenvalues, and the rows left behind, are those of fp64."""
    print(f"[case] floats on the way, D={D} r={r} {kind}", flush=True)
    rng = np.random.default_rng(D)
    lam = {"wide": np.linspace(2.0, 0.01, D), "geometric": 10.0 ** (-6.0 * np.arange(D) / D), "close": 1.0 + 1e-3 * np.arange(D)[::-1] / D,
           "half zero": np.where(np.arange(D) < D // 2, 1.0 / (1.0 + np.arange(D)), 0.0), "steps": np.repeat(2.0 ** -np.arange(D // 64), 64)}[kind]
    Q = torch.linalg.qr(torch.from_numpy(rng.standard_normal((D, D))).to(gu.DEV))[0]
    C = (Q * gu.to_dev(lam)) @ Q.T.contiguous()
    C = (0.5 * (C + C.T)).contiguous()
    rows = C.clone()
    got, U, sweeps = binding.calib_eigenvectors(rows, r, torch.float32)
    torch.cuda.synchronize()
    assert 0 < sweeps <= 20
    # (the matrix is that of `lam` to the rounding of its products; what the call adds is bounded as for transformations in general)
    eps = 4 * 60 * np.sqrt(D) * 2.0 ** -53
    np.testing.assert_allclose(got.cpu().numpy()[:r], lam[:r], rtol=0, atol=eps * lam[0])
    norm = rows.norm(dim=1)
    lead = torch.argsort(-norm)[:r]
    V = rows[lead] / norm[lead, None]
    keep = got[:r] > 1e-10 * lam[0]        # (eigenvectors of zero are some basis)
    V, L = V[keep], norm[lead][keep]
    assert float((V @ V.T.contiguous() - torch.eye(len(L), device=gu.DEV, dtype=torch.float64)).abs().max()) <= 2e-11
    assert float((V @ C - L[:, None] * V).norm(dim=1).max()) <= (2e-11 + eps) * lam[0]


def _rotated(lam, seed):
    rng = np.random.default_rng(seed)
    Q = torch.linalg.qr(torch.from_numpy(rng.standard_normal((len(lam), len(lam)))).to(gu.DEV))[0]
    C = (Q * gu.to_dev(lam)) @ Q.T.contiguous()
    return (0.5 * (C + C.T)).contiguous()


@pytest.mark.parametrize("D,r", [(512, 320), (1024, 640)])
def test_the_way_in_floats_is_gone(D, r):
    """A covariance of half the full rank and more eigenvectors than that: from the Cholesky factor on fp64 takes a sweep, its transformations and a
    second sweep; behind the way in floats, which counts as the first, there is none.  (Results alone would not tell whether it was gone.)"""
    print(f"[case] one sweep or two, D={D} r={r}", flush=True)
    C = _rotated(np.where(np.arange(D) < D // 2, 1.0 / (1.0 + np.arange(D)), 0.0), D + r)
    assert binding.calib_eigenvectors(C, r, torch.float32)[2] == 1


@pytest.mark.parametrize("D,kind", [(256, "wide"), (256, "geometric"), (512, "power"), (512, "six decades"), (1024, "geometric"), (1024, "twelve decades")])
def test_eigenvalues_beside_a_64_bit_eigensolver(D, kind):
    """The whole call against LAPACK on the same matrix.  Either is off by what fp64 sums of D products are, sqrt(D) 2^-53 of the largest
    eigenvalue, for each of the few products that the rows go through behind the floats: eight of them here (measured 2e-15 on average and 1e-14 at
    most, D = 256 to 1024).  A V that came out of the floats orthogonal to 5e-5 only, corrected to third order, leaves 4e-14."""
    print(f"[case] 64-bit eigensolver, D={D} {kind}", flush=True)
    c = np.arange(1, D + 1)
    lam = {"wide": 2.0 - 1.99 * c / D, "geometric": 10.0 ** (-2.0 * c / D), "power": c ** -2.0, "six decades": 10.0 ** (-6.0 * c / D),
           "twelve decades": 10.0 ** (-12.0 * c / D)}[kind]
    C = _rotated(lam, D)
    want = np.linalg.eigvalsh(C.cpu().numpy())[::-1]
    got, _, sweeps = binding.calib_eigenvectors(C, D, torch.float32)
    assert 0 < sweeps <= 20
    np.testing.assert_allclose(got.cpu().numpy(), want, rtol=0, atol=8 * np.sqrt(D) * 2.0 ** -53 * want[0])


@pytest.mark.parametrize("D,r,width", [(256, 256, 16), (512, 200, 32), (768, 768, 64), (768, 480, 96), (1024, 640, 128)])
def test_coupled_groups_of_neighbouring_rows(D, r, width):
    """Groups of `width` neighbouring channels that mix among themselves alone: rotations inside the small blocks of rows, inside blocks, inside
    pairs of them and across pairs, which the launches that rotate single pairs deal with before any transformation of all rows."""
    print(f"[case] groups of {width}, D={D} r={r}", flush=True)
    rng = np.random.default_rng(D + width)
    lam = np.linspace(2.0, 0.01, D)
    C = np.zeros((D, D))
    for a in range(0, D, width):
        Q = np.linalg.qr(rng.standard_normal((width, width)))[0]
        C[a:a + width, a:a + width] = (Q * lam[a:a + width]) @ Q.T
    C = gu.to_dev(0.5 * (C + C.T)).contiguous()
    rows = C.clone()
    got, U, sweeps = binding.calib_eigenvectors(rows, r, torch.float32)
    torch.cuda.synchronize()
    assert 0 < sweeps <= 20
    # (bounds as above)
    eps = 4 * 60 * np.sqrt(D) * 2.0 ** -53
    np.testing.assert_allclose(got.cpu().numpy()[:r], lam[:r], rtol=0, atol=eps * lam[0])
    norm = rows.norm(dim=1)
    lead = torch.argsort(-norm)[:r]
    V = rows[lead] / norm[lead, None]
    assert float((V @ V.T.contiguous() - torch.eye(r, device=gu.DEV, dtype=torch.float64)).abs().max()) <= 2e-11
    assert float((V @ C - norm[lead, None] * V).norm(dim=1).max()) <= (2e-11 + eps) * lam[0]


@pytest.mark.parametrize("D,r,turn", [(256, 160, 0.3), (512, 512, 0.3), (256, 256, 2.0), (768, 480, 2.0), (256, 100, 12.0), (1280, 64, 12.0)])
def test_polar_factors_that_steer(D, r, turn):
    """Eigenvectors turned out of the axes by angles whose squares sum to turn^2: polar factors of one, two and more steps in floats, the
    smallest width and one that is no power of two.  What they are rounded to must not be seen in the result."""
    print(f"[case] polar factors, D={D} r={r} turned by {turn:g}", flush=True)
    rng = np.random.default_rng(D + r)
    K = torch.from_numpy(np.triu(rng.standard_normal((D, D)), 1)).to(gu.DEV)
    K = (K - K.T) * (turn / D)
    Q = torch.linalg.matrix_exp(K)
    lam = np.linspace(3.0, 0.5, D)
    C = (Q * gu.to_dev(lam)) @ Q.T.contiguous()
    C = (0.5 * (C + C.T)).contiguous()
    rows = C.clone()
    got, U, sweeps = binding.calib_eigenvectors(rows, r, torch.float32)
    torch.cuda.synchronize()
    assert 0 < sweeps <= 20
    # (bounds as above: the matrix is that of `lam` to the rounding of its products, and at most 20 transformations)
    eps = 4 * 60 * np.sqrt(D) * 2.0 ** -53
    np.testing.assert_allclose(got.cpu().numpy()[:r], lam[:r], rtol=0, atol=eps * lam[0])
    norm = rows.norm(dim=1)
    lead = torch.argsort(-norm)[:r]
    V = rows[lead] / norm[lead, None]
    assert float((V @ V.T.contiguous() - torch.eye(r, device=gu.DEV, dtype=torch.float64)).abs().max()) <= 2e-11
    assert float((V @ C - norm[lead, None] * V).norm(dim=1).max()) <= (2e-11 + eps) * lam[0]


@pytest.mark.parametrize("large,width,n_large,r", [(1e5, 1e-11, 2, 3), (1e5, 1e-11, 4, 8), (10.0, 1e-10, 4, 8), (1e3, 1e-10, 4, 12)])
def test_rows_of_a_tight_cluster_are_asked_to_have_converged(large, width, n_large, r):
    """A few large eigenvalues and all others within a relative `width`, the r-th among these: its row's norm falls far while the large
    rows are found, and the call must not stop by what it was then.  (Sweeps and transformations take turns here.)"""
    print(f"[case] cluster of width {width:g} below {n_large} eigenvalues around {large:g}, r={r}", flush=True)
    D = 256
    for seed in range(4):
        rng = np.random.default_rng(seed)
        Q, _ = np.linalg.qr(rng.standard_normal((D, D)))
        C = (Q * np.concatenate([large * (1.0 + rng.random(n_large)), 1.0 + width * rng.random(D - n_large)])) @ Q.T
        Cg = gu.to_dev(0.5 * (C + C.T))
        _, _, sweeps = binding.calib_eigenvectors(Cg, r, torch.float32)
        torch.cuda.synchronize()
        assert sweeps > 0
        rows = Cg.cpu().numpy()
        lam = np.linalg.norm(rows, axis=1)
        order = np.argsort(-lam)
        V, lam = rows[order] / lam[order, None], lam[order]
        cos = np.abs(V[:r] @ V.T)
        cos[np.arange(r), np.arange(r)] = 0.0
        ab = cos * np.sqrt(np.outer(lam[:r], lam))
        turn = ab / np.maximum(np.maximum(np.abs(lam[:r, None] - lam), 2.0 * ab), 1e-300)
        # rows orthogonal to working precision are not rotated (1e-15 there, and sums of D products here)
        assert np.max(turn[cos > 4e-15], initial=0.0) <= 1e-11, (seed, sweeps)


def _spectrum_on_device(D, decay, mixed, seed=1):
    """A covariance of 4 D keys whose channels decay as c^-decay, along directions that mix all channels if `mixed`."""
    g = torch.Generator(device=gu.DEV)
    g.manual_seed(seed)
    X = torch.randn(4 * D, D, generator=g, device=gu.DEV, dtype=torch.float64)
    X *= torch.arange(1, D + 1, device=gu.DEV, dtype=torch.float64) ** -decay
    if mixed:
        X = X @ (torch.randn(D, D, generator=g, device=gu.DEV, dtype=torch.float64) / D ** 0.5)
    C = X.T.contiguous() @ X
    return (C + C.T) * 0.5


@pytest.mark.parametrize("D,r,decay,mixed", [(2048, 256, 1.0, False), (2048, 1280, 0.25, True), (1024, 512, 1.0, False)])
def test_the_call_repeats_bit_for_bit(D, r, decay, mixed):
    """No result depends on the order in which workgroups run.  These matrices leave angles between 1e-11 and 1e-9 in the end, for
    which one product of the closing series is enough (D = 2048: more workgroups than run at once)."""
    print(f"[case] eigenvectors repeated, D={D} r={r} decay={decay}", flush=True)
    C = _spectrum_on_device(D, decay, mixed)
    first = None
    for _ in range(3):
        rows = C.clone()
        lam, U, sweeps = binding.calib_eigenvectors(rows, r, torch.float32)
        torch.cuda.synchronize()
        if first is None:
            first = (rows, lam, U, sweeps)
        assert sweeps == first[3]
        assert torch.equal(lam, first[1]) and torch.equal(U, first[2]) and torch.equal(rows, first[0])


@pytest.mark.parametrize("D", [256, 512, 1024])
def test_transformations_are_orthogonal_to_rounding(D):
    """What transforms the rows leaves their products G^T G as they are: those behind the first sweep (a call of one sweep leaves its
    rows in the factor's place) against those at the end, which lie in one of the workspace's three matrices.  Eigenvalues between
    1 and 2, so that no direction of the rows is too small to show it."""
    print(f"[case] orthogonality of the transformations, D={D}", flush=True)
    rng = np.random.default_rng(D)
    V, _ = np.linalg.qr(rng.standard_normal((D, D)))
    C = (V * np.linspace(1.0, 2.0, D)) @ V.T
    C = 0.5 * (C + C.T)
    nbytes, size = binding._lib.sals_calib_eigenvectors_workspace_bytes(D), 8 * D * D
    lam = torch.empty(D, dtype=torch.float64, device=gu.DEV)
    U = torch.empty(D, D, dtype=torch.float32, device=gu.DEV)

    def products(limit):
        ws = torch.zeros(nbytes, dtype=torch.uint8, device=gu.DEV)
        n = ctypes.c_int32(0)
        st = binding._lib.sals_calib_eigenvectors(gu.to_dev(C).data_ptr(), D, D, binding.SALS_F32, lam.data_ptr(), U.data_ptr(), ws.data_ptr(),
                                                  nbytes, limit, ctypes.byref(n), None)
        torch.cuda.synchronize()
        assert binding.status_string(st) == "SALS_OK"
        return n.value, [M.T @ M for M in (ws[at:at + size].cpu().numpy().view(np.float64).reshape(D, D)
                                           for at in (0, nbytes - 2 * size, nbytes - size))]

    n, behind_one = products(1)
    assert n == -1 and np.max(np.abs(behind_one[0] - C)) <= 1e-12   # (the premise)
    n, at_end = products(80)
    assert n == 1                                                   # (no further sweep)
    change = min(np.linalg.norm(P - behind_one[0], 2) for P in at_end if np.all(np.abs(P) < 10.0))
    print(f"    G^T G changed by {change:.2e}", flush=True)
    # A product with an orthogonal matrix, sums of D terms, leaves its elements off by about half a 2^-53 at random, a matrix of norm
    # sqrt(D) 2^-53, and G^T G off by 2 sqrt(2) times that; two of them in each of at most eight transformations, which add up as squares.
    # (What an X with X X^T - I = 3e-5 leaves behind three orders of correction is 2e-14 by itself.)
    assert change <= 4 * 2.0 ** 1.5 * D ** 0.5 * 2.0 ** -53


@pytest.mark.parametrize("power", [200, -200, 400, -400])
@pytest.mark.parametrize("D,r,decay,mixed", [(512, 512, 0.25, True), (1024, 200, 1.0, False)])
def test_scale_of_the_covariance_changes_nothing(D, r, decay, mixed, power):
    """2^200 C and 2^-200 C, far outside the range of fp32: the same steps, and 2^200 times the eigenvalues, to the last bit (every
    quantity scales by a power of two)."""
    print(f"[case] eigenvectors of 2^{power} C, D={D} r={r} decay={decay}", flush=True)
    C = _spectrum_on_device(D, decay, mixed)
    lam, U, sweeps = binding.calib_eigenvectors(C.clone(), r, torch.float32)
    lam2, U2, sweeps2 = binding.calib_eigenvectors(C * 2.0 ** power, r, torch.float32)
    torch.cuda.synchronize()
    assert 0 < sweeps2 == sweeps
    assert torch.equal(lam2, lam * 2.0 ** power) and torch.equal(U2, U)


def _eig_with_workspace(C, r, nbytes, max_sweeps=80):
    """The call on a workspace of `nbytes`, which lies before bytes that must stay as they are."""
    D = C.shape[0]
    guard = 4096
    ws = torch.full((nbytes + guard,), 0xA5, dtype=torch.uint8, device=gu.DEV)
    lam = torch.empty(D, dtype=torch.float64, device=gu.DEV)
    U = torch.empty(D, r, dtype=torch.float32, device=gu.DEV)
    sweeps = ctypes.c_int32(0)
    st = binding._lib.sals_calib_eigenvectors(C.data_ptr(), D, r, binding.SALS_F32, lam.data_ptr(), U.data_ptr(), ws.data_ptr(), nbytes,
                                              max_sweeps, ctypes.byref(sweeps), None)
    torch.cuda.synchronize()
    assert bool((ws[nbytes:] == 0xA5).all())
    return binding.status_string(st), lam.cpu().numpy(), sweeps.value


@pytest.mark.parametrize("D,r", [(256, 256), (768, 500), (1024, 256), (1280, 1280)])
def test_eigenvectors_with_a_small_workspace(D, r):
    """From 8 D^2 + 900 D bytes on the call sweeps to the end, with fewer slices where all of them do not fit: the same
    decomposition.  With the full size rows are transformed all at once, which takes fewer sweeps on this spectrum and leaves
    the eigenvalues where sweeps would: what transforms the rows is orthogonal to rounding."""
    print(f"[case] eigenvectors, small workspace, D={D} r={r}", flush=True)
    rng = np.random.default_rng(3 * D)
    X = rng.standard_normal((4 * D, D)) * np.arange(1, D + 1) ** -0.5
    C = X.T @ X
    C = 0.5 * (C + C.T)
    lam_ref = np.linalg.eigvalsh(C)[::-1]
    full = binding._lib.sals_calib_eigenvectors_workspace_bytes(D)
    assert _eig_with_workspace(gu.to_dev(C), r, 8 * D * D)[0] == "SALS_ERR_WORKSPACE"
    ran, lams = {}, {}
    for nbytes in (8 * D * D + 900 * D, 10 * D * D + 2600 * D, full - 1, full):
        Cg = gu.to_dev(C)
        status, lam, ran[nbytes] = _eig_with_workspace(Cg, r, nbytes)
        assert status == "SALS_OK" and 0 < ran[nbytes] <= 30, (nbytes, status, ran)
        rows = Cg.cpu().numpy()
        norm = np.linalg.norm(rows, axis=1)
        lead = np.argsort(-norm)[:r]
        V = rows[lead] / norm[lead, None]
        # (the bounds of test_rows_left_behind_are_orthogonal_in_fp64)
        assert np.max(np.abs(V @ V.T - np.eye(r))) <= 2e-11
        np.testing.assert_allclose(lam[:r], lam_ref[:r], rtol=0, atol=1e-11 * lam_ref[0])
        lams[nbytes] = lam[:r]
    print("    sweeps", ran, "eigenvalues apart", np.max(np.abs(lams[full] / lams[full - 1] - 1.0)), flush=True)
    # one or two sweeps more: D / 32 steps each, sums of 64 products (2 sqrt(64) 2^-53 of a squared norm per step at most).  A
    # series cut one term too early, or used at twice the angles it may be, leaves 1e-11 and more
    np.testing.assert_allclose(lams[full], lams[full - 1], rtol=2 * D / 32 * 16 * 2.0 ** -53)
    assert all(ran[full] < n for nbytes, n in ran.items() if nbytes != full)


@pytest.mark.parametrize("D,r,large,width,n_large", [(256, 68, 10.0, 1e-10, 64), (256, 41, 1e4, 0.0, 40), (256, 20, 10.0, 1e-10, 16),
                                                      (512, 200, 10.0, 1.0, 100)])
def test_a_limit_of_sweeps_is_enough_with_transformations_too(D, r, large, width, n_large):
    """The sweeps that a call takes without transformations are enough with them, also where the two take turns."""
    print(f"[case] limit of sweeps, D={D}, cluster of width {width:g}", flush=True)
    rng = np.random.default_rng(D + n_large)
    Q, _ = np.linalg.qr(rng.standard_normal((D, D)))
    C = (Q * np.concatenate([large * (1.0 + rng.random(n_large)), 1.0 + width * rng.random(D - n_large)])) @ Q.T
    C = gu.to_dev(0.5 * (C + C.T))
    full = binding._lib.sals_calib_eigenvectors_workspace_bytes(D)
    status, alone, limit = _eig_with_workspace(C.clone(), r, full - 1)
    assert status == "SALS_OK" and limit > 0
    status, lam, sweeps = _eig_with_workspace(C.clone(), r, full, limit)
    print(f"    sweeps {sweeps}, without transformations {limit}", flush=True)
    assert status == "SALS_OK" and 0 < sweeps <= limit
    np.testing.assert_allclose(lam[:r], alone[:r], rtol=1e-13)


def test_eigenvectors_in_bf16_are_the_rounded_fp64_vectors():
    print("[case] eigenvectors bf16", flush=True)
    D, r = 256, 32
    X = synth.widen(synth.make_calibration_keys(3, 1024, D, "f32", decay=0.85))
    C = cal.covariance(X)
    _, U_ref = cal.leading_eigenvectors(C, r)
    _, U, _ = _eig_gpu(C, r, torch.bfloat16)
    # one rounding to bf16 (8 significant bits): half an ulp of the component, plus the fp64 agreement
    for i in range(r):
        ref = U_ref[:, i] * np.sign(U_ref[np.argmax(np.abs(U_ref[:, i])), i])
        assert np.all(np.abs(U[:, i] - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-7), i


def test_repeated_eigenvalues_give_a_valid_basis():
    print("[case] repeated eigenvalues", flush=True)
    D = 256
    rng = np.random.default_rng(5)
    Q, _ = np.linalg.qr(rng.standard_normal((D, D)))
    lam_true = np.concatenate([np.full(8, 5.0), np.full(8, 2.0), np.linspace(1.0, 0.1, D - 16)])
    C = (Q * lam_true) @ Q.T
    C = 0.5 * (C + C.T)
    lam, U, sweeps = _eig_gpu(C, 16)
    assert sweeps > 0
    np.testing.assert_allclose(lam[:16], np.sort(lam_true)[::-1][:16], rtol=0, atol=1e-11 * 5.0)
    np.testing.assert_allclose(U.T @ U, np.eye(16), atol=5e-7)
    # each block of columns spans the eigenspace of its eigenvalue: the projector is unique
    for a, b in ((0, 8), (8, 16)):
        P_ref = Q[:, a:b] @ Q[:, a:b].T
        P = U[:, a:b] @ U[:, a:b].T
        assert np.max(np.abs(P - P_ref)) <= 2e-6


def test_rank_deficient_covariance_and_diagonal_input():
    print("[case] rank deficient, diagonal", flush=True)
    D = 256
    X = synth.widen(synth.make_calibration_keys(9, 100, D, "f32", decay=0.9))   # 100 tokens: rank 100
    C = cal.covariance(X)
    lam_ref, U_ref = cal.leading_eigenvectors(C, 40)
    lam, U, sweeps = _eig_gpu(C, 40)
    assert sweeps > 0
    np.testing.assert_allclose(lam[:40], lam_ref[:40], rtol=0, atol=1e-10 * lam_ref[0])
    # past the r requested ones the values are the row norms when the leading rows had converged: approximations
    np.testing.assert_allclose(lam[40:], lam_ref[40:], rtol=0, atol=1e-3 * lam_ref[0])
    _same_up_to_sign(U, U_ref, 5e-7)
    # asked for as many vectors as the rank: every non-zero eigenvalue converges and what is left of the other rows
    # is zero to working precision
    lam_ref, U_ref = cal.leading_eigenvectors(C, 100)
    lam, U, sweeps = _eig_gpu(C, 100)
    assert sweeps > 0
    np.testing.assert_allclose(lam[:100], lam_ref[:100], rtol=0, atol=1e-10 * lam_ref[0])
    assert np.all(np.abs(lam[100:]) <= 1e-9 * lam_ref[0])
    _same_up_to_sign(U[:, :60], U_ref[:, :60], 5e-7)
    # a diagonal matrix needs no rotation: one sweep, eigenvalues sorted, unit vectors
    d = np.linspace(0.5, 3.0, D)
    lam, U, sweeps = _eig_gpu(np.diag(d), 5)
    assert sweeps == 1
    np.testing.assert_array_equal(lam, np.sort(d)[::-1])
    for i in range(5):
        e = np.zeros(D); e[D - 1 - i] = 1.0
        np.testing.assert_array_equal(U[:, i], e)


def _channels_of_different_scale(case, D):
    """Keys whose channels span 1 .. 1e-7 in amplitude (small ones ahead, behind or among the large ones), and keys in
    which one channel repeats another up to 1e-7 of it.  Their eigenvectors are well determined all the same."""
    rng = np.random.default_rng(41)
    mix = np.eye(D) + 0.3 / np.sqrt(D) * rng.standard_normal((D, D))
    scale = 10.0 ** -np.linspace(0.0, 7.0, D)
    X = rng.standard_normal((4 * D, D)) @ mix * scale
    if case == "rising":
        return X[:, ::-1]
    if case == "shuffled":
        return X[:, rng.permutation(D)]
    if case == "repeated":
        X[:, 1] = X[:, 0] + 1e-7 * np.std(X[:, 0]) / np.std(X[:, 80]) * X[:, 80]
    return X


@pytest.mark.parametrize("case", ["falling", "rising", "shuffled", "repeated"])
def test_eigenvectors_with_channels_of_very_different_scale(case):
    print(f"[case] eigenvectors, channel scales {case}", flush=True)
    D, r = 256, 180   # the eigenvalues asked for reach down to about 1e-10 of the largest
    X = _channels_of_different_scale(case, D)
    _, sv, Vt = np.linalg.svd(X, full_matrices=False)
    lam, U, sweeps = _eig_gpu(X.T @ X, r)
    assert sweeps > 0
    # the matrix in fp64 differs from X^T X by a few hundred 1e-16 of sqrt(C_ii C_jj), which moves an eigenvalue by as much of
    # itself; the singular vectors are good to 1e-16 sigma_0 / gap, gaps of about 1e-7 sigma_0 among the last; fp32 storage
    np.testing.assert_allclose(lam[:r], sv[:r] ** 2, rtol=1e-8)
    _same_up_to_sign(U, Vt[:r].T, 5e-7)
    np.testing.assert_allclose(U.T @ U, np.eye(r), atol=5e-7)


@pytest.mark.parametrize("D,n,r", [(256, 100, 40), (512, 500, 256)])
def test_eigenvectors_of_fewer_tokens_than_channels(D, n, r):
    """The covariance the library itself accumulates (fp32 sums) of fewer tokens than channels is indefinite at the
    level of those sums: the leading eigenvectors are those of the matrix as it is."""
    print(f"[case] eigenvectors of {n} tokens, D={D}", flush=True)
    C = _cov_gpu(synth.make_calibration_keys(17, n, D, "bf16", decay=0.97)).cpu().numpy()
    lam_ref, U_ref = cal.leading_eigenvectors(C, r)
    assert lam_ref[-1] < -1e-12 * lam_ref[0]   # (the premise)
    lam, U, sweeps = _eig_gpu(C, r)
    assert sweeps > 0
    np.testing.assert_allclose(lam[:r], lam_ref[:r], rtol=0, atol=1e-11 * lam_ref[0])
    # every column solves the defining equation to fp32 storage, against its own eigenvalue
    resid = np.linalg.norm(C @ U - U * lam[:r], axis=0)
    assert np.max(resid / lam_ref[0]) <= 1e-6
    np.testing.assert_allclose(U.T @ U, np.eye(r), atol=5e-7)
    assert np.all(lam >= 0.0) and np.all(np.diff(lam) <= 0.0)


def test_sweep_limit_is_reported():
    D = 256
    X = synth.widen(synth.make_calibration_keys(13, 1024, D, "f32", decay=0.9))
    lam, U, sweeps = _eig_gpu(cal.covariance(X), 8, max_sweeps=1)
    assert sweeps == -1


@pytest.mark.parametrize("D,r,decades", [(512, 320, 12), (512, 512, 12), (1024, 1024, 12), (2304, 1408, 8), (2560, 1600, 12)])
def test_wide_spectra_need_no_sweep_behind_the_floats(D, r, decades):
    """Eigenvalues over many decades, whose angles fall slowly at first: the way in floats, which counts as one sweep, is gone to its end, and what
    it leaves is for transformations at any width."""
    print(f"[case] wide spectrum, D={D} r={r} {decades} decades", flush=True)
    lam = 10.0 ** (-decades * np.arange(1, D + 1) / D)
    got, _, sweeps = binding.calib_eigenvectors(_rotated(lam, D + r), r, torch.float32)
    torch.cuda.synchronize()
    assert sweeps == 1
    # (bounds as above)
    eps = 4 * 60 * np.sqrt(D) * 2.0 ** -53
    np.testing.assert_allclose(got.cpu().numpy()[:r], lam[:r], rtol=0, atol=eps * lam[0])


@pytest.mark.parametrize("D,r,angle", [(256, 256, 0.1), (256, 85, 0.03), (512, 512, 0.01), (1024, 341, 0.03)])
def test_one_sweep_is_enough_where_it_was(D, r, angle):
    """Channels that mix in pairs far apart, by small angles: one sweep rotates them, so a limit of one sweep does."""
    print(f"[case] limit of one sweep, D={D} r={r} turned by {angle:g}", flush=True)
    rng = np.random.default_rng(D + r)
    lam = np.linspace(2.0, 0.1, D)
    turn = angle * rng.uniform(0.5, 1.0, D // 2) * rng.choice([-1, 1], D // 2)
    i, j = np.arange(D // 2), np.arange(D // 2, D)
    Q = np.zeros((D, D))
    Q[i, i] = Q[j, j] = np.cos(turn)
    Q[i, j], Q[j, i] = -np.sin(turn), np.sin(turn)
    at = rng.permutation(D)
    C = gu.to_dev((Q * lam[at]) @ Q.T).contiguous()
    C = (0.5 * (C + C.T)).contiguous()
    rows = C.clone()
    got, U, sweeps = binding.calib_eigenvectors(rows, r, torch.float32, max_sweeps=1)
    torch.cuda.synchronize()
    assert sweeps == 1
    # (bounds of one sweep's rotations, as for transformations above)
    eps = 4 * 60 * np.sqrt(D) * 2.0 ** -53
    np.testing.assert_allclose(got.cpu().numpy()[:r], lam[:r], rtol=0, atol=eps * lam[0])
    norm = rows.norm(dim=1)
    lead = torch.argsort(-norm)[:r]
    V = rows[lead] / norm[lead, None]
    assert float((V @ C - norm[lead, None] * V).norm(dim=1).max()) <= (2e-11 + eps) * lam[0]


def test_whole_calibration_captures_the_energy_of_the_oracle_basis():
    print("[case] keys -> covariance -> eigenvectors", flush=True)
    D, r, n = 512, 128, 6000
    Xs = synth.make_calibration_keys(21, n, D, "bf16", decay=0.97, heads=4)
    C_gpu = _cov_gpu(Xs)
    C_ref, lam_ref, U_ref = cal.calibrate(synth.widen(Xs), r)
    Cg = C_gpu.clone()
    lam, U, sweeps = binding.calib_eigenvectors(Cg, r, torch.bfloat16)
    torch.cuda.synchronize()
    assert sweeps > 0
    U = gu.from_dev(U)
    np.testing.assert_allclose(lam.cpu().numpy()[:r], lam_ref[:r], rtol=2e-5)
    e_ref = cal.captured_energy(C_ref, U_ref)
    # bf16 columns are no longer exactly orthonormal: measure the energy of their span
    Qn, _ = np.linalg.qr(U)
    assert cal.captured_energy(C_ref, Qn) >= (1.0 - 1e-5) * e_ref
    assert np.max(np.abs(U.T @ U - np.eye(r))) <= 2.0 ** -7


def test_bad_arguments_are_refused():
    C = torch.zeros(256, 256, dtype=torch.float64, device=gu.DEV)
    X = torch.zeros(10, 200, dtype=torch.bfloat16, device=gu.DEV)          # D not a multiple of 128
    assert binding._lib.sals_calib_accumulate_workspace_bytes(binding.SALS_BF16, 200) == 0
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=gu.DEV)
    st = binding._lib.sals_calib_accumulate(binding.SALS_BF16, X.data_ptr(), 10, 200, C.data_ptr(), ws.data_ptr(), 1 << 20, None)
    assert binding.status_string(st) == "SALS_ERR_INVALID_ARG"
    X = torch.zeros(10, 256, dtype=torch.bfloat16, device=gu.DEV)
    st = binding._lib.sals_calib_accumulate(binding.SALS_BF16, X.data_ptr(), 10, 256, C.data_ptr(), ws.data_ptr(), 1024, None)
    assert binding.status_string(st) == "SALS_ERR_WORKSPACE"
    ev = torch.empty(256, dtype=torch.float64, device=gu.DEV)
    U = torch.empty(256, 4, dtype=torch.float32, device=gu.DEV)
    n = ctypes.c_int32(0)
    st = binding._lib.sals_calib_eigenvectors(C.data_ptr(), 256, 0, binding.SALS_F32, ev.data_ptr(), U.data_ptr(), ws.data_ptr(),
                                              1 << 20, 5, ctypes.byref(n), None)
    assert binding.status_string(st) == "SALS_ERR_INVALID_ARG"
    st = binding._lib.sals_calib_eigenvectors(C.data_ptr(), 256, 4, binding.SALS_F32, ev.data_ptr(), U.data_ptr(), ws.data_ptr(),
                                              1024, 5, ctypes.byref(n), None)
    assert binding.status_string(st) == "SALS_ERR_WORKSPACE"
    torch.cuda.synchronize()


def test_calibrated_projector_feeds_the_decode_path(oracle):
    """The projector the calibration returns has the layout the rest of the library takes: pack it, compress keys
    with it and run a decode step; every stage against the oracle with the same projector."""
    print("[case] calibrated projector in a decode step", flush=True)
    w = synth.shrink(synth.CONFIGS["cfg2"], B=2, S=600, H=4, H_kv=4, r=128, top_k=64, n_layers=1, plant=2)
    keys = synth.make_calibration_keys(31, 3000, w.D_kv, w.dtype, decay=0.985)
    C = _cov_gpu(keys)
    _, U, sweeps = binding.calib_eigenvectors(C, w.r, torch.bfloat16)
    torch.cuda.synchronize()
    assert sweeps > 0
    L = synth.make_layer(w, 0)
    U_bits = U.view(torch.int16).cpu().numpy().view(np.uint16)
    L["Uk"] = U_bits.copy()
    L["Uv"] = U_bits.copy()
    ctx = gu.make_ctx(w)
    G = gu.upload(L, ctx)
    R = gu.run_stages(ctx, w, G)
    for b in range(w.B):
        gu.check_sequence(oracle, w, L, R, b)
    # compression with the calibrated projector keeps what the spectrum says it keeps
    x = synth.widen(keys[:64])
    kt = x @ synth.widen(U_bits)
    lam_ref, _ = cal.leading_eigenvectors(cal.covariance(synth.widen(keys)), w.r)
    kept = np.sum(kt * kt) / np.sum(x * x)
    assert abs(kept - np.sum(lam_ref[: w.r]) / np.sum(lam_ref)) < 0.05
    ctx.close()
