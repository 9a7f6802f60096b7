"""The divide-and-conquer path of bed_syevd and bed_spd_fn at the sizes where it can go wrong: leaves of two to
four rows, uneven halves, edges of the tiles, heavy deflation, rotations of close poles.  Same
bars as the rotation kernels (eigenvalues 1e-5 ||A||_2, residual and orthogonality 1e-5 n)."""
import numpy as np
import pytest

from test_gpu_parity import _check, _solve_gpu

pytestmark = pytest.mark.gpu

SIZES = [11, 12, 13, 14, 15, 16, 17, 20, 21, 24, 25, 28, 29, 31, 32,
         33, 36, 47, 48, 49, 63, 64, 65, 95, 96, 97, 100, 127, 128]


def _structured(n, seed):
    rng = np.random.default_rng(seed)
    one = np.eye(n, k=1) + np.eye(n, k=-1)
    wilkinson = np.tile(np.abs(np.arange(21) - 10.0), 1 + n // 21)[:n]
    weak = np.ones(n - 1)
    weak[20::21] = 1e-7                                     # glued: pairs equal to rounding
    split = rng.standard_normal(n - 1)
    split[::3] = 0.0
    x = rng.standard_normal(n)
    Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
    graded = 10.0 ** -np.linspace(0, 12, n)
    mats = [np.zeros((n, n)), np.eye(n), np.diag(x), 2 * np.eye(n) - one, np.ones((n, n)), np.eye(n) + 1e-7 * one,
            np.diag(wilkinson) + np.diag(weak, 1) + np.diag(weak, -1),
            np.diag(x) + np.diag(split, 1) + np.diag(split, -1),
            np.outer(x, x) + 0.5 * np.eye(n), -np.outer(x, x) - 0.5 * np.eye(n),
            np.diag(graded) + 0.5 * np.diag(graded[1:], 1) + 0.5 * np.diag(graded[1:], -1),
            (Q * np.repeat(x, 5)[:n]) @ Q.T]
    A = np.stack(mats)
    return (0.5 * (A + A.transpose(0, 2, 1))).astype(np.float32)


def _runs(A):
    """Is this batch on the path that the file is about?"""
    from paper_2207_04228_amd import binding
    return binding.bed_syevd_kernel(A.shape[0], A.shape[1]).startswith("dc_")


@pytest.mark.parametrize("n", SIZES)
def test_decomposition_and_eigenvalues_only(n):
    from paper_2207_04228_amd import workloads
    batch = 17 if n > 11 else 256
    for A, name in ((workloads.covariance(batch, n, 4 * n, 1e-4, 6100 + n), "full rank"),
                    (workloads.covariance(batch, n, max(1, n // 2), 1e-2, 6200 + n), "half rank"),
                    (np.tile(_structured(n, n), ((batch + 11) // 12, 1, 1)), "structured")):
        assert _runs(A)
        _check(A, f"divide and conquer, {name}, n={n}")
        lam, V = _solve_gpu(A)
        only, none = _solve_gpu(A, want_vectors=False)
        assert none is None
        norm = np.abs(lam).max(axis=1, keepdims=True)
        assert np.all(np.abs(lam - only) <= 1e-5 * norm)


def _solve_raw(A32):
    """(evals, evecs, info of the spectral function): _solve_gpu compares the input with itself, which NaN fails"""
    import torch
    from paper_2207_04228_amd import binding
    At = torch.from_numpy(A32).cuda()
    lam, V = binding.bed_syevd(At)
    return lam, V, binding.bed_spd_fn(At, binding.BED_FN_SQRT, 1e-6)[2]


@pytest.mark.parametrize("n", [13, 32, 48, 100])
def test_info_of_the_kernel_that_bed_syevd_runs(n):
    """Without rotation counts bed_syevd_info is bed_syevd with its diagnostics: 0 where every root was found, the number
    of non-finite eigenvalues otherwise."""
    import torch
    from paper_2207_04228_amd import binding, workloads
    A = np.concatenate([_structured(n, n), workloads.covariance(8, n, 3 * n // 4, 1e-2, 6950 + n)])
    A[3, 2, 1] = A[3, 1, 2] = np.nan
    At = torch.from_numpy(A).cuda()
    lam, V = binding.bed_syevd(At)
    lam1, V1, info, rotations = binding.bed_syevd_info(At, want_rotations=False)
    only, none, info_only, _ = binding.bed_syevd_info(At, want_vectors=False, want_rotations=False)
    assert rotations is None and none is None
    keep = [b for b in range(A.shape[0]) if b != 3]
    assert torch.equal(lam1[keep], lam[keep]) and torch.equal(V1[keep], V[keep]) and torch.equal(only[keep], lam[keep])
    assert (info[keep] == 0).all() and int(info[3]) == n and torch.equal(info, info_only)


def test_scales_and_non_finite_inputs():
    from paper_2207_04228_amd import workloads
    for n, copies in ((13, 1), (16, 1), (30, 1), (50, 1), (50, 43), (64, 43), (90, 1)):       # 33 to 64 rows: batch 256 and beyond reduce differently
        A = np.tile(workloads.covariance(6, n, 4 * n, 1e-4, 6300 + n), (copies, 1, 1))
        assert _runs(A)
        for s in (1e-30, 1e-20, 1e18):
            _check((A.astype(np.float64) * s).astype(np.float32), f"scaled by {s:g}, n={n}")
        good, _ = _solve_gpu(A)
        B = A.copy()
        B[1::6, 4, 2] = np.nan
        B[3::6, 5, 5] = np.inf
        lam, V, info = (t.cpu().numpy() for t in _solve_raw(B))
        lost = np.isin(np.arange(len(A)) % 6, (1, 3))
        assert np.array_equal(lam[~lost], good[~lost])          # the others are untouched
        assert np.isnan(lam[lost]).all() and np.isnan(V[lost]).all()
        assert (info[lost] > 0).all() and (info[~lost] == 0).all()


@pytest.mark.parametrize("n, copies", [(12, 1), (16, 1), (17, 1), (32, 1), (33, 1), (33, 5), (48, 1), (48, 5), (64, 1), (64, 5), (65, 1), (100, 1), (128, 1)])
def test_a_nan_that_only_its_own_column_sees(n, copies):
    """One non-finite entry below the first off-diagonal of a matrix whose other columns need no reflector, or in
    uncoupled channels in front of a dense block: no later step touches it, so its own column has to carry it into T."""
    import torch
    from paper_2207_04228_amd import binding, workloads
    h = n // 2
    block = np.diag(np.linspace(1.0, 2.0, n))
    block[h:, h:] = workloads.covariance(1, n - h, 4 * (n - h), 1e-4, 6800 + n)[0]
    one = np.eye(n, k=1) + np.eye(n, k=-1)
    mats = []
    for base, places in ((np.eye(n), ((5, 0), (n - 1, 0), (n - 1, n - 3))), (np.diag(np.arange(1.0, n + 1)), ((5, 0), (n - 1, n - 4))),
                         (2.0 * np.eye(n) - one, ((2, 0), (n - 1, n - 3))), (block, ((4, 0), (h - 1, h - 4)))):
        for i, j in places:
            for value in (np.nan, np.inf, -np.inf):
                for x in (base[i, j], value):           # the clean matrix, then the same with the entry
                    m = base.copy()
                    m[i, j] = m[j, i] = x
                    mats.append(m)
    A = np.tile(np.stack(mats).astype(np.float32), (copies, 1, 1))
    assert _runs(A) and (copies == 1) == (len(A) <= 256)             # 33 to 64 rows: beyond 256 matrices one wavefront reduces
    clean = A.copy()
    clean[1::2] = A[0::2]
    At, Ct = torch.from_numpy(A).cuda(), torch.from_numpy(clean).cuda()
    lam, V = binding.bed_syevd(At)
    only, _ = binding.bed_syevd(At, want_vectors=False)
    F, ev, info = binding.bed_spd_fn(At, binding.BED_FN_INV_SQRT, 1e-6, want_evals=True)
    F2, lam2, V2 = binding.bed_spd_fn_eigh(At, binding.BED_FN_SQRT, 1e-6)
    for t in (lam, V, only, F, ev, F2, lam2, V2):
        lost = torch.isfinite(t[1::2].flatten(1)).any(dim=1).nonzero().flatten().tolist()
        assert not lost, (n, lost)
    assert (info[1::2] > 0).all() and (info[0::2] == 0).all()
    lam_c, V_c = binding.bed_syevd(Ct)
    assert torch.equal(lam[0::2], lam_c[0::2]) and torch.equal(V[0::2], V_c[0::2])      # the others are untouched


@pytest.mark.parametrize("n", [16, 32, 64, 100, 128])
def test_small_eigenvalues_of_graded_covariances(n):
    """Power-law spectrum in a rotated basis, condition 1e3: the inverse square root needs the small eigenvalues
    to a few units of their own size (rounding of the large ones alone would show as 1e-4)."""
    import torch
    from paper_2207_04228_amd import binding
    rng = np.random.default_rng(n)
    Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
    X = (rng.standard_normal((6, 4 * n, n)) / np.arange(1, n + 1)) @ Q
    A = (np.einsum("bki,bkj->bij", X, X) / (4 * n) + 1e-3 * np.eye(n)).astype(np.float32)
    lam, V = np.linalg.eigh(A.astype(np.float64))
    ref = (V / np.sqrt(lam)[:, None, :]) @ V.transpose(0, 2, 1)
    F = binding.bed_spd_fn(torch.from_numpy(A).cuda(), binding.BED_FN_INV_SQRT, 1e-6)[0].cpu().numpy()
    err = np.linalg.norm(F - ref) / np.linalg.norm(ref)
    print(f"graded n={n}: relative error of A^(-1/2) {err:.1e}")
    assert err <= 1e-5          # the rotations reach 2e-6 (n = 16) to 6e-6 (n = 128)


@pytest.mark.parametrize("fn", [0, 1])
def test_spectral_function(fn):
    from test_gpu_spd_fn import _check as check_fn
    from paper_2207_04228_amd import workloads
    for n in (12, 13, 16, 19, 28, 32, 33, 64, 65, 128):
        A = workloads.covariance(7 if n > 12 else 17, n, 4 * n, 1e-3, 6400 + n)
        assert _runs(A)
        check_fn(A, fn, 1e-6, f"divide and conquer n={n}")


@pytest.mark.parametrize("n, batch", [(16, 2048), (32, 4096), (36, 768), (48, 1024), (64, 2048), (100, 1024), (128, 1024)])
def test_full_chip_of_copies(n, batch):
    """Copies of four matrices, several workgroups on every compute unit: all copies come out bit for bit
    the same whatever their neighbours do (wavefronts of a workgroup that run apart show here)."""
    import torch
    from paper_2207_04228_amd import binding, workloads
    A = torch.from_numpy(workloads.covariance(4, n, 2 * n, 1e-3, 6500 + n)).cuda().repeat(batch // 4, 1, 1)
    assert _runs(A)
    lam, V = binding.bed_syevd(A)
    only, _ = binding.bed_syevd(A, want_vectors=False)
    assert torch.equal(lam, lam[:4].repeat(batch // 4, 1)) and torch.equal(V, V[:4].repeat(batch // 4, 1, 1))
    assert torch.equal(lam, only)


@pytest.mark.parametrize("n", [12, 16, 24, 32])
def test_repeated_eigenvalues_take_no_longer(n):
    """Kernel time on rank-deficient covariances (three quarters of full rank, the rest of the spectrum at the ridge)
    against full rank, as in the application's own batches.  It was 1.4 times as long;
    the slowest matrix of the batch sets the time, and a few close poles must not make it visit all of them."""
    import torch
    from paper_2207_04228_amd import binding, workloads
    us = []
    for samples, ridge in ((4 * n, 1e-3), (3 * n // 4, 1e-2)):
        A = torch.from_numpy(workloads.covariance(512, n, samples, ridge, 6900 + n)).cuda()
        lam, V = binding.bed_syevd(A)
        for _ in range(20):
            binding.bed_syevd(A, lam, V)
        binding.bed_timing_begin(30)
        binding.bed_timing_arm(True)
        for _ in range(30):
            binding.bed_syevd(A, lam, V)
        us.append(float(binding.bed_timing_end(30)[0].min()))
    print(f"n={n}: full rank {us[0]:.1f} us, repeated eigenvalues {us[1]:.1f} us")
    assert us[1] <= 1.2 * us[0]


@pytest.mark.parametrize("n, batch", [(1, 5), (2, 67), (4, 1000), (8, 4099), (13, 2561), (16, 40), (18, 2561), (20, 5001), (22, 4096),
                                      (26, 6145), (32, 70), (40, 1025), (43, 769), (48, 2048),
                                      (64, 20), (65, 9), (128, 5)])
def test_function_with_its_decomposition(n, batch):
    """bed_spd_fn_eigh on both of its routes: the function as bed_spd_fn gives it, the decomposition as bed_syevd does."""
    import torch
    from paper_2207_04228_amd import binding, workloads
    A = torch.from_numpy(workloads.covariance(batch, n, 4 * n, 1e-3, 6600 + n)).cuda()
    for fn in (binding.BED_FN_SQRT, binding.BED_FN_INV_SQRT):
        out, lam, V = binding.bed_spd_fn_eigh(A, fn, 1e-6)
        ref, _, _ = binding.bed_spd_fn(A, fn, 1e-6)
        lam1, V1 = binding.bed_syevd(A)
        assert torch.equal(lam, lam1) and torch.equal(V, V1)
        err = ((out - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)).max()
        assert err <= 1e-5, err        # 32-bit sums of n terms, in another order


def test_training_step_saves_what_it_needs_and_notices_changes():
    import torch
    from paper_2207_04228_amd import autograd, binding, workloads
    A = torch.from_numpy(workloads.covariance(6, 20, 80, 1e-3, 6700)).cuda()
    G = torch.randn(6, 20, 20, device="cuda")
    x = A.clone().requires_grad_(True)
    out = autograd.spd_sqrt(x, 1e-6)
    (g,) = torch.autograd.grad(out, x, G)
    lam, V = binding.bed_syevd(A)
    assert torch.equal(g, binding.bed_spd_fn_backward(lam, V, G, binding.BED_FN_SQRT, 1e-6))
    with torch.no_grad():
        assert torch.equal(autograd.spd_sqrt(x, 1e-6), binding.bed_spd_fn(A, binding.BED_FN_SQRT, 1e-6)[0])
    out = autograd.spd_sqrt(x, 1e-6)
    with torch.no_grad():
        x.add_(1.0)
    with pytest.raises(RuntimeError):
        torch.autograd.grad(out, x, G)


@pytest.mark.parametrize("n", [34, 35, 50, 51, 66, 67, 82, 83, 98, 99, 114, 115, 126])
def test_edges_of_the_blocks_of_reflectors(n):
    """n - 2 reflectors are applied in blocks of sixteen; the structured matrices leave some of them out (zero columns)."""
    from paper_2207_04228_amd import workloads
    perm = np.random.default_rng(6990 + n).permutation(n)
    gaps = workloads.covariance(4, n, 4 * n, 1e-4, 6991 + n)
    gaps[:, ::5, :] *= np.eye(n, dtype=np.float32)[::5]         # every fifth row and column decoupled, anywhere in the order
    gaps[:, :, ::5] *= np.eye(n, dtype=np.float32)[:, ::5]
    for A, name in ((_structured(n, n + 1), "structured"), (gaps, "gaps"), (np.ascontiguousarray(gaps[:, perm][:, :, perm]), "shuffled")):
        assert _runs(A)
        _check(A, f"blocks of reflectors, {name}, n={n}")


@pytest.mark.parametrize("n", [12, 13, 19, 25, 33, 41, 52, 66, 72, 75, 85, 104, 113])
def test_leaves_of_two_to_four_rows_and_blocks_that_straddle_tiles(n):
    """Every split of n into leaves, with tridiagonal inputs (nothing to reduce: T is the matrix) that are graded, constant, split and
    have equal, zero and opposite diagonal entries next to each other."""
    rng = np.random.default_rng(6970 + n)
    off = rng.standard_normal(n - 1)
    small = 10.0 ** -rng.uniform(0, 8, n - 1)
    cases = [(2 * np.ones(n), -np.ones(n - 1)), (np.zeros(n), np.ones(n - 1)), (np.tile([1.0, -1.0], n)[:n], off), (np.ones(n), 1e-4 * off),
             (np.repeat(rng.standard_normal(n), 4)[:n], off * (np.arange(n - 1) % 4 != 3)), (10.0 ** -np.linspace(0, 10, n), small * 1e-6),
             (rng.standard_normal(n), small), (1e-20 * np.ones(n), 1e-20 * off)]
    A = np.stack([np.diag(d) + np.diag(e, 1) + np.diag(e, -1) for d, e in cases] * 2).astype(np.float32)
    assert _runs(A)
    _check(A, f"leaves, n={n}")
    lam, V = _solve_gpu(A)
    assert np.array_equal(_solve_gpu(A, want_vectors=False)[0], lam)


@pytest.mark.parametrize("n", [12, 13, 16, 17, 24, 31, 32, 33, 47, 64, 65, 100, 128])
def test_leaves_with_equal_diagonals_and_small_couplings_converge(n):
    """What a leaf leaves behind is dropped.  The bars are those of rounding: three times the residuals (5.3e-7 to 7.1e-7) and twice the
    errors of the eigenvalues (7.2e-7 to 1.15e-6) of leaves that ran to their end."""
    from oracle import jacobi
    from oracle.acceptance import evaluate
    from test_gpu_jacobi import near_diagonal
    A = near_diagonal(n, True, 7450 + n)
    assert _runs(A)
    lam, V = _solve_gpu(A)
    w = evaluate(A, lam, V, *jacobi.syevd(A)).worst()
    print(f"[parity] leaves near diagonal, n={n}: {w}", flush=True)
    assert w["eval_err"] <= 2e-6 and w["residual"] <= 2e-6
