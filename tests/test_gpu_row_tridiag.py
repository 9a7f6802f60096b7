"""The reduction of up to 32 rows, a row per lane: sizes at the edges of its register arrays (multiples of 4) and of the rows of 16 lanes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 15, 16, 17, 18, 20, 21, 24, 25, 28, 29, 30, 31, 32])
def test_row_tridiagonalisation(n):
    import torch
    from paper_2207_04228_amd import binding
    rng = np.random.default_rng(7700 + n)
    A = rng.standard_normal((5, n, n))
    A = (0.5 * (A + A.transpose(0, 2, 1))).astype(np.float32)
    A[1] = 0.0                                       # every reflector left out
    A[2] = np.diag(rng.standard_normal(n))
    A[3] *= np.float32(2.0 ** -40)                   # the pre-scaling
    given = A.copy()
    rows, cols = np.triu_indices(n, 1)
    given[:, rows, cols] = np.nan if n % 2 else 1e30                 # what stands above the diagonal is not read
    print(f"[row tridiag] n={n}", flush=True)
    At = torch.from_numpy(given).cuda()
    d, e, P = binding.bed_tridiag(At)
    d0, e0, _ = binding.bed_tridiag(At, want_P=False)
    assert torch.equal(d, d0) and torch.equal(e, e0)                # with and without P, the same bits
    d, e, P = (x.double().cpu().numpy() for x in (d, e, P))
    T = np.zeros((5, n, n))
    i = np.arange(n)
    T[:, i, i] = d
    T[:, i[1:], i[:-1]] = T[:, i[:-1], i[1:]] = e[:, :n - 1]
    A64 = A.astype(np.float64)
    # n reflectors, each backward stable to a few roundings (2^-24) of the norm: the bar of the stage tests, 1e-5 n
    size = np.maximum(np.sqrt((A64 ** 2).sum(axis=(1, 2))), 1e-300)
    assert (np.sqrt(((P @ T @ P.transpose(0, 2, 1) - A64) ** 2).sum(axis=(1, 2))) / size).max() <= 1e-5 * n
    assert np.sqrt(((P.transpose(0, 2, 1) @ P - np.eye(n)) ** 2).sum(axis=(1, 2))).max() <= 1e-5 * n
    # a NaN or an infinity below the diagonal reaches the outputs of its matrix and of no other
    bad = At.clone()
    bad[0, n - 1, 0] = float("nan")
    bad[4, n - 1, n // 2] = float("inf")
    lam, V = binding.bed_syevd(At)
    lam_b, V_b = binding.bed_syevd(bad)
    assert (~torch.isfinite(lam_b)).any(1)[[0, 4]].all() and (~torch.isfinite(V_b)).any(2).any(1)[[0, 4]].all()
    assert torch.equal(lam_b[1:4], lam[1:4]) and torch.equal(V_b[1:4], V[1:4])
