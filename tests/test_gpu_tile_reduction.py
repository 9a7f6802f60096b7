"""The reduction of 33 to 128 rows in tiles: up to 64 rows the first columns by four wavefronts up to batch 256, by one beyond; more rows in strips."""
import numpy as np
import pytest

from oracle import jacobi
from oracle.acceptance import evaluate

from test_gpu_divide_and_conquer import _structured

pytestmark = pytest.mark.gpu


def _matrices(n):
    """Full rank, rank 3 n / 4, decaying, columns that are reduced already (diagonal, tridiagonal, blocks of the tiles), a last coupling across the tiles."""
    rng = np.random.default_rng(n)
    out = []
    for samples, decay in ((4 * n, False), (3 * n // 4, False), (4 * n, True)):
        X = rng.standard_normal((7, samples, n))
        if decay:
            X = X / np.arange(1, n + 1) @ np.linalg.qr(rng.standard_normal((n, n)))[0]
        out += list(X.transpose(0, 2, 1) @ X / samples + 1e-3 * np.eye(n))
    full = out[0]
    r, c = np.indices((n, n))
    out += [np.diag(np.diag(full)), np.where(abs(r - c) < 2, full, 0), np.where((r < 32) == (c < 32), full, 0),
            np.where((r == c) | ((r == 31) & (c == 32)) | ((r == 32) & (c == 31)), full, 0), np.where((r < 32) & (c < 32), full, 0)]
    return np.stack(out).astype(np.float32)


@pytest.mark.parametrize("n", range(33, 65))
def test_both_ways_of_the_reduction(n):
    import torch

    import paper_2207_04228_amd as bed

    A = np.concatenate([_matrices(n), _structured(n, n)])
    lam_o, V_o = jacobi.syevd(A)
    for batch in (256, 257):
        many = np.resize(A, (batch, n, n))
        assert bed.binding.bed_syevd_kernel(batch, n) == "dc_block_kernel<64>"
        At = torch.from_numpy(many).cuda()
        lam, V = bed.bed_syevd(At)
        alone, _ = bed.bed_syevd(At, want_vectors=False)
        lam, V, alone = lam.cpu().numpy(), V.cpu().numpy(), alone.cpu().numpy()
        assert (lam == alone).all()                    # the same numbers without eigenvectors
        acc = evaluate(A, lam[:len(A)], V[:len(A)], lam_o, V_o)
        assert acc.passes(), (n, batch, acc.worst())
        copies = batch // len(A) * len(A)              # every copy of a matrix is treated alike
        assert (lam[:copies].reshape(-1, len(A), n) == lam[:len(A)]).all() and (V[:copies].reshape(-1, len(A), n, n) == V[:len(A)]).all()


@pytest.mark.parametrize("batch", [4, 260])
@pytest.mark.parametrize("n", [33, 48, 64])
def test_non_finite_entries(n, batch):
    """A matrix with a NaN or an infinity is all NaN, its neighbours are untouched; in the first columns and in the last tile."""
    import torch

    import paper_2207_04228_amd as bed

    A = np.repeat(_matrices(n)[:1], batch, axis=0)
    A[1::4, n - 1, 0] = np.nan
    A[2::4, 33 if n > 33 else 32, 32] = np.inf
    At = torch.from_numpy(A).cuda()
    lam, V = (x.cpu().numpy() for x in bed.bed_syevd(At))
    info = bed.bed_syevd_info(At, want_rotations=False)[2].cpu().numpy()
    lost = np.isin(np.arange(batch) % 4, (1, 2))
    assert np.isnan(lam[lost]).all() and np.isnan(V[lost]).all() and (info[lost] == n).all()
    assert np.isfinite(lam[~lost]).all() and (lam[~lost] == lam[0]).all() and (V[~lost] == V[0]).all() and (info[~lost] == 0).all()
    alone = bed.bed_syevd(At, want_vectors=False)[0].cpu().numpy()
    assert np.array_equal(alone, lam, equal_nan=True)


@pytest.mark.parametrize("n", [65, 79, 95, 96, 97, 127])
def test_strips(n):
    """65 to 96 rows in three strips of 32 columns, more in four."""
    import torch

    import paper_2207_04228_amd as bed

    A = _matrices(n)
    lam_o, V_o = jacobi.syevd(A)
    At = torch.from_numpy(A).cuda()
    lam, V = (x.cpu().numpy() for x in bed.bed_syevd(At))
    alone = bed.bed_syevd(At, want_vectors=False)[0].cpu().numpy()
    assert (lam == alone).all()
    acc = evaluate(A, lam, V, lam_o, V_o)
    assert acc.passes(), (n, acc.worst())
