"""Merges of the divide and conquer whose block is far smaller than the matrix: a root's iteration runs in units of the merge (its rho), so the
smallest distance that deflation leaves (about 1e-17 of the matrix) has a third power, and a block's size costs no evaluations."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BATCH = 256


def _matrices(n, size, spread):
    """Uncoupled halves: size * (I + spread * noise), eigenvalues about `spread` apart within a few percent of it, and one of norm one."""
    rng = np.random.default_rng(8100 + n)
    h = n // 2
    A = np.zeros((BATCH, n, n))
    noise = rng.standard_normal((BATCH, h, h))
    A[:, :h, :h] = size * (np.eye(h) + spread * 0.5 * (noise + noise.transpose(0, 2, 1)))
    X = rng.standard_normal((BATCH, 4 * (n - h), n - h))
    A[:, h:, h:] = X.transpose(0, 2, 1) @ X / (4 * (n - h))
    return A.astype(np.float32)


def _microseconds(A):
    import torch
    from paper_2207_04228_amd import binding
    lam, V, info, _ = binding.bed_syevd_info(A, want_rotations=False)
    assert (info == 0).all()
    for _ in range(20):
        binding.bed_syevd(A, lam, V)
    binding.bed_timing_begin(30)
    binding.bed_timing_arm(True)
    for _ in range(30):
        binding.bed_syevd(A, lam, V)
    return float(binding.bed_timing_end(30)[0].min()), lam, V


@pytest.mark.parametrize("n", [16, 32, 64, 128])
def test_small_blocks_take_no_longer(n):
    """With third powers in units of the matrix, which overflowed, these launches took 1.2 (128 rows) to 1.6 times (16 and 32) as long."""
    import torch
    h = n // 2
    one, _, _ = _microseconds(torch.from_numpy(_matrices(n, 1.0, 1e-2)).cuda())
    # at 1e-12 and 1e-3 deflation rotates so many close pairs, one after the other, that this shows
    for size, spread in ((1e-8, 1e-3), (1e-10, 1e-2), (1e-10, 1e-3), (1e-12, 1e-2)):
        A = _matrices(n, size, spread)
        us, lam, V = _microseconds(torch.from_numpy(A).cuda())
        print(f"n={n}: block of norm one {one:.1f} us, block of {size:g}, spread {spread:g}: {us:.1f} us", flush=True)
        got = lam.double().cpu().numpy()
        want = np.linalg.eigvalsh(A.astype(np.float64))
        assert (np.abs(got - want) <= 1e-5 * want[:, -1:]).all()
        assert us <= 1.15 * one, (n, size, spread)
