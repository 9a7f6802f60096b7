"""Gradients and spectral functions of 33 to 128 rows, formed in strips of 16 columns: edges of the tiles, rows that start off 128 bits."""
import numpy as np
import pytest

from oracle import backward

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
# around whole numbers of tiles, for each count of them
SIZES = [33, 34, 36, 47, 48, 49, 63, 64, 65, 79, 80, 81, 96, 97, 100, 112, 113, 127, 128]


def _device(x, shift):
    """x on the GPU, `shift` floats behind a boundary of 128 bits."""
    import torch
    flat = torch.empty(x.size + shift, dtype=torch.float32, device="cuda")[shift:]
    return flat.view(x.shape).copy_(torch.from_numpy(x))


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", SIZES)
def test_gradients(n, shift):
    """Against float64 from the same float32 inputs.  A sum of n products rounds to about sqrt(n) U of the sum of their magnitudes:
    T1 for the products that form C, T2 for the two behind; couplings to a few U (one a term of the series)."""
    import paper_2207_04228_amd as bed

    batch = 3
    rng = np.random.default_rng(1000 + n)
    lam = np.sort(rng.uniform(0.5, 4.0, (batch, n)).astype(np.float32), axis=1)
    V = np.linalg.qr(rng.standard_normal((batch, n, n)))[0].astype(np.float32)
    G = rng.standard_normal((batch, n, n)).astype(np.float32)
    g_lam = rng.standard_normal((batch, n)).astype(np.float32)
    dl, dV, dG, dg = (_device(x, shift) for x in (lam, V, G, g_lam))
    out = _device(np.zeros_like(G), shift)
    l64, V64, G64 = (x.astype(np.float64) for x in (lam, V, G))
    norm = lambda M: np.linalg.norm(M, axis=(1, 2))
    Vt = V64.transpose(0, 2, 1)

    for fn in (backward.FN_SQRT, backward.FN_INV_SQRT):
        for floor in (1e-6, 1.0):                      # no eigenvalue below it, some
            bed.bed_spd_fn_backward(dl, dV, dG, fn, floor, grad_A=out)
            got, want = out.cpu().numpy(), backward.spd_fn_backward(l64, V64, G, fn, floor)
            Phi = backward.divided_differences(l64, fn, floor)
            sym = 0.5 * (G64 + G64.transpose(0, 2, 1))
            T1 = norm(Phi * (np.abs(Vt) @ np.abs(sym) @ np.abs(V64)))
            T2 = norm(Phi * (Vt @ sym @ V64))
            tol = 4 * np.sqrt(n) * U * (2 * T1 + 2 * T2) + 16 * U * T2
            assert (np.abs(got - want).max(axis=(1, 2)) <= tol).all(), (fn, floor)

    bed.bed_syevd_backward(dl, dV, dg, dG, grad_A=out)
    got, want = out.cpu().numpy(), backward.syevd_backward(l64, V64, g_lam, G, backward.MODE_TAYLOR)
    K = backward.coupling_taylor(l64, 9)
    M = K * (Vt @ G64)
    T1 = norm(K * (np.abs(Vt) @ np.abs(G64)))
    T2 = norm(0.5 * (M + M.transpose(0, 2, 1)) + g_lam.astype(np.float64)[:, :, None] * np.eye(n))
    tol = 4 * np.sqrt(n) * U * (T1 + 2 * T2) + (4 + 11) * U * T2
    assert (np.abs(got - want).max(axis=(1, 2)) <= tol).all()
    bed.bed_syevd_backward(dl, dV, dg, grad_A=out)                # eigenvalues alone
    want = backward.syevd_backward(l64, V64, g_lam, None)
    assert (np.abs(out.cpu().numpy() - want).max(axis=(1, 2)) <= 4 * np.sqrt(n) * U * 2 * np.linalg.norm(g_lam, axis=1)).all()


@pytest.mark.parametrize("n", [33, 36, 47, 48, 49, 52])
def test_function_from_a_decomposition_of_the_rotations(n):
    """The function of the decomposition that the same call returns; f and the eigenvalues' rounding are a few U, the product sqrt(n) U."""
    import torch

    import paper_2207_04228_amd as bed

    batch = 1025
    gen = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn(batch, 2 * n, n, generator=gen, device="cuda")
    A = torch.matmul(X.transpose(1, 2).contiguous(), X) / (2 * n)
    F, lam, V = bed.bed_spd_fn_eigh(A, bed.BED_FN_SQRT, 1e-6)[:3]
    assert not bed.binding.bed_syevd_kernel(batch, n).startswith("dc_")
    F, lam, V = (x[-3:].cpu().numpy() for x in (F, lam, V))
    f = np.sqrt(np.maximum(lam.astype(np.float64), 1e-6))
    V64 = V.astype(np.float64)
    want = (V64 * f[:, None, :]) @ V64.transpose(0, 2, 1)
    bound = (np.abs(V64) * f[:, None, :]) @ np.abs(V64).transpose(0, 2, 1)
    assert (np.abs(F - want) <= (4 * np.sqrt(n) + 8) * U * bound).all()
