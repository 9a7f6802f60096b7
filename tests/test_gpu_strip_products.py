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


def inputs(n, batch=3):
    rng = np.random.default_rng(1000 + n)
    lam = np.sort(rng.uniform(0.5, 4.0, (batch, n)).astype(np.float32), axis=1)
    V = np.linalg.qr(rng.standard_normal((batch, n, n)))[0].astype(np.float32)
    return lam, V, rng.standard_normal((batch, n, n)).astype(np.float32), rng.standard_normal((batch, n)).astype(np.float32)


def _norm(M):
    return np.linalg.norm(M, axis=(1, 2))


def bar(n, couplings, G, M, products, roundings):
    """Frobenius bound of the error of V (couplings o C) V^T, C formed from G by `products` products with V (orthogonal: C has G's norm).
    A sum of n terms of random signs rounds by about sqrt(n / 6) U of its result's size, entry by entry, taken as sqrt(n) U; what C carries meets the couplings
    entry by entry, so their mean square; two products follow, and the couplings take `roundings` U themselves."""
    return U * (np.sqrt(n) * (products * _norm(G) * _norm(couplings) / n + 2 * _norm(M)) + roundings * _norm(M))


def agree(got, want, bound):
    """Within the bound as a whole, and no entry more than eight times its mean."""
    n = got.shape[-1]
    error = got - want
    return (_norm(error) <= bound).all() and (np.abs(error).max(axis=(1, 2)) <= 8 * bound / n).all()


def function_bar(lam, V, G, fn, floor):
    Phi = backward.divided_differences(lam, fn, floor)
    sym = 0.5 * (G + G.transpose(0, 2, 1))
    return bar(lam.shape[1], Phi, sym, Phi * (V.transpose(0, 2, 1) @ sym @ V), 2, 8)


def decomposition_bar(lam, V, g_lam, G):
    """The series of degree 9 adds a rounding a term."""
    n = lam.shape[1]
    K = backward.coupling_taylor(lam, 9)
    M = K * (V.transpose(0, 2, 1) @ G)
    M = 0.5 * (M + M.transpose(0, 2, 1)) + g_lam[:, :, None] * np.eye(n)
    return bar(n, K, G, M, 1, 4 + 11)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", SIZES)
def test_gradients(n, shift):
    """Against float64 from the same float32 inputs.  tests/test_strip_bar.py shows on the CPU that no product with operands of less than
    32 bits is within these bounds."""
    import paper_2207_04228_amd as bed

    lam, V, G, g_lam = inputs(n)
    dl, dV, dG, dg = (_device(x, shift) for x in (lam, V, G, g_lam))
    out = _device(np.zeros_like(G), shift)
    l64, V64, G64, g64 = (x.astype(np.float64) for x in (lam, V, G, g_lam))

    def check(want, bound, what):
        got = out.cpu().numpy().astype(np.float64)
        print(f"n={n} shift={shift} {what}: {(_norm(got - want) / bound).max():.3f} of the bound, "
              f"largest entry {(np.abs(got - want).max(axis=(1, 2)) / (8 * bound / n)).max():.3f}", flush=True)
        assert agree(got, want, bound), what

    for fn in (backward.FN_SQRT, backward.FN_INV_SQRT):
        for floor in (1e-6, 1.0):                      # no eigenvalue below it, some
            bed.bed_spd_fn_backward(dl, dV, dG, fn, floor, grad_A=out)
            check(backward.spd_fn_backward(l64, V64, G64, fn, floor), function_bar(l64, V64, G64, fn, floor), (fn, floor))
    bed.bed_syevd_backward(dl, dV, dg, dG, grad_A=out)
    check(backward.syevd_backward(l64, V64, g64, G64, backward.MODE_TAYLOR), decomposition_bar(l64, V64, g64, G64), "decomposition")
    bed.bed_syevd_backward(dl, dV, dg, grad_A=out)                # eigenvalues alone
    check(backward.syevd_backward(l64, V64, g64, None), 2 * np.sqrt(n) * U * np.linalg.norm(g64, axis=1), "eigenvalues alone")


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
