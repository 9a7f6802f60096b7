"""The bounds of tests/test_gpu_strip_products.py on the CPU: a float32 evaluation of the same chains is within them, one with a single product of
operands rounded to fewer bits (bfloat16: 8, TF32: 11) is not, at any size."""
import numpy as np
import pytest
from oracle import backward
from test_gpu_strip_products import SIZES, agree, decomposition_bar, function_bar, inputs


def _fewer(x, bits):
    """x rounded to `bits` significant bits."""
    m, e = np.frexp(x)
    return np.ldexp(np.round(np.ldexp(m, bits)), e - bits)


def _chain(lam, V, G, form, low, bits):
    """V form(C) V^T in float32, product `low` (from 0) with operands of `bits` bits; form also gets what is left of the count of products."""
    count = [0]

    def mul(X, Y):
        X, Y = X.astype(np.float32), Y.astype(np.float32)
        if count[0] == low:
            X, Y = _fewer(X, bits).astype(np.float32), _fewer(Y, bits).astype(np.float32)
        count[0] += 1
        return X @ Y

    Vt = V.transpose(0, 2, 1)
    return mul(mul(V, form(mul, Vt, V, G).astype(np.float32)), Vt), count[0]


@pytest.mark.parametrize("n", SIZES)
def test_bounds(n):
    lam, V, G, g_lam = inputs(n)
    l64, V64, G64, g64 = (x.astype(np.float64) for x in (lam, V, G, g_lam))
    cases = []
    for fn in (backward.FN_SQRT, backward.FN_INV_SQRT):
        for floor in (1e-6, 1.0):
            Phi = backward.divided_differences(l64, fn, floor)
            cases.append((lambda mul, Vt, V, G, Phi=Phi: Phi * mul(Vt, mul(0.5 * (G + G.transpose(0, 2, 1)), V)),
                          backward.spd_fn_backward(l64, V64, G64, fn, floor), function_bar(l64, V64, G64, fn, floor)))
    K = backward.coupling_taylor(l64, 9)

    def decomposition(mul, Vt, V, G):
        C = mul(Vt, G)
        return 0.5 * K * (C - C.transpose(0, 2, 1)) + g64[:, :, None] * np.eye(n)

    cases.append((decomposition, backward.syevd_backward(l64, V64, g64, G64, backward.MODE_TAYLOR), decomposition_bar(l64, V64, g64, G64)))
    for form, want, bound in cases:
        got, products = _chain(lam, V, G, form, -1, 24)
        assert agree(got, want, bound)
        wrong = got.copy()
        wrong[:, n - 1, 0] += 16 * bound / n
        assert not agree(wrong, want, bound)           # one entry off
        for low in range(products):
            for bits in (8, 11, 16):
                assert not agree(_chain(lam, V, G, form, low, bits)[0], want, bound), (low, bits)
