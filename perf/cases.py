"""The work that users of this library have it do, as measurable cases.

The library decomposes mini-batches of small symmetric matrices (n <= 128) inside larger
programs: whitening layers (decorrelated batch normalisation, whitening-and-colouring transform),
covariance pooling, spectra of feature covariances, and eigendecompositions kept for several later
uses.  The cases take that work through the public entry points over the range of sizes the
repository's configurations, tests and benchmark name: from 16 matrices of 4x4, where one launch
and its host path are everything, to 16384 of 32x32 and 256 of 128x128.

Kinds of use:
  whiten      out = A^(-1/2), inference (one fused call, no gradient)
  train_inv   A^(-1/2) as a layer: forward and backward through autograd
  train_sqrt  A^(1/2) as a layer (covariance pooling): forward and backward through autograd
  train_eigh  (lambda, V) as a layer with the series gradient of degree 9: forward and backward
  values      eigenvalues only
  eigh        (lambda, V) once, then the gradient of a spectral function from them: the program
              that keeps the decomposition.  Signs of eigenvectors, and bases of repeated
              eigenvalues, are free, so V itself is not comparable between two correct
              implementations; what the program makes of it is.

Inputs are feature covariances X^T X / samples + ridge I, X Gaussian.  `samples` below n gives the
repeated eigenvalues of a rank-deficient covariance (all at the ridge), `decay` a power-law
spectrum (features of standard deviation 1/i, rotated).
"""
import math

import numpy as np
import torch

import paper_2207_04228_amd as bed

FLOOR = 1e-6        # eigenvalue floor of the spectral functions
MAX_BATCH = 65536
MAX_CUBE = 16384 * 32 ** 3      # batch * n^3 of the largest listed cases
KINDS = ("whiten", "train_inv", "train_sqrt", "train_eigh", "values", "eigh")


def listed():
    def case(name, kind, batch, n, samples, ridge=1e-3, decay=False):
        return {"name": name, "kind": kind, "batch": batch, "n": n, "samples": samples, "ridge": ridge, "decay": decay}

    return [
        # 16 groups of 4 channels: the smallest call, one launch of a few microseconds
        case("whiten_16x4", "whiten", 16, 4, 16),
        # decorrelated batch normalisation with 8 groups of 8 channels, one training step
        case("train_inv_8x8", "train_inv", 8, 8, 128),
        # whitening half of a whitening-and-colouring transform, 64 groups of 16
        case("whiten_64x16", "whiten", 64, 16, 256),
        # the benchmark's dominant call: 512 matrices of 32x32
        case("eigh_512x32", "eigh", 512, 32, 128, 1e-4),
        # covariance pooling of tokens, 768 matrices of 36x36, one training step
        case("train_sqrt_768x36", "train_sqrt", 768, 36, 196),
        # spectra of 1000 covariances of an odd size
        case("values_1000x23", "values", 1000, 23, 92),
        # very many tiny matrices
        case("eigh_65536x4", "eigh", MAX_BATCH, 4, 64),
        # decaying spectra, differentiable decomposition
        case("train_eigh_4096x16", "train_eigh", 4096, 16, 64, 1e-3, True),
        # more channels than samples: a cluster of 15 equal eigenvalues per matrix
        case("eigh_256x64", "eigh", 256, 64, 49, 1e-2),
        # few large matrices of a ragged size: one training step of a pooling layer
        case("train_sqrt_50x100", "train_sqrt", 50, 100, 400),
        # the largest matrices the library takes
        case("eigh_256x128", "eigh", 256, 128, 512),
        # a full chip: whitening layer over 16384 groups of 32 channels, one training step
        case("train_inv_16384x32", "train_inv", 16384, 32, 128),
    ]


def draw(rng):
    n = min(128, max(2, int(round(math.exp(rng.uniform(math.log(2), math.log(128.999)))))))
    most = min(MAX_BATCH, MAX_CUBE // n ** 3)
    batch = max(1, min(most, int(round(math.exp(rng.uniform(0.0, math.log(most)))))))
    kind = KINDS[rng.randrange(len(KINDS))]
    samples, decay = 4 * n, False
    if kind != "train_eigh" and n >= 6 and rng.random() < 0.25:
        samples = 3 * n // 4
    elif rng.random() < 0.25:
        decay = True
    return {"kind": kind, "batch": batch, "n": n, "samples": samples,
            "ridge": 1e-2 if samples < n else 1e-3, "decay": decay}


def prepare(case, seed):
    batch, n, samples = case["batch"], case["n"], case["samples"]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    mix = None
    if case["decay"]:
        # features of standard deviation 1/i seen in a rotated basis
        basis = torch.linalg.qr(torch.randn(n, n, generator=torch.Generator().manual_seed(seed)))[0].cuda()
        mix = (1.0 / torch.arange(1, n + 1, device="cuda", dtype=torch.float32))[:, None] * basis
    A = torch.empty(batch, n, n, device="cuda")
    step = max(1, (1 << 25) // (samples * n))     # keep the samples small beside the result
    for lo in range(0, batch, step):
        X = normal(min(step, batch - lo), samples, n)
        if mix is not None:
            X = torch.matmul(X, mix)
        A[lo:lo + step] = torch.matmul(X.transpose(1, 2).contiguous(), X) / samples
    A = (0.5 * (A + A.transpose(1, 2))).contiguous()
    A.diagonal(dim1=1, dim2=2).add_(case["ridge"])
    state = {"kind": case["kind"], "A": A}
    if case["kind"] in ("train_inv", "train_sqrt", "train_eigh"):
        A.requires_grad_(True)
    if case["kind"] in ("train_inv", "train_sqrt", "eigh"):
        state["G"] = normal(batch, n, n)                       # upstream gradient
    if case["kind"] == "train_eigh":
        state["g_lam"], state["weight"] = normal(batch, n), normal(batch, n, n)
    return state


def run(state):
    kind, A = state["kind"], state["A"]
    if kind == "whiten":
        out, _, _ = bed.bed_spd_fn(A, bed.BED_FN_INV_SQRT, FLOOR)
        return out
    if kind == "values":
        lam, _ = bed.bed_syevd(A, want_vectors=False)
        return lam
    if kind == "eigh":
        lam, V = bed.bed_syevd(A)
        return lam, bed.bed_spd_fn_backward(lam, V, state["G"], bed.BED_FN_SQRT, FLOOR)
    if kind == "train_eigh":
        lam, V = bed.autograd.eigh(A)
        # loss = <g_lam, lambda> + 1/2 sum(weight * V^2), which no choice of signs changes
        (grad,) = torch.autograd.grad((lam, V), A, (state["g_lam"], state["weight"] * V.detach()))
        return lam.detach(), grad
    layer = bed.autograd.spd_inv_sqrt if kind == "train_inv" else bed.autograd.spd_sqrt
    out = layer(A, FLOOR)
    (grad,) = torch.autograd.grad(out, A, state["G"])
    return out.detach(), grad


def work(case):
    b, n, kind = case["batch"], case["n"], case["kind"]
    mats, vecs = {"whiten": (2, 0), "values": (1, 1), "eigh": (3, 1), "train_eigh": (3, 2)}.get(kind, (4, 0))
    # symmetric reduction 4/3 n^3; with eigenvectors 9 n^3 in all; V f V^T of a symmetric result n^3;
    # the gradients are four (three for train_eigh) n x n x n products
    cubes = {"whiten": 10, "values": 4 / 3, "eigh": 17, "train_eigh": 15}.get(kind, 18)
    return {"bytes": 4 * b * (mats * n * n + vecs * n), "flops": cubes * b * n ** 3}


def tolerance(case):
    # four times (largest single error: four to eight times) what the library differs by from the
    # same formulas in float64, over 130 drawn cases of at most 6e7 for batch * n^3
    if case["kind"] == "values":
        return {"rel": 2.5e-6, "max": 1e-5}
    if case["kind"] == "train_eigh":
        return {"rel": 2e-3, "max": 0.1}        # close pairs of eigenvalues: eigenvectors to 1e-7 / gap
    if case["samples"] < case["n"]:
        return {"rel": 2e-4, "max": 2e-3}       # eigenvalues at 1e-2 / ||A||, errors at 1e-7 ||A||
    if case["decay"]:
        return {"rel": 4e-5, "max": 8e-4}
    return {"rel": 4e-5, "max": 2e-4}


def _couplings(lam, degree):
    """[batch, n, n] antisymmetric K_ij: the series of 1 / (lam_j - lam_i) in the ratio smaller / larger magnitude."""
    a, b = lam[:, :, None], lam[:, None, :]
    later = np.triu(np.ones((lam.shape[1],) * 2, dtype=bool), 1)
    big_b = (np.abs(b) > np.abs(a)) | ((np.abs(b) == np.abs(a)) & later)
    den, num = np.where(big_b, b, a), np.where(big_b, a, b)
    K = sum((num / den) ** k for k in range(degree + 1)) / den
    return np.where(big_b, K, -K) * (1.0 - np.eye(lam.shape[1]))


def exact(case, seed):
    state = prepare(case, seed)
    host = {k: v.detach().double().cpu().numpy() for k, v in state.items() if isinstance(v, torch.Tensor)}
    kind, total = state["kind"], case["batch"]
    parts = []
    for lo in range(0, total, 2048):
        A, *rest = (host[k][lo:lo + 2048] for k in ("A", "G", "g_lam", "weight") if k in host)
        lam, V = np.linalg.eigh(A)
        if kind == "values":
            parts.append((lam,))
            continue
        Vt = np.ascontiguousarray(V.transpose(0, 2, 1))
        if kind == "train_eigh":
            g_lam, weight = rest
            C = _couplings(lam, 9) * (Vt @ (weight * V))
            C = 0.5 * (C + C.transpose(0, 2, 1))
            C[:, range(case["n"]), range(case["n"])] = g_lam
            parts.append((lam, V @ C @ Vt))
            continue
        root = np.sqrt(np.maximum(lam, FLOOR))
        inverse = kind in ("whiten", "train_inv")
        out = (V * (1.0 / root if inverse else root)[:, None, :]) @ Vt
        if kind == "whiten":
            parts.append((out,))
            continue
        # divided differences of f(max(x, floor)); every eigenvalue lies above the floor here
        assert lam.min() > FLOOR
        si, sj = root[:, :, None], root[:, None, :]
        phi = -1.0 / (si * sj * (si + sj)) if inverse else 1.0 / (si + sj)
        G = rest[0]
        grad = V @ (phi * (Vt @ (0.5 * (G + G.transpose(0, 2, 1))) @ V)) @ Vt
        parts.append((lam if kind == "eigh" else out, grad))
    outs = tuple(torch.from_numpy(np.concatenate(p)) for p in zip(*parts))
    return outs[0] if kind in ("whiten", "values") else outs
