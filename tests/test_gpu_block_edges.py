"""Pairs at the edges of the sweeps' blocks of 8 steps and strips of 64 rows
(one strip, strips without idle columns, partial last strips, columns that are
no multiple of 8, the exchange): values against the FP64 oracle, gradients
against the FP64 pipelined adjoint, which takes every step alike.

Bounds: a cell's outputs carry at most 2N + 6 = 22 roundings, errors add up
along a row of at most lx + ly cells, and the adjoint doubles them; in FP32
(coefficients 0 and 1 in FP64) those of the other coefficients come in with
the weight of |c| < 0.01."""
import numpy as np
import pytest
import torch

from tests.gpu_common import bm_paths, oracle_gram, rel_err_exp

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (1, 9), (63, 8), (64, 63), (64, 64), (2, 131), (64, 200), (65, 63), (65, 64), (65, 65),
          (129, 66), (130, 71), (128, 72), (191, 73), (70, 257), (130, 701)]


def paths(lx, ly):
    rng = np.random.default_rng(1000 * lx + ly)
    X, Y = bm_paths(rng, 3, lx, 3, 0.03), bm_paths(rng, 2, ly, 3, 0.03)
    gK = torch.tensor(rng.normal(size=(3, 2)), device="cuda")
    return X.astype(np.float32), Y.astype(np.float32), gK


@pytest.mark.parametrize("lx,ly", SHAPES)
@pytest.mark.parametrize("scheme,order", [("approx", 5), ("interp", 4)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_polynomial_sweeps_and_adjoints(lx, ly, scheme, order, dtype):
    import paper_2502_08470_amd as sk
    print(f"block edges {lx}x{ly} {scheme} {order} {dtype}", flush=True)
    X, Y, gK = paths(lx, ly)
    Xt, Yt = torch.tensor(X, device="cuda", dtype=dtype), torch.tensor(Y, device="cuda", dtype=dtype)
    m, e = oracle_gram(X, Y, scheme, order)
    n = 22 * (lx + ly)
    # (the oracle's own per-cell interpolation systems are a few 1e-17 off per cell)
    tol = 2e-5 if dtype == torch.float32 else 1.1e-16 * n + 1e-12 + 4e-17 * lx * ly
    K, E = sk.gram(Xt, Yt, scheme, order, algo="batched", return_exp=True)
    assert rel_err_exp(K.cpu().numpy(), E.cpu().numpy(), m, e).max() <= tol
    ref = sk.gram_backward(Xt.double(), Yt.double(), gK, scheme, order, algo="pipeline")
    gtol = 1e-5 if dtype == torch.float32 else 2 * 1.1e-16 * n + 1e-13
    for ckpt in (2, 4) if dtype == torch.float32 else (2,):
        for g, r in zip(sk.gram_backward(Xt, Yt, gK, scheme, order, algo="batched", ckpt=ckpt), ref):
            assert (g.double() - r).abs().max() <= gtol * r.abs().max(), ckpt


@pytest.mark.parametrize("lx,ly", SHAPES)
@pytest.mark.parametrize("scheme", ["fd", "fd2"])
def test_finite_difference_sweeps(lx, ly, scheme):
    import paper_2502_08470_amd as sk
    print(f"block edges {lx}x{ly} {scheme}", flush=True)
    X, Y, _ = paths(lx, ly)
    for lam in (0, 1):
        m, e = oracle_gram(X, Y, scheme, lam)
        Xt, Yt = (torch.tensor(v, device="cuda", dtype=torch.float64) for v in (X, Y))
        K, E = sk.gram(Xt, Yt, scheme, lam, algo="batched", return_exp=True)
        # every node sums three neighbours: an error of a few units per cell,
        # which adds up over the cells of the (refined) grid
        tol = 1e-11 + 2e-16 * lx * ly * 4.0 ** lam
        assert rel_err_exp(K.cpu().numpy(), E.cpu().numpy(), m, e).max() <= tol, lam
