"""Batched adjoints of orders and shapes that take kernels of their own: the
exchange of long pairs (more columns than the adjoint's ring) with full and
partial last strips, FP64 orders 6 to 8 of both schemes, FP32 interpolation;
against the FP64 pipelined adjoint, which takes every step alike.

Bounds as in the block-edge test: 2N + 6 roundings per cell along a row of
lx + ly cells, doubled by the adjoint; in FP32 with the weight of |c| < 0.01."""
import numpy as np
import pytest
import torch

from tests.gpu_common import bm_paths

pytestmark = pytest.mark.gpu

LONG32 = [(128, 1400), (65, 1401), (130, 1447)]  # FP32 order 5: 1389 columns in the ring
SHORT = [(64, 200), (65, 64), (129, 66), (130, 71), (191, 73), (300, 40)]
LONG64 = [(128, 704), (65, 701), (130, 1447)]    # FP64 orders 6..8: 648, 572 and 512


def check(lx, ly, scheme, order, dtype):
    import paper_2502_08470_amd as sk
    print(f"adjoint edges {lx}x{ly} {scheme} {order} {dtype}", flush=True)
    rng = np.random.default_rng(1000 * lx + ly + order)
    X, Y = (torch.tensor(bm_paths(rng, n, p, 3, 0.03).astype(np.float32), device="cuda", dtype=dtype)
            for n, p in ((3, lx), (2, ly)))
    gK = torch.tensor(rng.normal(size=(3, 2)), device="cuda")
    ref = sk.gram_backward(X.double(), Y.double(), gK, scheme, order, algo="pipeline")
    n = (2 * order + 6) * (lx + ly)
    tol = 2 * n * 2.0 ** -24 * 0.01 if dtype == torch.float32 else 2 * 1.1e-16 * n + 1e-13
    for ckpt in (2, 4) if dtype == torch.float32 else (2,):
        for g, r in zip(sk.gram_backward(X, Y, gK, scheme, order, algo="batched", ckpt=ckpt), ref):
            assert (g.double() - r).abs().max() <= tol * r.abs().max(), ckpt


@pytest.mark.parametrize("lx,ly", LONG32)
@pytest.mark.parametrize("scheme,order", [("approx", 5), ("approx", 8), ("interp", 6)])
def test_fp32_exchange(lx, ly, scheme, order):
    check(lx, ly, scheme, order, torch.float32)


@pytest.mark.parametrize("lx,ly", SHORT)
@pytest.mark.parametrize("order", [6, 7, 8])
def test_fp32_interpolation(lx, ly, order):
    check(lx, ly, "interp", order, torch.float32)


@pytest.mark.parametrize("lx,ly", SHORT + LONG64)
@pytest.mark.parametrize("scheme", ["approx", "interp"])
@pytest.mark.parametrize("order", [6, 7, 8])
def test_fp64_orders(lx, ly, scheme, order):
    check(lx, ly, scheme, order, torch.float64)


@pytest.mark.parametrize("lx,ly", [(64, 200), (66, 66), (130, 71), (129, 300)])
@pytest.mark.parametrize("second", [False, True])
@pytest.mark.parametrize("lam", [0, 1])
def test_fp32_finite_differences(lx, ly, second, lam):
    """Every node sums three neighbours: one rounding each, which add up over
    the cells of the refined grid."""
    import paper_2502_08470_amd as sk
    print(f"fd edges {lx}x{ly} {second} {lam}", flush=True)
    rng = np.random.default_rng(lx + ly)
    X, Y = (torch.tensor(bm_paths(rng, n, p, 3, 0.03).astype(np.float32), device="cuda") for n, p in ((3, lx), (2, ly)))
    scheme = "fd2" if second else "fd"
    K = sk.gram(X, Y, scheme, lam).double()
    R = sk.gram(X.double(), Y.double(), scheme, lam)
    assert ((K - R) / R).abs().max() <= 2.0 ** -23 * lx * ly * 4 ** lam
