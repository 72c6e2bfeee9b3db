"""Increment Gram kernels at the edges of their row blocks, strips and
coordinate paddings, against products of the same increments in FP64.

Bounds: a constant is a sum of d products, each step of which rounds once, and
the refinement's scale is a power of two; the BF16 split drops three products
below 2^-24 of |a||b| and rounds its six partial sums of 16 coordinates."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def check(lx, ly, d, dtype, mode, roundings):
    import paper_2502_08470_amd as sk
    print(f"gram edges {lx}x{ly} d={d} {dtype} {mode}", flush=True)
    rng = np.random.default_rng(7 * lx + ly + d)
    X = torch.tensor(rng.normal(size=(2, lx + 1, d)), dtype=dtype)
    Y = torch.tensor(rng.normal(size=(3, ly + 1, d)), dtype=dtype)
    x, y = X.diff(dim=1).double().numpy(), Y.diff(dim=1).double().numpy()
    C = sk.cell_constants(X.cuda(), Y.cuda(), gram_mode=mode).cpu().double().numpy()
    ref = np.einsum("aik,bjk->abij", x, y)
    mag = np.einsum("aik,bjk->abij", np.abs(x), np.abs(y))
    eps = 2.0 ** -24 if dtype == torch.float32 else 2.0 ** -53
    assert np.all(np.abs(C - ref) <= roundings * eps * mag)


@pytest.mark.parametrize("lx,ly", [(1, 1), (1, 7), (5, 3), (7, 8), (64, 7), (65, 8), (130, 9), (63, 300), (200, 61),
                                   (66, 64)])
@pytest.mark.parametrize("d", [1, 4, 5, 8, 9, 12, 16])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_direct_gram(lx, ly, d, dtype):
    check(lx, ly, d, dtype, "native", d + 2)


@pytest.mark.parametrize("lx,ly", [(700, 65), (65, 700), (129, 640), (1, 800), (800, 1)])
@pytest.mark.parametrize("d", [5, 17, 33, 48])
def test_split_bands(lx, ly, d):
    check(lx, ly, d, torch.float32, "bf16x3", d + 12)
