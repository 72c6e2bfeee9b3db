"""FP64 order 4 adjoints on both sides of the number of pairs from which a third
wave per SIMD pays: the same gradients of the same rows."""
import numpy as np
import pytest
import torch

from tests.gpu_common import bm_paths

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lx,ly", [(66, 65), (65, 64), (40, 71), (129, 90)])
def test_rows_of_a_large_call_match_smaller_calls(lx, ly):
    import paper_2502_08470_amd as sk
    print(f"adjoint waves {lx}x{ly}", flush=True)
    rng = np.random.default_rng(lx + ly)
    X, Y = (torch.tensor(bm_paths(rng, n, p, 3, 0.05), device="cuda") for n, p in ((46, lx), (45, ly)))
    gK = torch.tensor(rng.normal(size=(46, 45)), device="cuda")  # 2070 pairs, 1035 in each half
    gX, gY = sk.gram_backward(X, Y, gK, "approx", 4)
    parts = [sk.gram_backward(X[i:i + 23], Y, gK[i:i + 23], "approx", 4) for i in (0, 23)]
    tol = 2 * 1.1e-16 * 14 * (lx + ly) + 1e-13  # 2N + 6 roundings per cell along a row, both ways
    for g, r in ((gX, torch.cat([p[0] for p in parts])), (gY, parts[0][1] + parts[1][1])):
        assert (g - r).abs().max() <= tol * r.abs().max()
