"""Paths with a NaN or an infinity: their pairs are not finite, and every other
pair keeps its bits (lanes without a cell take part in the sweeps' votes, and
their constants may be NaN where the other path's are)."""
import numpy as np
import pytest
import torch

from tests.gpu_common import bm_paths

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lx,ly", [(130, 300), (64, 300), (65, 65), (30, 90), (300, 40)])
@pytest.mark.parametrize("scheme,order,dtype", [("approx", 5, torch.float32), ("interp", 6, torch.float32),
                                                ("approx", 6, torch.float64), ("interp", 4, torch.float64),
                                                ("fd", 0, torch.float32), ("fd2", 1, torch.float64)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_other_pairs_keep_their_bits(lx, ly, scheme, order, dtype, bad):
    import paper_2502_08470_amd as sk
    print(f"non-finite {lx}x{ly} {scheme} {order} {dtype} {bad}", flush=True)
    rng = np.random.default_rng(lx + 7 * ly)
    X, Y = (torch.tensor(bm_paths(rng, n, p, 3, 0.05).astype(np.float32), device="cuda", dtype=dtype)
            for n, p in ((4, lx), (3, ly)))
    gK = torch.tensor(rng.normal(size=(4, 3)), device="cuda", dtype=dtype)
    keep = [0, 2, 3]
    for at in (0, lx // 2, lx):
        Z = X.clone()
        Z[1, at, 1] = bad
        for algo in ("batched",) if scheme.startswith("fd") else ("batched", "pipeline"):
            K, K0 = sk.gram(Z, Y, scheme, order, algo=algo), sk.gram(X, Y, scheme, order, algo=algo)
            assert torch.equal(K[keep], K0[keep]) and not torch.isfinite(K[1]).any(), (at, algo)
            if not scheme.startswith("fd"):
                g, _ = sk.gram_backward(Z, Y, gK, scheme, order, algo=algo)
                g0, _ = sk.gram_backward(X, Y, gK, scheme, order, algo=algo)
                assert torch.equal(g[keep], g0[keep]), (at, algo)
    sk.device_status()  # (a cell that is not a number may report the end of the tail)
