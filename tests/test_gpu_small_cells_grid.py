"""FP32 cells of |c| <= 2^-6 (the short rows) over whole grids: their accuracy,
and that the batched sweep and the strip pipeline decide alike."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["approx", "interp"])
@pytest.mark.parametrize("order", [5, 6, 8])
def test_accuracy_over_a_large_grid(scheme, order):
    """512 x 512 cells of |c| about 0.003 against the FP64 sweep of the same
    points: with all rows the values' norm is 4.4e-8 to 5.4e-8 off and the
    gradients' 1.0e-5 to 2.9e-5; without the kept w_4 term, c^4/576 of one sign
    per cell, the values are 1.0e-7 off.  The bounds: half way in the values, a
    fifth above all rows in the gradients."""
    import paper_2502_08470_amd as sk
    print(f"small cells grid {scheme} {order}", flush=True)
    steps, d = 512, 4
    g = torch.Generator().manual_seed(1000 * order + steps)
    X, Y = (torch.cat([torch.zeros(24, 1, d), (torch.randn(24, steps, d, generator=g) * 0.0015 ** 0.5).cumsum(1)],
                      1).cuda() for _ in range(2))
    K64 = sk.gram(X.double(), Y.double(), scheme, order)
    g64 = sk.gram_backward(X.double(), Y.double(), 1 / K64, scheme, order)
    for algo in ("batched", "pipeline"):
        K = sk.gram(X, Y, scheme, order, algo=algo).double()
        assert (K - K64).norm() <= 7.7e-8 * K64.norm(), algo
        for ckpt in (2, 4):
            for a, b in zip(sk.gram_backward(X, Y, (1 / K64).float(), scheme, order, algo=algo, ckpt=ckpt), g64):
                assert (a.double() - b).norm() <= 3.5e-5 * b.norm(), (algo, ckpt)


@pytest.mark.parametrize("order", [5, 6, 7, 8])
@pytest.mark.parametrize("lx,ly", [(130, 300), (65, 65), (64, 300), (128, 72), (200, 64), (191, 201), (300, 97),
                                   (66, 3000)])
def test_both_algorithms_give_the_same_values(order, lx, ly):
    """Approximation, FP32, cells on both sides of the threshold: the batched
    sweep and the strip pipeline decide alike, to the last bit."""
    import paper_2502_08470_amd as sk
    print(f"small cells both algorithms {order} {lx}x{ly}", flush=True)
    rng = np.random.default_rng(100 * lx + ly + order)
    n, m = (24, 32) if ly < 1000 else (4, 6)
    std = np.sqrt(2.0 ** -6 / 3)  # a few cells in a hundred are larger
    for size in (std, std / 2, std / 3):
        X, Y = (torch.tensor(np.cumsum(rng.normal(0, size, (k, p + 1, 2)), 1), dtype=torch.float32, device="cuda")
                for k, p in ((n, lx), (m, ly)))
        a, b = (sk.gram(X, Y, "approx", order, algo=algo, return_exp=True) for algo in ("batched", "pipeline"))
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
