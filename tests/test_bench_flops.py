"""Operation counts of bench.py's roofline (no GPU)."""
import numpy as np
import pytest

import bench


@pytest.mark.parametrize("N", range(5, 9))
def test_short_rows_count_fewer_operations(N):
    # FMA by FMA: the weights w_1..w_3 and w_4, both edges
    fma = 0
    for r in range(N + 1):
        fma += min(r, 3)                   # Toeplitz row r
        fma += N + 1 if r <= 3 else 0      # Hankel row r and its weight
    assert bench.small_cell_flops(N) == 2 * 2 * (fma + 1) + 11
    assert bench.small_cell_flops(N) < bench.fwd_cell_flops(N, 0)


def test_share_of_cells_in_small_steps():
    C = np.full((2, 128, 80), 1e-3)
    # strips follow each other: steps 64 .. 159 hold a cell in every lane
    assert bench.small_cell_share(C) == pytest.approx(96 * 64 / (128 * 80))
    C[1, 70, 30] = -0.02  # one cell: the 64 cells of its step
    assert bench.small_cell_share(C) == pytest.approx((96 * 64 - 32) / (128 * 80))
    assert bench.small_cell_share(C * 100) == 0.0
