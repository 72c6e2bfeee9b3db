"""The rows of small |c| over whole grids (no GPU): a FP64 model of the cell
map with the constants of the device header, the kept w_4 term among them.
What the rows leave out must stay below the rounding of an FP32 value; without
the kept term it does not."""
import math
import os
import re

import numpy as np
import pytest

from paper_2502_08470_amd import build as B


def header(name):
    src = open(os.path.join(B.CSRC, "sk_device.h")).read()
    return eval(re.search(rf"#define {name} (.*)", src).group(1), {}, {})


SMALL_C, SMALL_M = header("SK_SMALL_C"), header("SK_SMALL_M")


def cell(P, Q, c, kept, corner):
    """Right and top edge (coefficients times n!) of a cell with bottom edge P
    and left edge Q: Toeplitz weights and Hankel rows up to `kept`, and the next
    weight's term of the corner value."""
    N = len(P) - 1
    out = []
    for a, b in ((P, Q), (Q, P)):
        o = np.zeros(N + 1)
        for r in range(N + 1):
            for k in range(r + 1):
                if r - k <= kept:
                    o[r] += c ** (r - k) / math.factorial(r - k) * a[k]
            if r <= kept:
                o[r] += c ** r * sum(b[k] / math.factorial(r + k) for k in range(1, N + 1))
        if corner:
            o[kept + 1] += c ** (kept + 1) / math.factorial(kept + 1) * a[0]
        out.append(o)
    return out


def value(N, n, sign, kept, corner):
    """k over n x n cells with constants SMALL_C sign_ij."""
    left = [np.eye(1, N + 1)[0] for _ in range(n)]
    for i in range(n):
        P = np.eye(1, N + 1)[0]
        for j in range(n):
            P, left[j] = cell(P, left[j], SMALL_C * sign(i, j), kept, corner)
    f = np.array([1 / math.factorial(r) for r in range(N + 1)])
    return 0.5 * (P @ f + left[-1] @ f)


@pytest.mark.parametrize("N", [5, 8])
def test_what_the_rows_leave_out_over_a_grid(N):
    # steps to and fro: paths within one unit of length, so that k stays near 1
    sign = lambda i, j: (-1) ** (i // 8) * (-1) ** (j // 8)
    n = 96
    full = value(N, n, sign, N, False)
    short = value(N, n, sign, SMALL_M, True)
    cut = value(N, n, sign, SMALL_M, False)
    assert abs(short / full - 1) <= 2.0 ** -24
    # c^4/576 per cell of one sign, of the kernel's mean value over the grid (1 to 2.3)
    drift = abs(cut / full - 1)
    assert 0.3 <= drift / (n * n * SMALL_C ** 4 / 576) <= 3
