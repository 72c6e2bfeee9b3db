"""The terms an FP32 cell leaves out when |c| <= 2^-6 (no GPU): their size
against the cell's coefficients, for every order that takes that path."""
import math

import numpy as np
import pytest

from paper_2502_08470_amd import _lib as L

C_MAX, M_KEPT = 2.0 ** -6, 3


def rows(P, Q, c, last, kept):
    """Rows 0..last of the untruncated map (top edge) from the Toeplitz weights
    and Hankel rows up to `kept`."""
    N = len(P) - 1
    out = np.zeros(last + 1)
    for r in range(last + 1):
        for k in range(min(r, N) + 1):
            if r - k <= kept:
                out[r] += c ** (r - k) / math.factorial(r - k) * P[k]
        if r <= kept:
            out[r] += c ** r * sum(Q[k] / math.factorial(r + k) for k in range(1, N + 1))
    return out


def derivative_rows(P, Q, c, kept):
    """dA_r/dc, r = 1..N: the Toeplitz row r-1 and r c^(r-1) times the Hankel row."""
    N = len(P) - 1
    out = np.zeros(N)
    for r in range(1, N + 1):
        out[r - 1] = sum(c ** (r - 1 - k) / math.factorial(r - 1 - k) * P[k] for k in range(r) if r - 1 - k <= kept)
        if r <= kept:
            out[r - 1] += r * c ** (r - 1) * sum(Q[k] / math.factorial(r + k) for k in range(1, N + 1))
    return out


@pytest.mark.parametrize("N", range(4, 9))
@pytest.mark.parametrize("c", [C_MAX, -C_MAX, C_MAX / 7])
def test_terms_left_out_are_below_the_fp32_state(N, c):
    """Coefficients up to 1: the edge moves by less than 2^-32 (an FP32
    coefficient is rounded to 2^-24), and its slope and the derivative in c by
    less than 2^-26."""
    rng = np.random.default_rng(N)
    cases = [(np.ones(N + 1), np.ones(N + 1)), (np.ones(N + 1) * (-1.0) ** np.arange(N + 1), np.ones(N + 1))]
    cases += [tuple(rng.uniform(-1, 1, size=(2, N + 1))) for _ in range(50)]
    u = np.linspace(0, 1, 33)
    f = np.array([math.factorial(r) for r in range(N + 1)], dtype=float)
    for P, Q in cases:
        d = rows(P, Q, c, N, 10 ** 6) - rows(P, Q, c, N, M_KEPT)
        assert np.max(np.abs(np.polyval((d / f)[::-1], u))) <= 2.0 ** -32
        assert abs(np.sum(d[1:] / f[:-1])) <= 2.0 ** -26
        dd = derivative_rows(P, Q, c, 10 ** 6) - derivative_rows(P, Q, c, M_KEPT)
        assert abs(np.sum(dd / f[1:])) <= 2.0 ** -26


@pytest.mark.parametrize("N", range(4, 9))
def test_first_tail_row_is_bounded_by_its_kept_terms(N):
    """The interpolation scheme's test takes the first tail row from three
    terms against half the tail rule's limit: what they miss stays below the
    other half, and the decay condition of the tail rule holds at |c| <= 2^-6."""
    _, rmax, cmax, _ = L.interp_table(N, L.SK_F32)
    assert cmax[0] >= C_MAX
    eps = 2.0 ** -26
    P = Q = np.ones(N + 1)
    full = rows(P, Q, C_MAX, N + 1, 10 ** 6)[N + 1]
    part = rows(P, Q, C_MAX, N + 1, M_KEPT)[N + 1]
    # both edges, against the smallest scale |P_0| + |Q_0| of unit coefficients
    assert 2 * rmax[0] * 2 * (full - part) <= 0.5 * eps * 2
