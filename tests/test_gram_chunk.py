"""Workspace of Gram calls whose whole state exceeds any device, or 64 bits:
a chunk of the default size, whatever the number of pairs (no GPU)."""
import ctypes

import pytest

from paper_2502_08470_amd import _lib as L


def workspace(nx, ny, dtype, algo, backward):
    p = L.SkParams(1, 4, dtype, algo, 0, 0, 0)
    return L.lib().sigkernel_gram_workspace(nx, 65, ny, 65, 3, ctypes.byref(p), backward)


@pytest.mark.parametrize("dtype", [L.SK_F32, L.SK_F64])
@pytest.mark.parametrize("backward", [0, 1])
def test_more_pairs_than_fit_take_the_default_chunk(dtype, backward):
    chunk = workspace(1 << 16, 1 << 16, dtype, 0, backward)
    assert 1 << 36 < chunk <= 160 << 30
    for bits in range(34, 62):  # 64 x 64 cells: 2^15 or 2^16 bytes of constants per pair
        assert workspace(1 << bits // 2, 1 << (bits - bits // 2), dtype, 0, backward) == chunk, bits


@pytest.mark.parametrize("backward", [0, 1])
def test_calls_that_fit_are_one_chunk(backward):
    sizes = [workspace(n, 128, L.SK_F32, 0, backward) for n in (1, 2, 64, 128)]
    assert sizes[0] < sizes[1] < sizes[2] < sizes[3] < 160 << 30
    # beyond the first pair only the pairs themselves add to it
    assert abs(sizes[3] - 2 * sizes[2]) < 16 * 256 * 2
