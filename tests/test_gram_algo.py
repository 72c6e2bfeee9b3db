"""The rule that takes Gram calls to the strip pipeline, on both sides of its
lines: few pairs of several strips whose rows are longer than the lag between
strips, fewer where strips are short against their skew, fewer in FP64."""
import pytest
import torch

from paper_2502_08470_amd.api import gram_algo


@pytest.mark.parametrize("nx,ny,lx,ly,dtype,expected", [
    (2, 3, 130, 70, torch.float64, "pipeline"),      # below 64 pairs every several-strip call
    (7, 9, 65, 2, torch.float32, "pipeline"),
    (8, 8, 130, 150, torch.float32, "batched"),      # 64 pairs of rows below the lag
    (8, 8, 130, 250, torch.float32, "pipeline"),
    (8, 8, 64, 500, torch.float32, "batched"),       # one strip
    (8, 8, 300, 0, torch.float32, "batched"),        # no columns
    (32, 32, 256, 256, torch.float32, "pipeline"),
    (32, 48, 256, 256, torch.float32, "batched"),
    (16, 24, 256, 256, torch.float64, "pipeline"),
    (24, 32, 256, 256, torch.float64, "batched"),
    (35, 40, 120, 1500, torch.float32, "pipeline"),
    (35, 40, 120, 1500, torch.float64, "pipeline"),
    (37, 29, 150, 202, torch.float64, "batched"),
    (40, 40, 300, 100, torch.float32, "batched"),
    (23, 89, 4000, 4000, torch.float32, "pipeline"),  # 2047 pairs
    (32, 64, 4000, 4000, torch.float32, "batched"),
    (32, 64, 4000, 4000, torch.float64, "batched"),
])
def test_rule(nx, ny, lx, ly, dtype, expected):
    X = torch.empty(nx, lx + 1, 2, dtype=dtype, device="meta")
    Y = torch.empty(ny, ly + 1, 2, dtype=dtype, device="meta")
    assert gram_algo(X, Y) == expected
    assert gram_algo(X, Y, "interp") == expected
    assert gram_algo(X, Y, "fd") == gram_algo(X, Y, "fd2") == "batched"
