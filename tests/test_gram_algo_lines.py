"""The Gram calls' choice of algorithm by sweep precision, direction and order
(no GPU): shapes on which the two algorithms' times are 20% or more apart."""
import pytest
import torch

from paper_2502_08470_amd import api


def choice(dtype, nx, ny, lx, ly, order, **kw):
    X = torch.empty(nx, lx + 1, 2, dtype=dtype, device="meta")
    Y = torch.empty(ny, ly + 1, 2, dtype=dtype, device="meta")
    return api.gram_algo(X, Y, "approx", order, **kw)


@pytest.mark.parametrize("dtype,kw", [(torch.float64, {}), (torch.float32, {"sweep": "f64"})])
def test_lines_follow_the_sweep(dtype, kw):
    # milliseconds (batched, pipelined) of FP64 sweeps
    assert choice(dtype, 25, 40, 256, 256, 4, **kw) == "batched"                     # 2.20, 2.75 (FP32: pipeline)
    assert choice(dtype, 25, 40, 1000, 300, 8, backward=False, **kw) == "pipeline"   # 6.82, 4.84
    assert choice(dtype, 34, 50, 66, 500, 4, **kw) == "batched"                      # 3.21, 4.06
    assert choice(dtype, 30, 40, 256, 256, 8, **kw) == "pipeline"                    # 7.15, 5.84
    assert choice(dtype, 30, 40, 1000, 300, 8, **kw) == "pipeline"                   # 32.7, 24.3
    assert choice(dtype, 40, 51, 1000, 300, 6, **kw) == "batched"                    # 25.1, 36.5


def test_forwards_have_their_own_line():
    assert choice(torch.float32, 25, 40, 256, 256, 4) == "pipeline"
    assert choice(torch.float32, 40, 51, 66, 2000, 8, backward=False) == "pipeline"  # 3.52, 2.59
    assert choice(torch.float32, 20, 35, 66, 200, 4, backward=False) == "batched"    # 0.16, 0.22
    assert choice(torch.float32, 40, 51, 500, 500, 8) == "pipeline"                  # 14.5, 11.9


@pytest.mark.parametrize("sweep", ["native", "f64"])
@pytest.mark.parametrize("grad", [False, True])
def test_autograd_asks_for_its_call(monkeypatch, sweep, grad):
    seen = []
    monkeypatch.setattr(api, "gram_algo", lambda *a: seen.append(a[2:]) or "batched")
    monkeypatch.setattr(api, "gram", lambda X, Y, *a, **k: X.new_zeros(X.shape[0], Y.shape[0]))
    monkeypatch.setattr(api, "gram_state_size", lambda *a: 1 << 62)
    monkeypatch.setattr(api, "_state_budget", lambda device: 0)
    X, Y = torch.zeros(8, 131, 2, requires_grad=grad), torch.zeros(9, 151, 2)
    api.sig_gram(X, Y, "approx", 6, sweep=sweep)
    assert seen == [("approx", 6, sweep, grad)]
