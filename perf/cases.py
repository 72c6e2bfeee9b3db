"""Performance cases: signature-kernel work as a user's program has it done.

A case is one call (or one training step) through the package's public entry
points, on synthetic Brownian paths drawn on the GPU from a seed.  Paths are
normalised as users do (increments of standard deviation vol / sqrt(steps) per
coordinate), which also keeps FP32 results well conditioned, except where a
case says otherwise.

Kinds of case ("op"):
  gram    Gram matrix, forward only (inference, kernel ridge regression)
  train   differentiable Gram matrix: K and the gradients of sum(W * K)
  log     kernels beyond the FP32 range: log2 |K| of a Gram call with exponents
          and the gradients of sum(log2 |K|), FP32 points swept in FP64
  pairs   one-shot kernels of a ragged pair list (offsets known at the call)
  plan    forward and backward of a plan kept for a fixed ragged batch
  mmd     MMD^2 of two path sets and its gradients
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2502_08470_amd as sk
from paper_2502_08470_amd import _lib

_DT = {"f32": torch.float32, "f64": torch.float64}


def _case(name, op, scheme, order, dtype, nx, lx, ny, ly, d, vol=0.5, **kw):
    """lx, ly: points per path (ragged lists: the range lo..lx, lo..ly)."""
    c = {"op": op, "scheme": scheme, "order": order, "dtype": dtype, "nx": nx, "lx": lx, "ny": ny,
         "ly": ly, "d": d, "vol": vol, "lo": 0, "lam": 0, "mode": "native", "sweep": "native",
         "shape": 0}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small FP64 Gram (R^3 and a time channel, 64 steps): the smallest
        # call in use, bound by launches and by the wavefront's depth
        _case("gram_small_f64", "gram", "approx", 4, "f64", 8, 65, 8, 65, 4, vol=1.0),
        # a small training step, as in a notebook or inside a larger model
        _case("train_small_f32", "train", "interp", 4, "f32", 24, 50, 17, 41, 3, vol=1.0),
        # inference: Gram matrix between a training and a test set
        _case("gram_f32", "gram", "interp", 6, "f32", 128, 257, 128, 257, 8),
        # the headline workload: 128 x 128 Gram, R^8, 256 steps, forward + backward
        _case("train_f32", "train", "interp", 6, "f32", 128, 257, 128, 257, 8),
        # FP64 training step on odd sizes, fewer pairs than the GPU has waves
        _case("train_odd_f64", "train", "approx", 6, "f64", 37, 151, 29, 203, 5, vol=1.0),
        # a fixed batch of uneven pairs trained through a plan
        _case("plan_uneven_f32", "plan", "approx", 8, "f32", 512, 2048, 512, 2048, 16, lo=32),
        # one-shot kernel values of a ragged pair list (similarity queries)
        _case("pairs_ragged_f64", "pairs", "approx", 5, "f64", 300, 400, 300, 300, 3, vol=1.0, lo=17),
        # rows of a large Gram in R^32 (BF16-split increments), forward + backward
        _case("train_wide_f32", "train", "approx", 8, "f32", 16, 1025, 160, 1025, 32, mode="bf16x3"),
        # rows of a Gram of unit-variance cell constants (values beyond the FP32
        # range), FP32 points swept in FP64, forward + backward through log K
        _case("log_wide_f64sweep", "log", "approx", 8, "f32", 8, 513, 128, 513, 32,
              vol=math.sqrt(512.0 / math.sqrt(32.0)), sweep="f64"),
        # two-sample statistic with gradients (two clearly different samples)
        _case("mmd_f32", "mmd", "approx", 8, "f32", 64, 513, 64, 513, 5, vol=1.0),
        # few very long paths
        _case("train_long_f32", "train", "approx", 8, "f32", 4, 8193, 4, 8193, 8),
        # the finite-difference baseline on its refined grid
        _case("gram_fd_f32", "gram", "fd", 1, "f32", 64, 129, 64, 129, 6),
    ]


def _lens(case):
    """Points per path of a ragged list: fixed by the case."""
    r = random.Random(1000 + case["shape"])
    lx = [r.randint(case["lo"], case["lx"]) for _ in range(case["nx"])]
    ly = [r.randint(case["lo"], case["ly"]) for _ in range(case["nx"])]
    return lx, ly


def _cells(case):
    if case["op"] in ("pairs", "plan"):
        n = sum((a - 1) * (b - 1) for a, b in zip(*_lens(case)))
    elif case["op"] == "mmd":
        n = (case["nx"] * (case["nx"] - 1) // 2 + case["ny"] * (case["ny"] - 1) // 2
             + case["nx"] * case["ny"]) * (case["lx"] - 1) * (case["ly"] - 1)
    else:
        n = case["nx"] * case["ny"] * (case["lx"] - 1) * (case["ly"] - 1)
    lam = case["order"] if case["scheme"] in ("fd", "fd2") else case["lam"]
    return n, n << (2 * lam)


def work(case):
    """Inputs read once and outputs written once; the products of the cell map
    (Toeplitz and Hankel parts of both edges), twice that again for its
    transpose and the derivatives, and the increment Gram."""
    es = 4 if case["dtype"] == "f32" else 8
    n, refined = _cells(case)
    bwd = case["op"] in ("train", "log", "plan", "mmd")
    if case["op"] in ("pairs", "plan"):
        lx, ly = _lens(case)
        pts, vals = sum(lx) + sum(ly), case["nx"]
    else:
        pts = case["nx"] * case["lx"] + case["ny"] * case["ly"]
        vals = 1 if case["op"] == "mmd" else case["nx"] * case["ny"]
    if case["scheme"] in ("fd", "fd2"):
        cell = 5
    else:
        N = case["order"]
        cell = 2 * (N + 1) * (3 * N + 4)
    return {"bytes": float(pts * case["d"] * es * (2 if bwd else 1) + vals * es * (2 if bwd else 1)),
            "flops": float(refined * cell * (3 if bwd else 1) + n * 2 * case["d"] * (3 if bwd else 1))}


def draw(rng):
    """One more case: the same kinds over the ranges the listed ones stand for."""
    while True:
        op = rng.choice(["gram", "gram", "train", "train", "train", "pairs", "plan", "mmd", "log"])

        def size(lo, hi):
            return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

        dtype = "f32" if rng.random() < 0.65 else "f64"
        scheme = rng.choice(["approx", "approx", "interp"])
        order = rng.randint(2, 8)
        if op == "gram" and rng.random() < 0.2:
            scheme, order = rng.choice(["fd", "fd2"]), rng.randint(0, 2)
        d = size(2, 40)
        kw = {"vol": rng.choice([0.5, 1.0]) * math.sqrt(4.0 / max(d, 4)), "shape": rng.randrange(1 << 30)}
        nx, ny = size(2, 160), size(2, 160)
        lx, ly = size(9, 2049), size(9, 2049)
        if op in ("pairs", "plan"):
            nx = ny = size(8, 600)
            kw["lo"] = rng.randint(2, max(2, min(lx, ly) // 2))
        elif op == "mmd":
            nx, ny = max(nx, 4), max(ny, 4)
            if rng.random() < 0.7:
                ly = lx
        elif op == "log":
            dtype, scheme, order, kw["sweep"] = "f32", "approx", max(order, 4), "f64"
            lx, ly = min(lx, 513), min(ly, 513)
            kw["vol"] = math.sqrt(math.sqrt(lx * ly) / math.sqrt(d))
        elif scheme in ("approx", "interp"):
            if dtype == "f32" and d > 8 and rng.random() < 0.4:
                kw["mode"] = "bf16x3"
            if rng.random() < 0.1:
                kw["lam"] = 1
        c = _case(None, op, scheme, order, dtype, nx, lx, ny, ly, d, **kw)
        bwd = op in ("train", "log", "plan", "mmd")
        cost = _cells(c)[1] * (order + 3) ** 2 * (3 if bwd else 1) * (2 if dtype == "f64" or "sweep" in kw else 1)
        if 1e6 < cost < 3e11:
            return c


def _paths(g, n, pts, d, vol, dtype, drift=0.0):
    dx = torch.randn(n, pts, d, generator=g, device="cuda", dtype=torch.float64)
    dx = dx * (vol / math.sqrt(max(pts - 1, 1))) + drift / max(pts - 1, 1)
    dx[:, 0] = 0.0
    return dx.cumsum(1).to(dtype).contiguous()


def _ragged(case, g):
    """(points, offsets) of both sides of a ragged pair list, and seeds dL/dk."""
    dt = _DT[case["dtype"]]

    def side(lens):
        off = [0]
        for n in lens:
            off.append(off[-1] + n)
        n = torch.tensor(lens, device="cuda")
        scale = (case["vol"] / torch.sqrt(torch.clamp(n - 1, min=1).double())).repeat_interleave(n)
        dx = torch.randn(off[-1], case["d"], generator=g, device="cuda", dtype=torch.float64) * scale[:, None]
        x = dx.cumsum(0)
        first = torch.tensor(off[:-1], device="cuda")
        return (x - x[first].repeat_interleave(n, 0)).to(dt).contiguous(), off

    lx, ly = _lens(case)
    return side(lx), side(ly), torch.randn(case["nx"], generator=g, device="cuda", dtype=dt)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dt = _DT[case["dtype"]]
    st = {"case": case}
    if case["op"] in ("pairs", "plan"):
        st["x"], st["y"], st["gk"] = _ragged(case, g)
        if case["op"] == "plan":
            st["plan"] = sk.PairsPlan(st["x"], st["y"], case["scheme"], case["order"], backward=True,
                                      dyadic=case["lam"])
            st["k"] = torch.empty_like(st["gk"])
            st["gx"], st["gy"] = torch.empty_like(st["x"][0]), torch.empty_like(st["y"][0])
        return st
    st["X"] = _paths(g, case["nx"], case["lx"], case["d"], case["vol"], dt)
    st["Y"] = _paths(g, case["ny"], case["ly"], case["d"], case["vol"], dt,
                     drift=2.0 if case["op"] == "mmd" else 0.0)
    if case["op"] in ("train", "mmd"):
        st["X"].requires_grad_(True)
        st["Y"].requires_grad_(True)
    if case["op"] == "train":
        st["W"] = torch.randn(case["nx"], case["ny"], generator=g, device="cuda", dtype=dt)
    return st


def run(state):
    c = state["case"]
    op, scheme, order = c["op"], c["scheme"], c["order"]
    if op == "gram":
        return sk.gram(state["X"], state["Y"], scheme, order, gram_mode=c["mode"], dyadic=c["lam"])
    if op == "train":
        X, Y = state["X"], state["Y"]
        K = sk.sig_gram(X, Y, scheme, order, gram_mode=c["mode"], dyadic=c["lam"])
        gX, gY = torch.autograd.grad(K, [X, Y], state["W"])
        return K.detach(), gX, gY
    if op == "log":
        X, Y = state["X"], state["Y"]
        K, E = sk.gram(X, Y, scheme, order, return_exp=True, sweep="f64")
        gX, gY = sk.gram_backward(X, Y, 1.0 / K, scheme, order, gK_exp=-E, sweep="f64")
        return torch.log2(K.abs()) + E, gX, gY
    if op == "pairs":
        return sk.pairs(state["x"], state["y"], scheme, order)
    if op == "plan":
        p, x, y = state["plan"], state["x"][0], state["y"][0]
        try:
            p.forward_save(x, y, state["k"])
            p.backward_saved(x, y, state["gk"], state["gx"], state["gy"])
        except sk.SigKernelError as e:  # a backward of several chunks keeps no state
            if e.status != _lib.SK_EWORKSPACE:
                raise
            p.forward(x, y, state["k"])
            p.backward(x, y, state["gk"], state["gx"], state["gy"])
        return state["k"], state["gx"], state["gy"]
    X, Y = state["X"], state["Y"]
    m = sk.mmd2(X, Y, scheme, order)
    gX, gY = torch.autograd.grad(m, [X, Y])
    return m.detach(), gX, gY


# ---------------------------------------------------------------------------
# the same values in 64 bits, by plain torch: the schemes on all cells of an
# anti-diagonal at once, and the transpose of the same recursion
# ---------------------------------------------------------------------------
_TAIL = 24


def _interp_tail(N):
    """Rows n = 0..N of the interpolation of u^r, r = N+1 .. N+_TAIL, at the
    N + 1 Chebyshev extrema of [0, 1], in the basis n! x (coefficient n) for
    r! x (coefficient r)."""
    u = (1 - np.cos(np.pi * np.arange(N + 1, dtype=np.longdouble) / N)) / 2
    out = np.zeros((_TAIL, N + 1), dtype=np.longdouble)
    for m in range(N + 1):
        p = np.array([1], dtype=np.longdouble)
        for q in range(N + 1):
            if q != m:
                p = np.convolve(p, np.array([-u[q], 1], dtype=np.longdouble)) / (u[m] - u[q])
        for t in range(_TAIL):
            out[t] += u[m] ** (N + 1 + t) * p
    for t in range(_TAIL):
        for n in range(N + 1):
            out[t, n] *= np.longdouble(math.factorial(n)) / math.factorial(N + 1 + t)
    return out.astype(np.float64)


class _Exact:
    """Kernels of P pairs (P, lx, ly) of cell constants (already refined), and
    dL/dc for seeds g.  ends: last cell (row, column) of each pair."""

    def __init__(self, scheme, order):
        self.scheme, self.N = scheme, order
        if scheme in ("approx", "interp"):
            N, R = order, order + (_TAIL if scheme == "interp" else 0)
            self.R = R
            H = torch.zeros(R + 1, N + 1, dtype=torch.float64)
            for r in range(R + 1):
                for k in range(1, N + 1):
                    H[r, k] = 1.0 / math.factorial(r + k)
            self.H = H.cuda()
            self.f = torch.tensor([1.0 / math.factorial(m) for m in range(R + 1)], dtype=torch.float64).cuda()
            self.rs = torch.from_numpy(_interp_tail(N)).cuda() if scheme == "interp" else None

    def _rows(self, S, c, deriv=False):
        N, R = self.N, self.R
        cp = c[..., None] ** torch.arange(R + 1, device=c.device, dtype=torch.float64)
        w = cp * self.f
        T = torch.zeros(*S.shape[:-1], R + 1, device=c.device, dtype=torch.float64)
        for k in range(N + 1):
            T[..., k:] += S[..., k:k + 1] * w[..., :R + 1 - k]
        Hk = (S @ self.H.T).flip(0)
        if not deriv:
            return T + cp * Hk, w, cp
        D = torch.zeros_like(T)
        r = torch.arange(1, R + 1, device=c.device, dtype=torch.float64)
        D[..., 1:] = T[..., :-1] + r * cp[..., :-1] * Hk[..., 1:]
        return D, w, cp

    def _sweep(self, C, ends, keep):
        P, lx, ly = C.shape
        N = self.N
        Cr = C.flip(2)
        A = torch.zeros(P, ly, N + 1, device=C.device, dtype=torch.float64)  # bottom edges, columns reversed
        B = torch.zeros(P, lx, N + 1, device=C.device, dtype=torch.float64)  # left edges
        A[..., 0] = 1.0
        B[..., 0] = 1.0
        k = torch.zeros(P, device=C.device, dtype=torch.float64)
        done = {}
        for p, (i, j) in enumerate(ends):
            done.setdefault(i + j, []).append((p, i, j))
        kept = []
        for g in range(lx + ly - 1):
            i0, i1 = max(0, g - ly + 1), min(lx - 1, g) + 1
            q0 = ly - 1 - g + i0
            sa, sb = A[:, q0:q0 + i1 - i0], B[:, i0:i1]
            S = torch.stack([sa, sb])
            c = torch.diagonal(Cr, offset=ly - 1 - g, dim1=1, dim2=2)
            rows, _, _ = self._rows(S, c)
            out = rows[..., :N + 1]
            if self.rs is not None:
                out = out + rows[..., N + 1:] @ self.rs
            A[:, q0:q0 + i1 - i0] = out[0]
            B[:, i0:i1] = out[1]
            if keep:
                kept.append(S)
            if g in done:
                p = torch.tensor([e[0] for e in done[g]], device=C.device)
                i = torch.tensor([e[1] for e in done[g]], device=C.device)
                k[p] = 0.5 * ((out[0][p, i - i0] + out[1][p, i - i0]) * self.f[:N + 1]).sum(-1)
        return k, kept, done

    def forward(self, C, ends):
        if self.scheme in ("fd", "fd2"):
            return self._fd(C)
        return self._sweep(C, ends, False)[0]

    def backward(self, C, ends, seed):
        P, lx, ly = C.shape
        N, R = self.N, self.R
        k, kept, done = self._sweep(C, ends, True)
        Cr = C.flip(2)
        G = torch.zeros(P, lx, ly, device=C.device, dtype=torch.float64)  # columns reversed
        A = torch.zeros(P, ly, N + 1, device=C.device, dtype=torch.float64)
        B = torch.zeros(P, lx, N + 1, device=C.device, dtype=torch.float64)
        for g in range(lx + ly - 2, -1, -1):
            i0, i1 = max(0, g - ly + 1), min(lx - 1, g) + 1
            q0 = ly - 1 - g + i0
            S = kept.pop()
            c = torch.diagonal(Cr, offset=ly - 1 - g, dim1=1, dim2=2)
            a = torch.stack([A[:, q0:q0 + i1 - i0], B[:, i0:i1]])
            if g in done:
                p = torch.tensor([e[0] for e in done[g]], device=C.device)
                i = torch.tensor([e[1] for e in done[g]], device=C.device)
                a[:, p, i - i0] = 0.5 * seed[p][:, None] * self.f[:N + 1]
            if self.rs is not None:
                a = torch.cat([a, a @ self.rs.T], -1)
            D, w, cp = self._rows(S, c, deriv=True)
            torch.diagonal(G, offset=ly - 1 - g, dim1=1, dim2=2).copy_((a * D).sum((0, 3)))
            out = (a * cp).flip(0) @ self.H
            for m in range(N + 1):
                out[..., m] += (a[..., m:] * w[..., :R + 1 - m]).sum(-1)
            A[:, q0:q0 + i1 - i0] = out[0]
            B[:, i0:i1] = out[1]
        return k, G.flip(2)

    def _fd(self, C):
        P, lx, ly = C.shape
        Cr = C.flip(2)
        d1 = torch.ones(P, lx + 1, device=C.device, dtype=torch.float64)  # node diagonal g + 1, by row
        d0 = d1.clone()
        for g in range(lx + ly - 1):
            i0, i1 = max(0, g - ly + 1), min(lx - 1, g) + 1
            c = torch.diagonal(Cr, offset=ly - 1 - g, dim1=1, dim2=2)
            a, b, z = d1[:, i0 + 1:i1 + 1], d1[:, i0:i1], d0[:, i0:i1]
            v = a + b - z + 0.5 * c * (a + b)
            if self.scheme == "fd2":
                v = v + c * c / 12.0 * (a + b + z)
            d2 = torch.ones_like(d1)
            d2[:, i0 + 1:i1 + 1] = v
            d0, d1 = d1, d2
        return d1[:, lx]


def _solve(case, dX, dY, ends, seed):
    """Kernels and dL/dc of a batch of pairs' increments (chunked by memory)."""
    poly = case["scheme"] in ("approx", "interp")
    lam = case["lam"] if poly else case["order"]
    ex = _Exact(case["scheme"], case["order"])
    P, lx, ly = dX.shape[0], dX.shape[1] << lam, dY.shape[1] << lam
    m = min(lx, ly)
    if seed is None:
        per = (lx * ly * 3 + m * 400) * 8
    else:
        per = (lx * ly * 4 + m * 400 + (lx + ly) * m * 2 * (case["order"] + 1)) * 8
    step = int(max(1, min(P, 6e10 // per)))
    ks, gx, gy = [], [], []
    for p in range(0, P, step):
        x, y = dX[p:p + step], dY[p:p + step]
        C = torch.bmm(x, y.transpose(1, 2).contiguous()) / 4.0 ** lam
        C = C.repeat_interleave(1 << lam, 1).repeat_interleave(1 << lam, 2)
        e = [(((a + 1) << lam) - 1, ((b + 1) << lam) - 1) for a, b in ends[p:p + step]]
        if seed is None:
            ks.append(ex.forward(C, e))
            continue
        k, G = ex.backward(C, e, seed(p, p + step))
        n = x.shape[0]
        G = G.reshape(n, x.shape[1], 1 << lam, y.shape[1], 1 << lam).sum((2, 4)) / 4.0 ** lam
        ks.append(k)
        gx.append(torch.bmm(G, y))
        gy.append(torch.bmm(G.transpose(1, 2).contiguous(), x))
    k = torch.cat(ks)
    return k if seed is None else (k, torch.cat(gx), torch.cat(gy))


def _points(g):
    """dL/dX from dL/d(dx): (..., L, d) -> (..., L + 1, d)."""
    z = torch.zeros_like(g[..., :1, :])
    return torch.cat([z, g], -2) - torch.cat([g, z], -2)


def _seconds(case, pairs, lx, ly, bwd):
    """About how long the 64-bit computation takes."""
    poly = case["scheme"] in ("approx", "interp")
    lam = case["lam"] if poly else case["order"]
    lx, ly, N = lx << lam, ly << lam, case["order"]
    R = N + (_TAIL if case["scheme"] == "interp" else 0) if poly else 1
    m = min(lx, ly)
    state = (lx + ly) * m * 2 * (N + 1) * 8 if bwd else 0
    chunks = max(1.0, pairs * (state + lx * ly * 32 + m * 3200) / 6e10)
    bytes_ = pairs * float(lx) * ly * 2 * (R + 1) * 8 * (2 * N + 12) * (3 if bwd else 1)
    return (lx + ly) * chunks * (N + 25) * 12e-6 * (3 if bwd else 1) + bytes_ / 2.5e12


def exact(case, seed):
    st = prepare(dict(case, op="pairs") if case["op"] == "plan" else case, seed)  # (no plan needed)
    op = case["op"]
    most = 19.0
    with torch.no_grad():
        if op in ("pairs", "plan"):
            lx, ly = _lens(case)
            n, gk = case["nx"], st["gk"].double()
            # pairs sorted by size, in groups of similar sizes, padded within a group
            order = sorted(range(n), key=lambda p: max(lx[p], ly[p]))
            size = max(1, -(-n // 8))
            groups = [order[i:i + size] for i in range(0, n, size)]

            def dims(q):
                return max(max(lx[p] for p in q) - 1, 1), max(max(ly[p] for p in q) - 1, 1)

            bwd = op == "plan"
            if bwd and sum(_seconds(case, len(q), *dims(q), True) for q in groups) > most:
                bwd = False
            if sum(_seconds(case, len(q), *dims(q), bwd) for q in groups) > most:
                return None
            k = torch.ones(n, device="cuda", dtype=torch.float64)
            gx, gy = (torch.zeros(t[0].shape, device="cuda", dtype=torch.float64) for t in (st["x"], st["y"]))
            xs, ys = st["x"][0].double(), st["y"][0].double()
            xo, yo = st["x"][1], st["y"][1]
            for q in groups:
                q = [p for p in q if lx[p] > 1 and ly[p] > 1]
                if not q:
                    continue
                mx, my = dims(q)
                dX = torch.zeros(len(q), mx, case["d"], device="cuda", dtype=torch.float64)
                dY = torch.zeros(len(q), my, case["d"], device="cuda", dtype=torch.float64)
                for i, p in enumerate(q):
                    dX[i, :lx[p] - 1] = xs[xo[p]:xo[p + 1]].diff(dim=0)
                    dY[i, :ly[p] - 1] = ys[yo[p]:yo[p + 1]].diff(dim=0)
                ends = [(lx[p] - 2, ly[p] - 2) for p in q]
                idx = torch.tensor(q, device="cuda")
                if not bwd:
                    k[idx] = _solve(case, dX, dY, ends, None)
                    continue
                s = gk[idx]
                k[idx], a, b = _solve(case, dX, dY, ends, lambda u, v: s[u:v])
                for i, p in enumerate(q):
                    gx[xo[p]:xo[p + 1]] = _points(a[i, :lx[p] - 1])
                    gy[yo[p]:yo[p + 1]] = _points(b[i, :ly[p] - 1])
            if op == "pairs":
                return k
            return (k, gx, gy) if bwd else (k, None, None)
        X, Y = st["X"].detach().double(), st["Y"].detach().double()
        nx, ny = X.shape[0], Y.shape[0]
        dX, dY = X.diff(dim=1), Y.diff(dim=1)
        ends1 = (dX.shape[1] - 1, dY.shape[1] - 1)
        if op == "mmd":
            Z = [X, Y]
            tri = [torch.triu_indices(n, n, 1, device="cuda") for n in (nx, ny)]
            w = (2.0 / (nx * (nx - 1)), 2.0 / (ny * (ny - 1)), -2.0 / (nx * ny))
            lists = [(0, 0, tri[0][0], tri[0][1], w[0]), (1, 1, tri[1][0], tri[1][1], w[1]),
                     (0, 1, torch.arange(nx, device="cuda").repeat_interleave(ny),
                      torch.arange(ny, device="cuda").repeat(nx), w[2])]
            if sum(_seconds(case, len(i), Z[a].shape[1], Z[b].shape[1], True) for a, b, i, _, _ in lists) > most:
                return None
            val, grads = 0.0, [torch.zeros_like(X), torch.zeros_like(Y)]
            for a, b, i, j, wt in lists:
                dA, dB = Z[a].diff(dim=1)[i], Z[b].diff(dim=1)[j]
                ends = [(dA.shape[1] - 1, dB.shape[1] - 1)] * len(i)
                k, u, v = _solve(case, dA, dB, ends,
                                 lambda p, q: torch.full((min(q, len(i)) - p,), wt, device="cuda", dtype=torch.float64))
                val = val + wt * k.sum()
                grads[a].index_add_(0, i, _points(u))
                grads[b].index_add_(0, j, _points(v))
            return val, grads[0], grads[1]
        bwd = op in ("train", "log") and _seconds(case, nx * ny, dX.shape[1], dY.shape[1], True) <= most
        if not bwd and _seconds(case, nx * ny, dX.shape[1], dY.shape[1], False) > most:
            return None
        K = torch.empty(nx, ny, device="cuda", dtype=torch.float64)
        gX, gY = torch.zeros_like(X), torch.zeros_like(Y)
        rows = max(1, 4096 // ny)  # a block of rows of the Gram at a time
        for a in range(0, nx, rows):
            n = min(rows, nx - a)
            bx, by = dX[a:a + n].repeat_interleave(ny, 0), dY.repeat(n, 1, 1)
            ends = [ends1] * (n * ny)
            if not bwd:
                K[a:a + n] = _solve(case, bx, by, ends, None).reshape(n, ny)
                continue
            if op == "log":  # d log2|K| / d K = 1 / (K ln 2); the case seeds 1 / K
                seeds = 1.0 / _solve(case, bx, by, ends, None)
            else:
                seeds = st["W"][a:a + n].double().reshape(-1)
            k, u, v = _solve(case, bx, by, ends, lambda p, q: seeds[p:q])
            K[a:a + n] = k.reshape(n, ny)
            gX[a:a + n] = _points(u.reshape(n, ny, *u.shape[1:]).sum(1))
            gY += _points(v.reshape(n, ny, *v.shape[1:]).sum(0))
        if op == "gram":
            return K
        if op == "log":
            K = torch.log2(K.abs())
        return (K, gX, gY) if bwd else (K, None, None)
