"""The calls this library is measured on, made through its public Python entry points.

A case is a dict of plain values:

  op      "tsm2r", "tsm2l"   C = A*B (`tsm2r`, `tsm2l`), F64 or F32
          "lowp"             C = A*B on A's 16-bit planes (`tsm2r` on a SplitA)
          "autograd"         forward and both gradients (`matmul`, `autograd.grad`)
          "kmeans"           labels and distances (`kmeans.assign`)
          "tsmttsm"          C = A^T*B of two tall matrices (`tsmttsm`)
  m, k, n sizes: A is m x k, B is k x n (tsmttsm: A m x k and B m x n;
          kmeans: m points of k coordinates, n centroids)
  dtype   "f64" or "f32"; autograd: the mode ("f64", "f32", "bf16", "bf16_split",
          "f16", "f16_split"); lowp: the storage form (the last four)
  a, b    "col" or "row": how A (or the points) and B are held
  planes  autograd in a 16-bit mode: A is kept as its planes across calls
          (a SplitA) instead of being split in every forward

Values are those of the library's workloads: A and B uniform in [-1, 1), the
upstream gradient N(0, 1), K-means points scattered about their centroids.
"""
import math

import torch

import paper_2002_03258_amd as tsm
from paper_2002_03258_amd import kmeans

_DT = {"f64": torch.float64, "f32": torch.float32}
_LOWP = {"bf16": ("bf16", False), "bf16_split": ("bf16", True), "f16": ("f16", False),
         "f16_split": ("f16", True)}


def _case(op, m, k, n, dtype, a="col", b="row", planes=False):
    c = {"op": op, "m": m, "k": k, "n": n, "dtype": dtype}
    if op in ("tsm2r", "tsm2l"):
        c.update(a=a, b=b)
    elif op in ("kmeans", "tsmttsm"):
        c.update(a=a)
    elif op == "autograd":
        c.update(planes=planes)
    return c


def listed():
    return [
        # one small product of tensors as torch makes them (row-major): latency
        dict(_case("tsm2r", 1024, 1024, 4, "f64", a="row"), name="r_small_row_f64"),
        # the large FP64 product of the TSM2R grid, column-major
        dict(_case("tsm2r", 30720, 30720, 16, "f64", b="col"), name="r_square_f64"),
        # a matrix of odd sizes, whose columns start at odd addresses
        dict(_case("tsm2r", 10007, 9973, 5, "f32"), name="r_ragged_f32"),
        # more right-hand sides than one kernel pass takes
        dict(_case("tsm2r", 20480, 20480, 64, "f64", b="col"), name="r_wide_f64"),
        # the widest of the tall-and-skinny grid, at its largest m
        dict(_case("tsm2l", 1 << 24, 32, 32, "f64", b="col"), name="l_tall_f64"),
        # a tall matrix with an odd number of rows, few columns
        dict(_case("tsm2l", 1000003, 8, 8, "f32"), name="l_ragged_f32"),
        # a tall matrix as torch holds it: one point a row
        dict(_case("tsm2l", 1 << 22, 16, 16, "f32", a="row"), name="l_row_f32"),
        # the precision form: A read at two bytes an element
        dict(_case("lowp", 32768, 32768, 16, "bf16"), name="lowp_bf16"),
        # training step on a tall float matrix, kept to bf16 hi + lo planes
        dict(_case("autograd", 8388608, 16, 16, "bf16_split"), name="step_l_bf16_split"),
        # training step on a large float matrix
        dict(_case("autograd", 16384, 16384, 8, "f32"), name="step_r_f32"),
        # K-means assignment of row-major points
        dict(_case("kmeans", 1 << 24, 16, 16, "f32", a="row"), name="kmeans_f32"),
        # Gram matrix of row-major points
        dict(_case("tsmttsm", 1 << 20, 16, 16, "f32", a="row"), name="gram_f32"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _size(rng, lo, hi):
    """Over the logarithm of the range; half of them whole multiples of 64."""
    v = _log(rng, lo, hi)
    return max(lo, v // 64 * 64) if rng.random() < 0.5 and v >= 128 else v


def draw(rng):
    """One more case: sizes over the ranges of the listed ones."""
    top = max(_cost(c) for c in listed())
    while True:
        op = rng.choice(("tsm2r", "tsm2r", "tsm2r", "tsm2l", "tsm2l", "lowp", "autograd", "autograd",
                         "kmeans", "tsmttsm"))
        plain = rng.choice(("f64", "f32"))
        side = rng.choice(("col", "row"))
        if op == "tsm2r":
            c = _case(op, _size(rng, 256, 30720), _size(rng, 256, 30720), _log(rng, 1, 64), plain,
                      side, rng.choice(("col", "row")))
        elif op == "tsm2l":
            c = _case(op, _size(rng, 1 << 14, 1 << 24), rng.randint(1, 32), rng.randint(1, 32), plain,
                      side, rng.choice(("col", "row")))
        elif op == "lowp":
            c = _case(op, _size(rng, 1024, 32768), _size(rng, 1024, 32768), _log(rng, 1, 32),
                      rng.choice(sorted(_LOWP)))
        elif op == "autograd":
            mode = rng.choice(("f64", "f32", "f32", "bf16_split", "bf16_split", "bf16", "f16_split",
                               "f16"))
            planes = mode in _LOWP and rng.random() < 0.5
            if rng.random() < 0.5:
                c = _case(op, _size(rng, 1 << 14, 1 << 23), rng.randint(2, 32), rng.randint(2, 32), mode,
                          planes=planes)
            else:
                c = _case(op, _size(rng, 1024, 16384), _size(rng, 1024, 16384), _log(rng, 1, 32), mode,
                          planes=planes)
        elif op == "kmeans":
            c = _case(op, _size(rng, 1 << 14, 1 << 24), _log(rng, 2, 64), _log(rng, 2, 64), plain, side)
        else:
            c = _case(op, _size(rng, 1 << 14, 1 << 23), rng.randint(2, 32), rng.randint(2, 32), plain,
                      side)
        if _cost(c) <= top:
            return c


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def work(case):
    m, k, n = case["m"], case["k"], case["n"]
    op, dt = case["op"], case["dtype"]
    es = 8 if dt == "f64" else 4
    flops = 2.0 * m * k * n
    if op in ("tsm2r", "tsm2l"):
        return {"bytes": es * (m * k + k * n + m * n), "flops": flops}
    if op == "lowp":
        stored = 4 if _LOWP[dt][1] else 2
        return {"bytes": stored * m * k + 4 * (k * n + m * n), "flops": flops}
    if op == "autograd":
        # C, dA and dB out; A, B and dC in.  A float A in a 16-bit mode is read
        # once: its planes are the library's own.  A kept as planes is read as such.
        a_in = m * k * ((4 if _LOWP[dt][1] else 2) if case["planes"] else es)
        return {"bytes": a_in + es * (k * n + m * n + m * n + m * k + k * n), "flops": 3 * flops}
    if op == "kmeans":
        return {"bytes": es * (m * k + k * n + m) + 4 * m, "flops": flops}
    return {"bytes": es * (m * k + m * n + k * n), "flops": flops}      # tsmttsm


def _uniform(g, rows, cols, dtype, side):
    """rows x cols in [-1, 1), held by columns or by rows."""
    shape = (cols, rows) if side == "col" else (rows, cols)
    x = torch.empty(shape, dtype=dtype, device=g.device).uniform_(-1, 1, generator=g)
    return x.t() if side == "col" else x


def _inputs(case, seed):
    """The tensors of the call, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    m, k, n, op = case["m"], case["k"], case["n"], case["op"]
    dt = _DT.get(case["dtype"], torch.float32)
    if op in ("tsm2r", "tsm2l"):
        return _uniform(g, m, k, dt, case["a"]), _uniform(g, k, n, dt, case["b"])
    if op == "lowp":
        return _uniform(g, m, k, dt, "col"), _uniform(g, k, n, dt, "row")
    if op == "autograd":
        A, B = _uniform(g, m, k, dt, "col"), _uniform(g, k, n, dt, "row")
        dC = torch.empty((n, m), dtype=dt, device=g.device).normal_(generator=g).t()
        return A, B, dC
    if op == "kmeans":
        mu = _uniform(g, n, k, dt, "row")
        shape = (k, m) if case["a"] == "col" else (m, k)
        X = torch.empty(shape, dtype=dt, device=g.device).normal_(0, 0.3, generator=g)
        X = X.t() if case["a"] == "col" else X
        for j in range(k):          # one coordinate at a time: little scratch memory
            X[:, j] += mu[:, j].repeat(-(-m // n))[:m]
        return X, mu
    return _uniform(g, m, k, dt, case["a"]), _uniform(g, m, n, dt, case["a"])


def prepare(case, seed):
    ins = _inputs(case, seed)
    op, dt = case["op"], case["dtype"]
    if op == "lowp":
        A, B = ins
        return {"op": op, "A": tsm.split(A, *_LOWP[dt]), "B": B}
    if op == "autograd":
        A, B, dC = ins
        A, B = A.requires_grad_(), B.requires_grad_()
        S = tsm.split(A, *_LOWP[dt]) if case["planes"] else None
        return {"op": op, "A": A, "B": B, "dC": dC, "mode": dt, "planes": S}
    if op == "kmeans":
        return {"op": op, "X": ins[0], "mu": ins[1]}
    return {"op": op, "A": ins[0], "B": ins[1]}


def run(state):
    op = state["op"]
    if op in ("tsm2r", "lowp"):
        return tsm.tsm2r(state["A"], state["B"])
    if op == "tsm2l":
        return tsm.tsm2l(state["A"], state["B"])
    if op == "autograd":
        if state["planes"] is not None:
            C = tsm.matmul(state["planes"], state["B"])
        else:
            C = tsm.matmul(state["A"], state["B"], mode=state["mode"])
        dA, dB = torch.autograd.grad(C, (state["A"], state["B"]), state["dC"])
        return C.detach(), dA, dB
    if op == "kmeans":
        return kmeans.assign(state["X"], state["mu"])
    return tsm.tsmttsm(state["A"], state["B"])


def _stored(A, dt):
    """The float64 values A's 16-bit planes hold: hi, or hi + lo."""
    fmt, lo = _LOWP[dt]
    t = torch.bfloat16 if fmt == "bf16" else torch.float16
    hi = A.to(t)
    v = hi.double()
    return v + (A - hi.float()).to(t).double() if lo else v


def exact(case, seed):
    ins = [x.detach() for x in _inputs(case, seed)]
    op, dt = case["op"], case["dtype"]
    if op in ("tsm2r", "tsm2l"):
        return torch.matmul(ins[0].double(), ins[1].double())
    if op == "lowp":
        return torch.matmul(_stored(ins[0], dt), ins[1].double())
    if op == "autograd":
        A = _stored(ins[0], dt) if dt in _LOWP else ins[0].double()
        B, dC = ins[1].double(), ins[2].double()
        return torch.matmul(A, B), torch.matmul(dC, B.t()), torch.matmul(A.t(), dC)
    if op == "kmeans":
        X, mu = ins
        d = torch.empty(X.shape[0], dtype=torch.float64, device=X.device)
        step = 1 << 18
        for i in range(0, X.shape[0], step):
            x, best = X[i:i + step].double(), None
            for c in mu.double():
                s = (x - c).square_().sum(1)
                best = s if best is None else torch.minimum(best, s)
            d[i:i + step] = best
        return None, d              # labels are whole numbers
    return torch.matmul(ins[0].double().t(), ins[1].double())
