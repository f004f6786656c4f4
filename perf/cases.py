"""Performance cases of the multi-component (MC) floating-point library.

The listed cases are the calls a program built on the library makes, over the sizes it makes
them at: MC-SGD weight updates of a small layer and of a large odd-sized one, elementwise
products, the matrix products from a 64-wide one to the 8192-wide benchmark product, batched
and matrix-vector products, MC-Linear training steps of a small binary32 layer and of a large
binary16 one, the exact binary16 layer, and the linear-regression gradient step.  ``draw``
gives further cases of the same ranges: other sizes (odd ones among them), component formats,
component counts and operand kinds.

Every result of the library is a fixed function of its inputs -- each operation is a stated
sequence of correctly rounded steps in a stated order -- so any correct implementation
returns the same values and the tolerance of every case is "exact".
"""
from __future__ import annotations

import math

import torch

import paper_2207_08867_amd as mcf

DTYPES = {"f16": torch.float16, "f32": torch.float32, "f64": torch.float64}
SIZE = {"f16": 2, "f32": 4, "f64": 8}


def listed():
    return [
        # MC-SGD update of a small layer's weight and bias (784 x 10 + 10): a latency-bound call.
        dict(name="update_small", kind="update", dtype="f32", nc=2, n=7850),
        # The same update over a large odd-sized binary16 parameter buffer.
        dict(name="update_large_odd", kind="update", dtype="f16", nc=3, n=12345677),
        # Elementwise product of two MC tensors (Mult-MCN): a gating or mask-like layer's activations.
        dict(name="mult", kind="elementwise", op="mul", dtype="f16", nc=3, n=1 << 22),
        # The smallest matrix product: a 64-wide hidden layer.
        dict(name="mm_64", kind="matmul", dtype="f32", nc=2, M=64, N=64, K=64, a_mc=True, b_mc=True),
        # The paper's batched product, MC x plain.
        dict(name="bmm", kind="batched", dtype="f32", nc=3, B=16, M=500, N=50, K=200, a_mc=True, b_mc=False),
        # Binary16 MC x MC product.
        dict(name="mm_f16_1024", kind="matmul", dtype="f16", nc=2, M=1024, N=1024, K=1024, a_mc=True, b_mc=True),
        # The largest product: the benchmark's headline workload.
        dict(name="mm_f32_8192", kind="matmul", dtype="f32", nc=3, M=8192, N=8192, K=8192, a_mc=True, b_mc=True),
        # One training step (forward, all gradients) of a small binary32 MC-Linear layer on an odd batch.
        dict(name="linear_train_small", kind="linear", dtype="f32", nc=2, batch=100, inp=784, out=99),
        # One training step of the benchmark's binary16 MC-Linear layer.
        dict(name="linear_train_f16", kind="linear", dtype="f16", nc=3, batch=4096, inp=1024, out=1024),
        # Inference with the exact binary16 layer, a ragged request batch.
        dict(name="linear_exact", kind="linear_exact", dtype="f16", nc=3, batch=1000, inp=1024, out=1024),
        # One gradient-descent step of the paper's linear regression.
        dict(name="linreg", kind="linreg", dtype="f32", nc=2, n=10000, d=2),
        # Matrix-vector product, MC matrix by plain vector, with the K-split reduction.
        dict(name="mv", kind="splitk", dtype="f32", nc=3, M=8192, N=1, K=8192, a_mc=True, b_mc=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["update", "elementwise", "matmul", "batched", "linear", "linear_exact", "linreg", "splitk"])
    dtype = rng.choice(["f16", "f32", "f32", "f64"])
    nc = rng.choice([1, 2, 2, 3, 3, 4])
    a_mc, b_mc = rng.choice([(True, True), (True, False), (False, True)])
    if kind == "update":
        return dict(kind=kind, dtype=dtype, nc=nc, n=_log(rng, 100, 12000000))
    if kind == "elementwise":
        return dict(kind=kind, op=rng.choice(["mul", "div"]), dtype=dtype, nc=nc, n=_log(rng, 1000, 1 << 22))
    if kind == "matmul":
        return dict(kind=kind, dtype=dtype, nc=nc, M=_log(rng, 16, 1200), N=_log(rng, 16, 1200), K=_log(rng, 16, 1200),
                    a_mc=a_mc, b_mc=b_mc)
    if kind == "batched":
        return dict(kind=kind, dtype=dtype, nc=nc, B=_log(rng, 2, 32), M=_log(rng, 16, 500), N=_log(rng, 16, 500),
                    K=_log(rng, 16, 300), a_mc=a_mc, b_mc=b_mc)
    if kind == "linear":
        return dict(kind=kind, dtype=dtype, nc=nc, batch=_log(rng, 16, 1200), inp=_log(rng, 16, 1200),
                    out=_log(rng, 8, 1200))
    if kind == "linear_exact":
        return dict(kind=kind, dtype="f16", nc=nc, batch=_log(rng, 16, 4096), inp=_log(rng, 64, 2048),
                    out=_log(rng, 64, 2048))
    if kind == "linreg":
        return dict(kind=kind, dtype=dtype, nc=nc, n=_log(rng, 500, 20000), d=rng.randint(1, 8))
    return dict(kind=kind, dtype=dtype, nc=nc, M=_log(rng, 16, 4096), N=1, K=_log(rng, 1024, 8192), a_mc=a_mc,
                b_mc=b_mc)


class _Draws:
    """Float64 draws on the GPU from one seed, and their rounding into components."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dtype, self.nc = DTYPES[case["dtype"]], case["nc"]

    def normal(self, *shape, scale=1.0):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float64) * scale

    def uniform(self, lo, hi, *shape):
        return torch.rand(*shape, generator=self.g, device="cuda", dtype=torch.float64) * (hi - lo) + lo

    def plain(self, v):
        return v.to(self.dtype)

    def mc(self, v):
        """(nc, *shape): v split by successive rounding.  binary64 components below the
        first are drawn, each within a quarter ulp of the one before (a float64 draw
        has nothing left to split)."""
        planes = [v.to(self.dtype)]
        rest = v - planes[0].double()
        for _ in range(1, self.nc):
            if self.dtype == torch.float64:
                ulp = torch.ldexp(torch.ones_like(v), torch.frexp(planes[-1]).exponent - 53)
                planes.append(ulp * self.uniform(-0.25, 0.25, *v.shape))
            else:
                planes.append(rest.to(self.dtype))
                rest = rest - planes[-1].double()
        return torch.stack(planes)

    def operand(self, v, is_mc):
        return self.mc(v) if is_mc else self.plain(v)[None]


def prepare(case, seed):
    """Inputs on the GPU: weights U(+-1/32) or 1/sqrt(K)-scaled normals, unit-scale
    activations, gradients of a mean loss."""
    d, kind = _Draws(case, seed), case["kind"]
    s = {"case": case}
    if kind == "update":
        n = case["n"]
        s["W"] = d.mc(d.uniform(-1 / 32, 1 / 32, n))
        s["G"] = d.mc(d.normal(n, scale=0.05))
        s["neg_lr"] = torch.full((n,), -0.05, dtype=d.dtype, device="cuda")
    elif kind == "elementwise":
        s["x"] = d.mc(d.uniform(-0.5, 0.5, case["n"]))
        s["y"] = d.mc(d.uniform(0.5, 1.5, case["n"]))
    elif kind in ("matmul", "splitk"):
        M, N, K = case["M"], case["N"], case["K"]
        s["A"] = d.operand(d.normal(M, K, scale=K ** -0.5), case["a_mc"])
        s["B"] = d.operand(d.normal(K, N, scale=K ** -0.5), case["b_mc"])
    elif kind == "batched":
        B, M, N, K = case["B"], case["M"], case["N"], case["K"]
        s["A"] = d.operand(d.normal(B, M, K, scale=K ** -0.5), case["a_mc"])
        s["B"] = d.operand(d.normal(B, K, N, scale=K ** -0.5), case["b_mc"])
    elif kind in ("linear", "linear_exact"):
        T, I, O = case["batch"], case["inp"], case["out"]
        s["x"] = d.plain(d.normal(T, I))
        s["W"] = d.mc(d.uniform(-1 / 32, 1 / 32, O, I))
        s["b"] = d.mc(d.uniform(-1 / 32, 1 / 32, O))
        if kind == "linear":
            s["dY"] = d.plain(d.normal(T, O, scale=T ** -0.5))
    else:
        n, m = case["n"], case["d"]
        X = d.plain(d.normal(n, m, scale=0.5) - 0.5)
        target = d.normal(m, scale=0.5) - 0.5
        s["X"] = X
        s["y_neg"] = d.plain(-(X.double() @ target))
        s["W"] = d.mc(d.uniform(-1.0, 1.0, m) * m ** -0.5)
        s["loss"] = torch.empty(case["nc"], dtype=d.dtype, device="cuda")
        code = {"f16": mcf.MCF_F16, "f32": mcf.MCF_F32, "f64": mcf.MCF_F64}[case["dtype"]]
        s["workspace"] = torch.empty(mcf.mc_linreg_workspace(code, case["nc"], n, m), dtype=torch.uint8, device="cuda")
    return s


def run(state):
    s, case = state, state["case"]
    kind, nc = case["kind"], case["nc"]
    if kind == "update":  # W <- Grow-ExpN(W, the leading component of ScalingN(G, -lr))
        step = mcf.mc_mul(s["G"], s["neg_lr"], nc=nc, y_mc=False)
        return mcf.mc_add(s["W"], step[0], nc=nc, y_mc=False)
    if kind == "elementwise":
        return (mcf.mc_mul if case["op"] == "mul" else mcf.mc_div)(s["x"], s["y"], nc=nc)
    if kind == "matmul":
        return mcf.mc_matmul(s["A"], s["B"], nc=nc, a_mc=case["a_mc"], b_mc=case["b_mc"])
    if kind == "splitk":
        return mcf.mc_matmul_splitk(s["A"], s["B"], nc=nc, a_mc=case["a_mc"], b_mc=case["b_mc"])
    if kind == "batched":
        return mcf.mc_bmm(s["A"], s["B"], nc=nc, a_mc=case["a_mc"], b_mc=case["b_mc"])
    if kind == "linear":
        y = mcf.mc_linear_fwd(s["x"], s["W"], s["b"])
        dX, dW, db = mcf.mc_linear_bwd(s["x"], s["W"], s["dY"], dy_mc=False)
        return y, dX, dW, db
    if kind == "linear_exact":
        return mcf.mc_linear_fwd_exact(s["x"], s["W"], s["b"])
    mcf.mc_linreg_gd_step(s["X"], s["y_neg"], s["W"], 0.05, loss=s["loss"], workspace=s["workspace"])
    return s["W"], s["loss"]


def _scaling_ops(nc):
    """Operations of ScalingN that its nc kept terms need."""
    return 1 if nc == 1 else 4 + 9 * (nc - 2)


def _add_ops(nc):
    """Operations of Add-MCN that its nc kept terms need."""
    return 1 if nc == 1 else 8 + 13 * (nc - 2)


def _product_work(case, outputs, K, a, b, terms, planes_a, planes_b):
    nc, e = case["nc"], SIZE[case["dtype"]]
    return {"bytes": e * (a * planes_a + b * planes_b + outputs * nc),
            "flops": float(outputs) * K * terms * (_scaling_ops(nc) + _add_ops(nc))}


def work(case):
    """Each input read once, each output written once; the arithmetic of the kept terms."""
    kind, nc, e = case["kind"], case["nc"], SIZE[case["dtype"]]
    if kind == "update":  # reads G, -lr and W, writes W; only the leading product is used
        return {"bytes": e * case["n"] * (1 + 1 + 2 * nc), "flops": case["n"] * (1.0 + 6 * nc)}
    if kind == "elementwise":
        ops = (nc + 1) + nc * (_scaling_ops(nc) + _add_ops(nc))
        return {"bytes": e * case["n"] * 3 * nc, "flops": float(case["n"]) * ops * (2 if case["op"] == "mul" else 1)}
    if kind in ("matmul", "batched", "splitk"):
        batch, M, N, K = case.get("B", 1), case["M"], case["N"], case["K"]
        both = case["a_mc"] and case["b_mc"]
        return _product_work(case, batch * M * N, K, batch * M * K, batch * K * N, nc if both else 1,
                             nc if case["a_mc"] else 1, nc if case["b_mc"] else 1)
    if kind in ("linear", "linear_exact"):
        T, I, O = case["batch"], case["inp"], case["out"]
        w = _product_work(case, T * O, I, T * I, O * I, 1, 1, nc)
        if kind == "linear_exact":  # one exact multiply-add per component of W
            w["flops"] = 2.0 * nc * T * O * I
            return w
        return {"bytes": w["bytes"] + e * (T * O + nc * (T * I + O * I + O)), "flops": 3 * w["flops"]}
    n, m = case["n"], case["d"]
    per = _scaling_ops(nc) + _add_ops(nc)
    return {"bytes": e * (n * (m + 1) + 2 * nc * m + nc), "flops": float(n) * (2 * m + nc) * per}


def tolerance(case):
    """Every output is a fixed sequence of correctly rounded operations of the inputs."""
    return "exact"


def _value(t):
    """The value of an MC tensor in float64."""
    return t.double().flip(0).sum(0)


def _split(v, case):
    """v as the library lays an MC result out: (nc, *shape), by successive rounding."""
    planes = []
    for _ in range(case["nc"]):
        planes.append(v.to(DTYPES[case["dtype"]]).double())
        v = v - planes[-1]
    return torch.stack(planes)


def exact(case, seed):
    """What run() returns for these inputs as plain float64 arithmetic gives it."""
    s, kind = prepare(case, seed), case["kind"]
    if kind == "update":
        step = _split(_value(s["G"]) * s["neg_lr"].double(), case)[0]
        return _split(_value(s["W"]) + step, case)
    if kind == "elementwise":
        x, y = _value(s["x"]), _value(s["y"])
        return _split(x * y if case["op"] == "mul" else x / y, case)
    if kind in ("matmul", "splitk", "batched"):
        return _split(_value(s["A"]) @ _value(s["B"]).contiguous(), case)
    if kind in ("linear", "linear_exact"):
        x, W, b = s["x"].double(), _value(s["W"]), _value(s["b"])
        y = _split(x @ W.t().contiguous() + b, case)
        if kind == "linear_exact":
            return y
        dY = s["dY"].double()
        return y, _split(dY @ W, case), _split(dY.t().contiguous() @ x, case), _split(dY.sum(0), case)
    X, W = s["X"].double(), _value(s["W"])
    r = X @ W + s["y_neg"].double()
    grad = _split((2.0 / case["n"]) * (r @ X), case)[0]
    return _split(W - 0.05 * grad, case), _split((r * r).mean(), case)
