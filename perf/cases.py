"""The workloads by which the library's speed is measured.

Each case is one use of the public entry points over fixed sizes, drawn from
the library's own benchmark (the vector, matrix, paper-suite, view, tape,
batch and launch-model workloads) and from the sizes between and around them:
calls so small that only their latency counts, odd and ragged shapes, the
largest arrays, every storage type.  draw() gives further cases of the same
ranges.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2604_22242_amd as fx

TORCH = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16,
         "f16": torch.float16, "u32": torch.int32}
CODE = {"f32": fx.F32, "f64": fx.F64, "bf16": fx.BF16, "f16": fx.F16, "u32": fx.U32}
SIZE = {"f32": 4, "f64": 8, "bf16": 2, "f16": 2, "u32": 4}
DEV = "cuda"


def listed():
    return [
        # a fused expression and its sum on a vector of a few hundred elements:
        # launch latency and the host path
        {"name": "vec_1k_f32", "family": "vec", "dtype": "f32", "n": 1000, "shift": 0},
        # the 2^20 vector workload: everything fits the last-level cache
        {"name": "vec_1m_f32", "family": "vec", "dtype": "f32", "n": 1 << 20, "shift": 0},
        # the 2^28 low-precision workload: half storage streamed from HBM
        {"name": "vec_268m_bf16", "family": "vec", "dtype": "bf16", "n": 1 << 28, "shift": 0},
        # the matrix workload, its result and all its reductions
        {"name": "mat_8192_f32", "family": "mat", "dtype": "f32", "rows": 8192, "cols": 8192,
         "shift": 0},
        # the same in BF16 storage: half the bytes, the same arithmetic
        {"name": "mat_8192_bf16", "family": "mat", "dtype": "bf16", "rows": 8192, "cols": 8192,
         "shift": 0},
        # a matrix whose columns are no whole number of vectors, FP16 storage
        {"name": "mat_odd_f16", "family": "mat", "dtype": "f16", "rows": 6001, "cols": 2999,
         "shift": 0},
        # the paper's element-wise expressions at its size
        {"name": "paper_10k_f32", "family": "paper", "dtype": "f32", "rows": 10000, "cols": 10000},
        # the paper's submatrix, transpose and diagonal expressions at its size
        {"name": "views_10k_f32", "family": "views", "dtype": "f32", "m": 10000},
        # the same over an odd leading dimension in FP64
        {"name": "views_odd_f64", "family": "views", "dtype": "f64", "m": 3001},
        # a deep tree known only at run time, its values and its sum
        {"name": "tape_16m_f32", "family": "tape", "dtype": "f32", "rows": 4096, "cols": 4096,
         "tree": 30, "depth": 8, "kinds": "ew+accu", "mode": "tape"},
        # thousands of uneven expressions replayed as one launch
        {"name": "batch_4096_f32", "family": "batch", "dtype": "f32", "count": 4096, "tree": 4,
         "graph": True},
        # the launch-configuration model fitted to a tuning database and applied to it
        {"name": "model_20k", "family": "model", "rows": 20000, "batch": 256, "epochs": 2},
    ]


# ---- draws ---------------------------------------------------------------------------


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: a workload at random, sizes log-uniform over its range."""
    family = rng.choice(("vec", "vec", "mat", "mat", "mat", "paper", "views", "views", "tape",
                         "tape", "batch", "model"))
    if family == "vec":
        dtype = rng.choice(("f32", "f64", "bf16", "f16", "u32"))
        return {"family": family, "dtype": dtype, "n": _log_int(rng, 500, (1 << 29) // SIZE[dtype]),
                "shift": rng.choice((0, 0, 0, 1))}
    if family == "mat":
        dtype = rng.choice(("f32", "f64", "bf16", "f16"))
        size = _log_int(rng, 1 << 10, (1 << 27) // SIZE[dtype])
        rows = _log_int(rng, 4, 1 << 15)
        return {"family": family, "dtype": dtype, "rows": rows,
                "cols": max(1, min(1 << 15, size // rows)), "shift": rng.choice((0, 0, 0, 1))}
    if family == "paper":
        return {"family": family, "dtype": rng.choice(("f32", "bf16")),
                "rows": _log_int(rng, 16, 10000), "cols": _log_int(rng, 16, 10000)}
    if family == "views":
        return {"family": family, "dtype": rng.choice(("f32", "f64", "bf16")),
                "m": _log_int(rng, 60, 7000)}
    if family == "tape":
        size = _log_int(rng, 1 << 12, 1 << 24)
        rows = _log_int(rng, 64, 1 << 13)
        return {"family": family, "dtype": rng.choice(("f32", "f64", "bf16", "f16")),
                "rows": rows, "cols": max(1, size // rows), "tree": rng.randrange(1 << 20),
                "depth": rng.randint(2, 8),
                "kinds": rng.choice(("ew", "ew+accu", "accu", "norm", "colsum", "rowsum")),
                "mode": rng.choice(("tape", "tape", "rtc"))}
    if family == "batch":
        return {"family": family, "dtype": rng.choice(("f32", "f64", "bf16", "f16")),
                "count": _log_int(rng, 8, 2048), "tree": rng.randrange(1 << 20),
                "graph": rng.choice((True, False))}
    return {"family": family, "rows": _log_int(rng, 300, 20000), "batch": rng.choice((64, 128, 256, 500)),
            "epochs": rng.randint(1, 2)}


# ---- inputs --------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _uniform(g, n, dtype, lo=-1.0, hi=1.0, shift=0):
    """n values of U[lo, hi) (31-bit integers for u32), rounded once to the
    storage type, starting `shift` elements into their buffer."""
    if dtype == "u32":
        buf = torch.randint(0, 1 << 31, (n + shift,), generator=g, device=DEV, dtype=torch.int32) \
            if n + shift else torch.empty(0, device=DEV, dtype=torch.int32)
    else:
        wide = torch.float64 if dtype == "f64" else torch.float32
        buf = torch.rand(n + shift, generator=g, device=DEV, dtype=wide)
        buf = buf.mul_(hi - lo).add_(lo).to(TORCH[dtype])
    return buf[shift:]


def _empty(n, dtype, shift=0):
    return torch.empty(n + shift, dtype=TORCH[dtype], device=DEV)[shift:]


def _acc(dtype):
    return torch.float64 if dtype == "f64" else torch.float32


def _wide(t):
    return t.to(torch.float64)


# ---- vectors: Z = X % Y + 2W (u32: (X ^ Y) + 3W) and accu(X % Y) ----------------------------


def _vec_prepare(c, seed):
    g, n, d, k = _gen(seed), c["n"], c["dtype"], c["shift"]
    X, Y, W = (_uniform(g, n, d, shift=k) for _ in range(3))
    s = torch.zeros(1, dtype=torch.int64 if d == "u32" else torch.float64, device=DEV)
    return {"X": X, "Y": Y, "W": W, "Z": _empty(n, d, k), "s": s,
            "ws": fx.workspace(fx.R_ACCU, CODE[d], (n, 1))}


def _vec_run(s):
    fx.fx_c1_z(s["X"], s["Y"], s["W"], s["Z"])
    fx.fx_accu_xy(s["X"], s["Y"], s["s"], s["ws"])
    return {"Z": s["Z"], "accu": s["s"]}


def _vec_exact(c, s):
    if c["dtype"] == "u32":
        return None
    X, Y, W = _wide(s["X"]), _wide(s["Y"]), _wide(s["W"])
    XY = X * Y
    return {"Z": XY + 2 * W, "accu": XY.sum().reshape(1)}


def _vec_work(c):
    b = SIZE[c["dtype"]]
    return {"bytes": (4 + 2) * b * c["n"] + 8, "flops": 5 * c["n"]}


# ---- matrices: C2's result, column sums, row sums and norm_fro(X - Y) ----------------------


def _mat_prepare(c, seed):
    g, d, k = _gen(seed), c["dtype"], c["shift"]
    r, q = c["rows"], c["cols"]
    X, Y, W = (_uniform(g, r * q, d, shift=k) for _ in range(3))
    code = CODE[d]
    return {"X": X, "Y": Y, "W": W, "Z": _empty(r * q, d, k), "shape": (r, q),
            "col": torch.empty(q, dtype=_acc(d), device=DEV),
            "row": torch.empty(r, dtype=_acc(d), device=DEV),
            "norm": torch.zeros(1, dtype=torch.float64, device=DEV),
            "wc": fx.workspace(fx.R_COLSUM, code, (r, q)),
            "wr": fx.workspace(fx.R_ROWSUM, code, (r, q)),
            "wn": fx.workspace(fx.R_NORM, code, (r, q))}


def _mat_run(s):
    X, Y, W, sh = s["X"], s["Y"], s["W"], s["shape"]
    fx.fx_c2_z(X, Y, W, s["Z"], sh)
    fx.fx_c2_colsum(X, Y, W, s["col"], sh, s["wc"])
    fx.fx_c2_rowsum(X, Y, W, s["row"], sh, s["wr"])
    fx.fx_norm_fro_diff(X, Y, s["norm"], sh, s["wn"])
    return {"Z": s["Z"], "col": s["col"], "row": s["row"], "norm": s["norm"]}


def _mat_exact(c, s):
    X, Y, W = _wide(s["X"]), _wide(s["Y"]), _wide(s["W"])
    Z = (X + Y) * torch.exp(-W.abs()) / (1 + X * X)
    M = Z.view(c["cols"], c["rows"])  # column-major: one row of M per column
    return {"Z": Z, "col": M.sum(1), "row": M.sum(0),
            "norm": (X - Y).square().sum().sqrt().reshape(1)}


def _mat_work(c):
    n, b = c["rows"] * c["cols"], SIZE[c["dtype"]]
    a = 8 if c["dtype"] == "f64" else 4
    return {"bytes": (4 + 3 + 3 + 2) * b * n + a * (c["rows"] + c["cols"]) + 8, "flops": 27 * n}


# ---- the paper's element-wise expressions ----------------------------------------------------

_PAPER = ("add4", "relu", "sigmoid", "swish", "gelu", "expr3")
_ALPHA, _BETA = 0.044715, 1.0


def _paper_prepare(c, seed):
    g, d, n = _gen(seed), c["dtype"], c["rows"] * c["cols"]
    A, B, C = (_uniform(g, n, d) for _ in range(3))
    D = _uniform(g, n, d, 1.0, 2.0)   # expr3's W: both logarithms stay finite
    Y = _uniform(g, n, "f64")         # expr3's Y, converted inside the expression
    return {"A": A, "B": B, "C": C, "D": D, "Y": Y, "shape": (c["rows"], c["cols"]),
            "out": {e: _empty(n, d) for e in _PAPER}}


def _paper_run(s):
    A, sh, o = s["A"], s["shape"], s["out"]
    fx.fx_paper_expr("add4", [A, s["B"], s["C"], s["D"]], o["add4"], sh)
    fx.fx_paper_expr("relu", [A], o["relu"], sh)
    fx.fx_paper_expr("sigmoid", [A], o["sigmoid"], sh)
    fx.fx_paper_expr("swish", [A], o["swish"], sh, scalars=(_BETA,))
    fx.fx_paper_expr("gelu", [A], o["gelu"], sh, scalars=(_ALPHA,))
    fx.fx_paper_expr("expr3", [A, s["Y"], s["D"]], o["expr3"], sh)
    return dict(o)


def _paper_exact(c, s):
    A, B, C, D = (_wide(s[k]) for k in "ABCD")
    r = {"add4": A + B + C + D, "relu": A * (A > 0), "sigmoid": 1 / (1 + torch.exp(-A)),
         "swish": A / (1 + torch.exp(-_BETA * A)),
         "gelu": (A / 2) * (1 + torch.tanh(math.sqrt(2 / math.pi) * (A + _ALPHA * A ** 3)))}
    # expr3 divides by a sum that cancels to nearly nothing here and there:
    # no accuracy can be asked of it
    r["expr3"] = None
    return r


def _paper_work(c):
    n, b = c["rows"] * c["cols"], SIZE[c["dtype"]]
    return {"bytes": n * ((5 + 2 * 4 + 3) * b + 8), "flops": 40 * n}


# ---- the paper's strided views ------------------------------------------------------------

_VIEWS = ("addsub2", "addsub4", "expr1", "expr2", "diagsum")


def _views_prepare(c, seed):
    g, d, m = _gen(seed), c["dtype"], c["m"]
    A, B, C = (_uniform(g, m * m, d) for _ in range(3))
    D = _uniform(g, m * m, d, 1.0, 2.0)
    out = {}
    for e in _VIEWS:
        r, q = fx.fx_paper_view_shape(e, (m, m))
        out[e] = _empty(r * q, d)
    return {"A": A, "B": B, "C": C, "D": D, "shape": (m, m), "out": out}


def _views_run(s):
    A, B, C, D, sh, o = s["A"], s["B"], s["C"], s["D"], s["shape"], s["out"]
    fx.fx_paper_view_expr("addsub2", [A, B], o["addsub2"], sh)
    fx.fx_paper_view_expr("addsub4", [A, B, C, D], o["addsub4"], sh)
    fx.fx_paper_view_expr("expr1", [A, B], o["expr1"], sh)
    fx.fx_paper_view_expr("expr2", [A, B, C, D], o["expr2"], sh, scalars=(1.5,))
    fx.fx_paper_view_expr("diagsum", [A, B], o["diagsum"], sh)
    return dict(o)


def _views_exact(c, s):
    m = c["m"]
    A, B, C, D = (_wide(s[k]).view(m, m).t() for k in "ABCD")  # t(): rows first
    h, o = m // 2, (m - m // 2) // 2
    cut = [M[o:o + h, o:o + h] for M in (A, B, C, D)]
    X, Y = A, B
    r = {"addsub2": cut[0] + cut[1], "addsub4": cut[0] + cut[1] + cut[2] + cut[3],
         "expr1": 2 * (X.t() + Y) + 2 * (X + Y.t()),
         "expr2": 1.5 * A + (B + C).t() + torch.log(D * D)}
    r = {k: v.t().contiguous().reshape(-1) for k, v in r.items()}
    r["diagsum"] = (torch.diagonal(X, -1) + torch.diagonal(X, 1)) * \
        (torch.diagonal(Y, -1) + torch.diagonal(Y, 1))
    return r


def _views_work(c):
    n, b = c["m"] ** 2, SIZE[c["dtype"]]
    return {"bytes": n * b * (3 / 4 + 5 / 4 + 3 + 5) + 5 * b * c["m"],
            "flops": n * (1 / 4 + 3 / 4 + 5 + 24)}


# ---- run-time trees --------------------------------------------------------------------------


def _tree(rng, depth, n_inputs):
    """A random tree as the library's batch and tuning workloads draw them:
    one branch forced to `depth`, every other operand internal with
    probability 1/2, and guards that keep every value finite."""
    nodes = []

    def add(op, a=-1, b=-1, inp=-1, val=0.0):
        nodes.append((op, a, b, inp, val))
        return len(nodes) - 1

    def grow(d, forced):
        if d == depth or (not forced and rng.random() < 0.5):
            if rng.random() < 0.1:
                return add("const", val=rng.choice((0.5, 1.0, 2.0, 3.0)))
            return add("leaf", inp=rng.randrange(n_inputs))
        op = rng.choice(("add", "sub", "mul", "div", "exp", "abs", "sqrt"))
        if op in ("exp", "abs", "sqrt"):
            a = grow(d + 1, forced)
            if op == "abs":
                return add("abs", a)
            if op == "sqrt":
                return add("sqrt", add("abs", a))
            return add("exp", add("sub", add("const", val=0.0), add("abs", a)))
        left = rng.random() < 0.5
        a = grow(d + 1, forced and left)
        b = grow(d + 1, forced and not left)
        if op == "div":
            b = add("add", add("const", val=1.0), add("abs", b))
        return add(op, a, b)

    grow(0, True)
    used = {}
    nodes = [(op, a, b, used.setdefault(i, len(used)) if op == "leaf" else i, v)
             for op, a, b, i, v in nodes]
    return nodes, len(used)


def _tree_value(nodes, inputs, n):
    """The tree in FP64, one operator at a time."""
    v = []
    for op, a, b, i, val in nodes:
        if op == "leaf":
            v.append(inputs[i])
        elif op == "const":
            v.append(torch.full((n,), val, dtype=torch.float64, device=DEV))
        elif op in ("abs", "exp", "sqrt"):
            v.append(getattr(torch, op)(v[a]))
        else:
            v.append(getattr(torch, op)(v[a], v[b]))
    return v[-1]


_KIND = {"ew": 0, "accu": fx.R_ACCU, "norm": fx.R_NORM, "colsum": fx.R_COLSUM,
         "rowsum": fx.R_ROWSUM}


def _tape_tree(c):
    rng = random.Random(c["tree"])
    nodes, k = _tree(rng, c["depth"], 4)
    while len(nodes) > 64 or k == 0:  # within the tape's limits, and with an input
        nodes, k = _tree(rng, c["depth"], 4)
    return nodes, k


def _tape_prepare(c, seed):
    g, d, r, q = _gen(seed), c["dtype"], c["rows"], c["cols"]
    nodes, k = _tape_tree(c)
    kinds, code = c["kinds"].split("+"), CODE[d]
    out, ws, prog = {}, {}, {}
    tape = fx.Tape(nodes) if c["mode"] == "tape" else None
    for kind in kinds:
        out[kind] = (_empty(r * q, d) if kind == "ew"
                     else torch.empty(q if kind == "colsum" else r, dtype=_acc(d), device=DEV)
                     if kind in ("colsum", "rowsum")
                     else torch.zeros(1, dtype=torch.float64, device=DEV))
        ws[kind] = fx.workspace(_KIND[kind], code, (r, q)) if kind != "ew" else None
        prog[kind] = tape if tape is not None else fx.Rtc(nodes, code, _KIND[kind])
    return {"in": [_uniform(g, r * q, d) for _ in range(k)], "shape": (r, q), "kinds": kinds,
            "out": out, "ws": ws, "prog": prog, "rtc": tape is None}


def _tape_run(s):
    for kind in s["kinds"]:
        if s["rtc"]:
            s["prog"][kind].eval(s["in"], s["out"][kind], s["shape"], s["ws"][kind])
        else:
            fx.fx_tape_eval(s["prog"][kind], s["in"], s["out"][kind], s["shape"], _KIND[kind],
                            s["ws"][kind])
    return dict(s["out"])


def _tape_exact(c, s):
    nodes, _ = _tape_tree(c)
    r, q = c["rows"], c["cols"]
    Z = _tree_value(nodes, [_wide(t) for t in s["in"]], r * q)
    M = Z.view(q, r)
    every = {"ew": lambda: Z, "accu": lambda: Z.sum().reshape(1),
             "norm": lambda: Z.square().sum().sqrt().reshape(1),
             "colsum": lambda: M.sum(1), "rowsum": lambda: M.sum(0)}
    return {k: every[k]() for k in c["kinds"].split("+")}


def _tape_work(c):
    nodes, k = _tape_tree(c)
    n, b = c["rows"] * c["cols"], SIZE[c["dtype"]]
    kinds = c["kinds"].split("+")
    ops = sum(op not in ("leaf", "const") for op, *_ in nodes)
    return {"bytes": n * b * sum(k + (kind == "ew") for kind in kinds) + 8,
            "flops": n * ops * len(kinds)}


# ---- batches -------------------------------------------------------------------------------


def _batch_items(c):
    """(nodes, inputs, n, reduces) of every expression: depth 2 to 6, sizes
    lognormal in [256, 2^20], every other one ending in accu."""
    rng = random.Random(c["tree"])
    items = []
    for e in range(c["count"]):
        nodes, k = _tree(rng, rng.randint(2, 6), rng.randint(1, 4))
        n = 0
        while not 256 <= n <= 1 << 20:
            n = int(round(math.exp(rng.gauss(math.log(2 ** 14), 2 * math.log(2)))))
        items.append((nodes, k, n, e % 2 == 1))
    return items


def _batch_layout(c):
    """Offsets of the items' inputs and outputs in two buffers, each a whole
    number of 16-byte vectors from the next."""
    at_in, at_out, pos_in, pos_out = [], [], 0, 0
    for nodes, k, n, reduces in _batch_items(c):
        step = (n + 7) // 8 * 8
        at_in.append(pos_in)
        pos_in += k * step
        at_out.append(pos_out)
        pos_out += 0 if reduces else step
    return at_in, at_out, pos_in, pos_out


def _batch_prepare(c, seed):
    d = c["dtype"]
    at_in, at_out, n_in, n_out = _batch_layout(c)
    data = _uniform(_gen(seed), n_in, d)
    Z = torch.zeros(max(1, n_out), dtype=TORCH[d], device=DEV)
    sums = torch.zeros(max(1, c["count"] // 2), dtype=torch.float64, device=DEV)
    items = []
    for e, (nodes, k, n, reduces) in enumerate(_batch_items(c)):
        step = (n + 7) // 8 * 8
        ins = [data[at_in[e] + q * step:at_in[e] + q * step + n] for q in range(k)]
        out = sums[e // 2:] if reduces else Z[at_out[e]:at_out[e] + n]
        items.append((fx.Tape(nodes), ins, out, n, fx.R_ACCU if reduces else 0))
    torch.cuda.synchronize()  # the batch runs on a stream of its own
    return {"batch": fx.Batch(items, CODE[d]), "stream": torch.cuda.Stream(), "data": data,
            "Z": Z, "sums": sums, "graph": c["graph"]}


def _batch_run(s):
    if s["graph"]:
        s["batch"].graph(s["stream"])
    else:
        s["batch"].launch(s["stream"])
    return {"Z": s["Z"], "sums": s["sums"]}


def _batch_exact(c, s):
    at_in, at_out, _, n_out = _batch_layout(c)
    Z = torch.zeros(max(1, n_out), dtype=torch.float64, device=DEV)
    sums = torch.zeros(max(1, c["count"] // 2), dtype=torch.float64, device=DEV)
    for e, (nodes, k, n, reduces) in enumerate(_batch_items(c)):
        step = (n + 7) // 8 * 8
        ins = [_wide(s["data"][at_in[e] + q * step:at_in[e] + q * step + n]) for q in range(k)]
        v = _tree_value(nodes, ins, n)
        if reduces:
            sums[e // 2] = v.sum()
        else:
            Z[at_out[e]:at_out[e] + n] = v
    return {"Z": Z, "sums": sums}


def _batch_work(c):
    b, total, ops = SIZE[c["dtype"]], 0, 0
    for nodes, k, n, reduces in _batch_items(c):
        total += n * b * (k + (not reduces)) + (8 if reduces else 0)
        ops += n * sum(op not in ("leaf", "const") for op, *_ in nodes)
    return {"bytes": total, "flops": ops}


# ---- the launch-configuration model --------------------------------------------------------

_F, _H, _HEADS = 25, 64, (4, 3, 3, 4)
_LR = 2e-3


def _model_init(seed):
    r = np.random.default_rng(seed)
    C = sum(_HEADS)
    p = [r.standard_normal((_H, _F)) / math.sqrt(_F), np.zeros(_H),
         r.standard_normal((C, _H)) / math.sqrt(_H), np.zeros(C)]
    mean, std = r.uniform(0, 8, _F), r.uniform(0.5, 4, _F)
    return (np.concatenate([a.ravel() for a in p]).astype(np.float32), mean.astype(np.float32),
            std.astype(np.float32))


def _model_prepare(c, seed):
    n, g = c["rows"], _gen(seed)
    params, mean, std = _model_init(seed)
    X = torch.randn(n, _F, generator=g, device=DEV)
    T = torch.randn(_F, sum(_HEADS), generator=g, device=DEV)  # what the labels follow
    scores = X @ T + torch.randn(n, sum(_HEADS), generator=g, device=DEV)
    labels = torch.stack([s.argmax(1) for s in scores.split(_HEADS, 1)], 1).to(torch.int32)
    X = (X * torch.from_numpy(std).to(DEV) + torch.from_numpy(mean).to(DEV)).contiguous()
    r = np.random.default_rng(seed + 1)
    perm = np.stack([r.permutation(n) for _ in range(c["epochs"])]).astype(np.int32)
    m = fx.Model(_F, _H, _HEADS)
    m.set(params, mean, std)
    return {"m": m, "params": params, "mean": mean, "std": std, "X": X,
            "labels": labels.contiguous(), "perm": perm, "epochs": c["epochs"],
            "batch": c["batch"], "losses": torch.zeros(c["epochs"], device=DEV),
            "logits": torch.empty(n, sum(_HEADS), device=DEV)}


def _model_run(s):
    m = s["m"]
    m.set(s["params"])  # a fresh fit, as each new database gets
    m.train(s["X"], s["labels"], s["epochs"], s["batch"], _LR, s["perm"], s["losses"])
    m.forward(s["X"], s["logits"])
    return {"params": m.get()[0], "losses": s["losses"], "logits": s["logits"]}


def _model_exact(c, s):
    X = (_wide(s["X"]) - _wide(torch.from_numpy(s["mean"]).to(DEV))) / \
        _wide(torch.from_numpy(s["std"]).to(DEV))
    labels, n, C = s["labels"].long(), c["rows"], sum(_HEADS)
    flat = torch.from_numpy(s["params"].astype(np.float64)).to(DEV)
    cuts = (_H * _F, _H, C * _H, C)

    def net(p, x):
        w1, b1, w2, b2 = p.split(cuts)
        h = torch.relu(x @ w1.view(_H, _F).t() + b1)
        return h @ w2.view(C, _H).t() + b2

    mom, var, step, losses = torch.zeros_like(flat), torch.zeros_like(flat), 0, []
    for e in range(c["epochs"]):
        order = torch.from_numpy(s["perm"][e].astype(np.int64)).to(DEV)
        for at in range(0, n, c["batch"]):
            rows = order[at:at + c["batch"]]
            p = flat.clone().requires_grad_(True)
            loss = sum(torch.nn.functional.cross_entropy(z, labels[rows, q], reduction="sum")
                       for q, z in enumerate(net(p, X[rows]).split(_HEADS, 1))) / len(rows)
            loss.backward()
            step += 1
            mom = 0.9 * mom + 0.1 * p.grad
            var = 0.999 * var + 0.001 * p.grad ** 2
            flat = flat - _LR * (mom / (1 - 0.9 ** step)) / \
                ((var / (1 - 0.999 ** step)).sqrt() + 1e-8)
        losses.append(loss.detach())
    return {"params": flat.cpu().numpy(), "losses": torch.stack(losses), "logits": net(flat, X)}


def _model_work(c):
    C = sum(_HEADS)
    macs = _F * _H + _H * C
    return {"bytes": 4 * c["rows"] * ((c["epochs"] + 1) * _F + c["epochs"] * (len(_HEADS) + 1) + C),
            "flops": 2 * macs * c["rows"] * (3 * c["epochs"] + 1)}


# ---- the interface --------------------------------------------------------------------------

_FAMILY = {
    "vec": (_vec_prepare, _vec_run, _vec_exact, _vec_work),
    "mat": (_mat_prepare, _mat_run, _mat_exact, _mat_work),
    "paper": (_paper_prepare, _paper_run, _paper_exact, _paper_work),
    "views": (_views_prepare, _views_run, _views_exact, _views_work),
    "tape": (_tape_prepare, _tape_run, _tape_exact, _tape_work),
    "batch": (_batch_prepare, _batch_run, _batch_exact, _batch_work),
    "model": (_model_prepare, _model_run, _model_exact, _model_work),
}


def prepare(case, seed):
    """The case's inputs, buffers and handles on the GPU."""
    return {"run": _FAMILY[case["family"]][1], "state": _FAMILY[case["family"]][0](case, seed)}


def run(state):
    """One pass; returns its outputs whole."""
    return state["run"](state["state"])


def exact(case, seed):
    """What run() returns, from plain torch in FP64."""
    p, _, e, _ = _FAMILY[case["family"]]
    return e(case, p(case, seed))


def work(case):
    """Bytes and operations of one pass that the path cannot do without."""
    return _FAMILY[case["family"]][3](case)
