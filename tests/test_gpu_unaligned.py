"""GPU tests of 16-byte vectors at any element: arrays that start at odd
elements of their buffers (each at another), columns that are no whole number
of vectors, and outputs whose neighbours must stay untouched; against the
oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import TORCH_DT, assert_close, from_dev, inputs, need_gpu

pytestmark = pytest.mark.gpu

CODE = {"f32": "F32", "f64": "F64", "bf16": "BF16", "f16": "F16", "u32": "U32"}
PAD = 16


def _shifted(torch, t, shift):
    """A copy of t that starts `shift` elements into its buffer."""
    buf = torch.zeros(t.numel() + 2 * PAD, dtype=t.dtype, device="cuda")
    at = buf[PAD + shift:PAD + shift + t.numel()]
    at.copy_(t) if t.dtype != torch.uint32 else at.view(torch.int32).copy_(t.view(torch.int32))
    return at


def _output(torch, n, dtype, shift):
    """n elements between sentinels, `shift` elements into their buffer."""
    dt = getattr(torch, TORCH_DT[dtype])
    buf = torch.full((n + 2 * PAD,), 77, dtype=torch.int32 if dtype == "u32" else dt, device="cuda")
    buf = buf.view(dt) if dtype == "u32" else buf
    return buf, buf[PAD + shift:PAD + shift + n]


def _margins_kept(torch, buf, n, shift):
    b = buf.view(torch.int32) if buf.dtype == torch.uint32 else buf
    return bool((b[:PAD + shift] == 77).all()) and bool((b[PAD + shift + n:] == 77).all())


@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16", "f16", "u32"])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 8191, 8193, 70001])
def test_element_wise_and_accu(dtype, n):
    torch, fx = need_gpu()
    host, dev = inputs(31, n, dtype)
    if dtype != "u32":
        v, mu = oracle.evaluate(oracle.EXPRS["c1_z"], host, dtype)
        sv, smu = oracle.evaluate(oracle.EXPRS["xy"], host, dtype, reduce="accu")
    dc = getattr(fx, CODE[dtype])
    ws = fx.workspace(fx.R_ACCU, dc, (n, 1))
    for shifts in ((1, 2, 3, 5), (0, 1, 0, 0), (7, 7, 7, 7), (0, 0, 0, 1)):
        X, Y, W = (_shifted(torch, t, k) for t, k in zip(dev, shifts))
        buf, Z = _output(torch, n, dtype, shifts[3])
        s = torch.zeros(1, dtype=torch.int64 if dtype == "u32" else torch.float64, device="cuda")
        fx.fx_c1_z(X, Y, W, Z)
        fx.fx_accu_xy(X, Y, s, ws)
        torch.cuda.synchronize()
        assert _margins_kept(torch, buf, n, shifts[3])
        if dtype == "u32":
            x, y, w = (h.astype(np.uint64) for h in host)
            want = ((x ^ y) + 3 * w) & 0xFFFFFFFF
            assert np.array_equal(from_dev(Z, dtype).astype(np.uint64), want)
            assert int(s.item()) & (2 ** 64 - 1) == int(((x * y) & 0xFFFFFFFF).sum()) & (2 ** 64 - 1)
        else:
            half = dtype if dtype in ("bf16", "f16") else None
            assert_close(from_dev(Z, dtype), v, mu, dtype, "Z %d %s" % (n, shifts), half)
            assert_close(s.cpu().numpy(), sv, smu, dtype, "accu %d %s" % (n, shifts))


@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(1, 9), (3, 40), (7, 33), (9, 65), (33, 50), (63, 20), (129, 17),
                                   (1025, 9), (4099, 5), (65, 700), (8191, 3)])
def test_dimension_sums_of_ragged_columns(dtype, shape):
    torch, fx = need_gpu()
    rows, cols = shape
    host, dev = inputs(32, rows * cols, dtype)
    dc = getattr(fx, CODE[dtype])
    acc = torch.float64 if dtype == "f64" else torch.float32
    nodes = [("leaf", -1, -1, 0, 0), ("leaf", -1, -1, 1, 0), ("mul", 0, 1, -1, 0)]
    tape = fx.Tape(nodes)
    for kind, name, call, nout in ((fx.R_COLSUM, "colsum", fx.fx_c2_colsum, cols),
                                   (fx.R_ROWSUM, "rowsum", fx.fx_c2_rowsum, rows)):
        v, mu = oracle.evaluate(oracle.EXPRS["c2_z"], host, dtype, shape=shape, reduce=name)
        xv, xmu = oracle.evaluate(oracle.EXPRS["xy"], host, dtype, shape=shape, reduce=name)
        for shifts in ((0, 0, 0), (1, 3, 2)):
            X, Y, W = (_shifted(torch, t, k) for t, k in zip(dev, shifts))
            for cfg in (None, (64, 1, 16, 3), (256, 2, 16, 1)):
                out = torch.full((nout,), np.nan, dtype=acc, device="cuda")
                call(X, Y, W, out, shape, fx.workspace(kind, dc, shape, cfg), cfg)
                torch.cuda.synchronize()
                assert_close(out.cpu().numpy(), v, mu, dtype, "%s %s %s" % (name, shifts, cfg))
            for cfg in (None, (128, 2, 8 if dtype != "f64" else 16, 2)):
                out = torch.full((nout,), np.nan, dtype=acc, device="cuda")
                fx.fx_tape_eval(tape, [X, Y], out, shape, kind, fx.workspace(kind, dc, shape, cfg), cfg)
                torch.cuda.synchronize()
                assert_close(out.cpu().numpy(), xv, xmu, dtype, "tape %s %s" % (name, cfg))
        rtc = fx.Rtc(nodes, dc, kind)
        out = torch.full((nout,), np.nan, dtype=acc, device="cuda")
        rtc.eval(dev[:2], out, shape, fx.workspace(kind, dc, shape))
        torch.cuda.synchronize()
        assert_close(out.cpu().numpy(), xv, xmu, dtype, "source %s" % name)


def test_non_finite_neighbours_stay_out():
    """The vector that overlaps the one before must not let a repeated lane
    into a sum: a column's last vector repeats elements that are infinite."""
    torch, fx = need_gpu()
    rows, cols = 8 * 5 + 3, 6
    x = torch.ones(cols, rows, dtype=torch.bfloat16, device="cuda")
    x[:, 37] = float("inf")                  # row 37: inside the overlap of the last vector
    y = torch.ones_like(x)
    y[:, 37] = 0.0                           # inf * 0: NaN in every column's sum
    out = torch.empty(cols, device="cuda")
    fx.fx_colsum_xy(x, y, out, (rows, cols), fx.workspace(fx.R_COLSUM, fx.BF16, (rows, cols)))
    torch.cuda.synchronize()
    assert torch.isnan(out).all()
    y[:, 37] = 1.0                           # one infinity per column, counted once
    fx.fx_colsum_xy(x, y, out, (rows, cols), fx.workspace(fx.R_COLSUM, fx.BF16, (rows, cols)))
    torch.cuda.synchronize()
    assert torch.isinf(out).all()
    row = torch.empty(rows, device="cuda")
    fx.fx_reduce(fx.R_ROWSUM, x, None, row, (rows, cols), fx.workspace(fx.R_ROWSUM, fx.BF16, (rows, cols)))
    torch.cuda.synchronize()
    want = torch.full((rows,), float(cols), device="cuda")
    want[37] = float("inf")
    assert torch.equal(row, want)
