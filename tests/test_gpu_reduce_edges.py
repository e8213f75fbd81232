"""GPU tests of the reductions at the sizes where their launch rule changes,
against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, inputs, need_gpu

pytestmark = pytest.mark.gpu

CODE = {"f32": "F32", "f64": "F64", "bf16": "BF16", "f16": "F16"}
SIZE = {"f32": 4, "f64": 8, "bf16": 2, "f16": 2}


@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("edge", ["one_block", "one_block+1", "deep-1", "deep"])
def test_full_reduction_edges(dtype, edge):
    """The largest single-block input (32 KB), one element more, and both
    sides of the size from which blocks take deeper tiles (2^21)."""
    torch, fx = need_gpu()
    n = {"one_block": 32768 // SIZE[dtype], "one_block+1": 32768 // SIZE[dtype] + 1,
         "deep-1": (1 << 21) - 1, "deep": 1 << 21}[edge]
    host, (X, Y) = inputs(21, n, dtype, k=2)
    dc = getattr(fx, CODE[dtype])
    split = fx.fx_resolve_launch(fx.R_ACCU, dc, (n, 1))[3]
    assert (split == 1) == (edge == "one_block")
    ws = fx.workspace(fx.R_ACCU, dc, (n, 1))
    out = torch.full((1,), np.nan, dtype=torch.float64, device="cuda")
    nodes = [("leaf", -1, -1, 0, 0), ("leaf", -1, -1, 1, 0), ("mul", 0, 1, -1, 0)]
    rtc = fx.Rtc(nodes, dc, fx.R_ACCU)
    v, mu = oracle.evaluate(oracle.EXPRS["xy"], host, dtype, shape=(n, 1), reduce="accu")
    for what, call in (("fused", lambda: fx.fx_accu_xy(X, Y, out, ws)),
                       ("source", lambda: rtc.eval([X, Y], out, (n, 1), ws))):
        for rep in range(2):                      # the workspace is left as it was found
            out.fill_(float("nan"))
            call()
            torch.cuda.synchronize()
            assert_close(out.cpu().numpy(), v, mu, dtype, "%s %s %d" % (what, edge, rep))


@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("shape", [(1, 5000), (5, 4097), (64, 3000), (72, 1000), (200, 333),
                                   (512, 700), (1000, 129), (4096, 3), (33000, 2)])
def test_row_sum_tiles(dtype, shape):
    """Row tiles from one row to the full 64 vectors, remainders of the row
    tile and of the column step, chunk counts from one to more than there are
    steps; through the fused, source and tape paths."""
    torch, fx = need_gpu()
    rows, cols = shape
    host, (X, Y, W) = inputs(22, rows * cols, dtype)
    dc = getattr(fx, CODE[dtype])
    acc = torch.float64 if dtype == "f64" else torch.float32
    out = torch.empty(rows, dtype=acc, device="cuda")
    v, mu = oracle.evaluate(oracle.EXPRS["c2_z"], host, dtype, shape=shape, reduce="rowsum")
    for cfg in (None, (64, 1, 16, 1), (256, 2, 16, 3), (512, 4, 16, 40), (192, 2, SIZE[dtype], 5)):
        ws = fx.workspace(fx.R_ROWSUM, dc, shape, cfg)
        for rep in range(2):
            out.fill_(float("nan"))
            fx.fx_c2_rowsum(X, Y, W, out, shape, ws, cfg)
            torch.cuda.synchronize()
            assert_close(out.cpu().numpy(), v, mu, dtype, "%s %s %d" % (shape, cfg, rep))
    nodes = [("leaf", -1, -1, 0, 0), ("leaf", -1, -1, 1, 0), ("mul", 0, 1, -1, 0)]
    v, mu = oracle.evaluate(oracle.EXPRS["xy"], host, dtype, shape=shape, reduce="rowsum")
    ws = fx.workspace(fx.R_ROWSUM, dc, shape)
    rtc, tape = fx.Rtc(nodes, dc, fx.R_ROWSUM), fx.Tape(nodes)
    for what, call in (("source", lambda: rtc.eval([X, Y], out, shape, ws)),
                       ("tape", lambda: fx.fx_tape_eval(tape, [X, Y], out, shape, fx.R_ROWSUM, ws))):
        out.fill_(float("nan"))
        call()
        torch.cuda.synchronize()
        assert_close(out.cpu().numpy(), v, mu, dtype, "%s %s" % (what, shape))
