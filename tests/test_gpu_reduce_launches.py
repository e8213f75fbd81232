"""GPU tests of the dimension sums at both sides of their launch rules' lines,
against FP64 sums."""
import ctypes

import pytest

from gpu_util import need_gpu
from test_gpu_user_views import _lib

pytestmark = pytest.mark.gpu

NODES = [("leaf", -1, -1, 0, 0.0), ("leaf", -1, -1, 1, 0.0), ("mul", 0, 1, -1, 0.0)]


def _inputs(torch, rows, cols, dtype):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    return [(torch.rand(rows * cols, generator=g, device="cuda", dtype=torch.float64) * 2 - 1)
            .to(getattr(torch, dtype)) for _ in range(2)]


def _sums(torch, x, y, rows, cols, dim):
    terms = (x.to(torch.float64) * y.to(torch.float64)).view(cols, rows)
    return terms.sum(1 - dim), terms.abs().sum(1 - dim)


def _check(torch, run, n, acc, want, scale, dtype, terms, what):
    # products rounded to the compute type, FP64 sums, one rounding to the output
    u = 2.0 ** -53 * (terms + 8) if dtype == "float64" else 2.0 ** -24
    for _ in range(2):      # the workspace is left zeroed for the next call
        out = torch.full((n,), float("nan"), dtype=acc, device="cuda")
        run(out)
        torch.cuda.synchronize()
        err = (out.to(torch.float64) - want).abs()
        assert bool((err <= 2.01 * u * scale).all()), what


@pytest.mark.parametrize("dtype", ["float32", "float64", "bfloat16", "float16"])
@pytest.mark.parametrize("rows", [1, 2, 3, 4, 5, 7, 8, 9, 11, 13, 16, 17, 23, 31, 32, 33])
@pytest.mark.parametrize("cols", [4095, 4096, 70001])
def test_short_columns(dtype, rows, cols):
    torch, fx = need_gpu()
    x, y = _inputs(torch, rows, cols, dtype)
    want, scale = _sums(torch, x, y, rows, cols, 0)
    acc = torch.float64 if dtype == "float64" else torch.float32
    ws = fx.workspace(fx.R_COLSUM, fx.dtype_code(x), (rows, cols))
    _check(torch, lambda o: fx.fx_colsum_xy(x, y, o, (rows, cols), ws), cols, acc, want, scale, dtype, rows,
           (rows, cols))


def test_more_short_columns_than_waves_in_a_grid():
    """17 x (2^26 + 5) FP32: a wave per column would be 2^32 threads."""
    torch, fx = need_gpu()
    rows, cols = 17, (1 << 26) + 5
    x = torch.ones(rows * cols, dtype=torch.float32, device="cuda")
    x[-1] = 3.0
    out = torch.zeros(cols, dtype=torch.float32, device="cuda")
    fx.fx_colsum_xy(x, x, out, (rows, cols))
    torch.cuda.synchronize()
    assert bool((out[:-1] == 17).all()) and float(out[-1]) == 25.0


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("kind,rows,cols", [
    (1, (1 << 24) - 1, 1), (1, (1 << 24) + 5, 1), (1, 1000, 1000),     # one and two blocks per CU
    (2, 70001, 3), (2, 40000, 1023), (2, 40000, 1024), (2, 16383, 300)])    # chunked and whole columns
def test_sums_of_functions(dtype, kind, rows, cols):
    """Expressions with divisions and functions in a user's program."""
    torch, fx = need_gpu()
    x, y = _inputs(torch, rows, cols, dtype)
    X, Y = (v.to(torch.float64).view(cols, rows) for v in (x, y))
    terms = X / (1 + Y * Y) if kind == 1 else X.exp() * Y.abs().sqrt() / (1 + Y * Y)
    want, scale = (terms.sum().view(1), terms.abs().sum().view(1)) if kind == 1 else (terms.sum(1), terms.abs().sum(1))
    n, acc = (1, torch.float64) if kind == 1 else (cols, getattr(torch, dtype))
    out = torch.full((n,), float("nan"), dtype=acc, device="cuda")
    ws = fx.workspace(kind, fx.dtype_code(x), (rows, cols))
    ptr = lambda t: ctypes.c_void_p(t.data_ptr() if t is not None else 0)
    f = getattr(_lib(), "user_sums_f32" if dtype == "float32" else "user_sums_f64")
    # each term: exp and sqrt within 2 units together, three roundings, the sum's own
    # (FP64: the reference's too), one rounding to the output
    u = 2.0 ** -24 if dtype == "float32" else 2.0 ** -53 * 2
    for _ in range(2):
        assert f(kind, ptr(x), ptr(y), fx.Shape(rows, cols), ptr(out), ptr(ws),
                 ctypes.c_size_t(ws.numel() if ws is not None else 0),
                 ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        torch.cuda.synchronize()
        err = (out.to(torch.float64) - want).abs()
        bound = (6.5 * u + 2.0 ** -52 * rows * cols / n) * scale
        assert bool((err <= bound).all()), float((err / scale).max())


@pytest.mark.parametrize("dtype", ["float32", "float64", "bfloat16"])
@pytest.mark.parametrize("cols", [7, 300, 5000])
def test_generated_column_sums(dtype, cols):
    """Generated kernels, with as many threads per column as it has work for."""
    torch, fx = need_gpu()
    code = {"float32": fx.F32, "float64": fx.F64, "bfloat16": fx.BF16}[dtype]
    rtc = fx.Rtc(NODES, code, fx.R_COLSUM)
    for rows in (1, 8, 24, 33, 64, 136, 257, 513, 1032, 2049, 8200):
        x, y = _inputs(torch, rows, cols, dtype)
        want, scale = _sums(torch, x, y, rows, cols, 0)
        acc = torch.float64 if dtype == "float64" else torch.float32
        ws = fx.workspace(fx.R_COLSUM, code, (rows, cols))
        for run in (lambda o: rtc.eval([x, y], o, (rows, cols), ws),
                    lambda o: fx.fx_source_eval("colsum_xy", [x, y], o, (rows, cols), ws)):
            _check(torch, run, cols, acc, want, scale, dtype, rows, (rows, cols))


# shapes at the lines of the row sums' lanes: half a wave down a column, a wave,
# two and four waves, the whole block; ragged rows; with one block per row tile and
# with several (the caller's split)
@pytest.mark.parametrize("dtype", ["float32", "float64", "bfloat16"])
@pytest.mark.parametrize("shape", [(1, 70000), (130001, 1), (131072, 2), (32769, 20), (32768, 5), (65537, 33),
                                   (65536, 64), (200003, 1), (262144, 6), (262144, 64), (262151, 9), (1048579, 3),
                                   (1000000, 7), (4194304, 1), (3000001, 2)])
def test_row_sums(dtype, shape):
    torch, fx = need_gpu()
    rows, cols = shape
    code = {"float32": fx.F32, "float64": fx.F64, "bfloat16": fx.BF16}[dtype]
    x, y = _inputs(torch, rows, cols, dtype)
    want, scale = _sums(torch, x, y, rows, cols, 1)
    acc = torch.float64 if dtype == "float64" else torch.float32
    tape, rtc = fx.Tape(NODES), fx.Rtc(NODES, code, fx.R_ROWSUM)
    for cfg in ((0, 0, 0, 0), (0, 0, 0, 2), (192, 1, 0, 3), (64, 2, 16, 0), (512, 2, 0, 2)):
        ws = fx.workspace(fx.R_ROWSUM, code, (rows, cols), cfg)
        runs = [lambda o: fx.fx_tape_eval(tape, [x, y], o, (rows, cols), fx.R_ROWSUM, ws, cfg)]
        if not any(cfg):
            runs.append(lambda o: rtc.eval([x, y], o, (rows, cols), ws))
        for run in runs:
            _check(torch, run, rows, acc, want, scale, dtype, cols, (rows, cols, cfg))


def test_more_rows_than_threads_in_a_grid():
    """2^32 + 8 rows of half storage: with 64 lanes down a column a grid of blocks of
    512 would be 2^32 threads and more."""
    torch, fx = need_gpu()
    rows = (1 << 32) + 8
    x = torch.ones(rows, dtype=torch.bfloat16, device="cuda")
    y = torch.full((rows,), 2.0, dtype=torch.bfloat16, device="cuda")
    y[-1] = 3.0
    out = torch.zeros(rows, dtype=torch.float32, device="cuda")
    ws = fx.workspace(fx.R_ROWSUM, fx.BF16, (rows, 1))
    fx.fx_tape_eval(fx.Tape(NODES), [x, y], out, (rows, 1), fx.R_ROWSUM, ws)
    torch.cuda.synchronize()
    assert bool((out[:-1] == 2).all()) and float(out[-1]) == 3.0
