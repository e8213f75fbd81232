"""GPU tests of the dimension sums at both sides of their launch rules' lines,
against FP64 sums."""
import pytest

from gpu_util import need_gpu

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
