"""GPU tests of the column sums' launch over column lengths and counts: at both
sides of the lines between one thread, one wave and more threads per column, and
between whole and chunked columns, against FP64 sums."""
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

NODES = [("leaf", -1, -1, 0, 0.0), ("leaf", -1, -1, 1, 0.0), ("mul", 0, 1, -1, 0.0)]
ROWS = [8, 9, 16, 17, 32, 33, 64, 255, 256, 257, 513, 1025, 2049, 4097]


@pytest.mark.parametrize("dtype", ["float32", "float64", "bfloat16"])
@pytest.mark.parametrize("cols", [1, 5, 63, 64, 255, 256, 513, 1024])
def test_lines(dtype, cols):
    torch, fx = need_gpu()
    tape = fx.Tape(NODES)
    for rows in ROWS + ([300001] if cols <= 5 else []):
        n = rows * cols
        g = torch.Generator(device="cuda").manual_seed(rows)
        x, y = ((torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 2 - 1).to(getattr(torch, dtype))
                for _ in range(2))
        terms = (x.to(torch.float64) * y.to(torch.float64)).view(cols, rows)
        want, scale = terms.sum(1), terms.abs().sum(1)
        acc = torch.float64 if dtype == "float64" else torch.float32
        ws = fx.workspace(fx.R_COLSUM, fx.dtype_code(x), (rows, cols))
        # terms rounded to the compute type, FP64 sums, one rounding to the output
        u = 2.0 ** -53 * (rows + 8) if dtype == "float64" else 2.0 ** -24
        for run in (lambda o: fx.fx_colsum_xy(x, y, o, (rows, cols), ws),
                    lambda o: fx.fx_tape_eval(tape, [x, y], o, (rows, cols), fx.R_COLSUM, ws)):
            for _ in range(2):
                out = torch.full((cols,), float("nan"), dtype=acc, device="cuda")
                run(out)
                torch.cuda.synchronize()
                err = (out.to(torch.float64) - want).abs()
                assert bool((err <= 2.01 * u * scale).all()), (rows, float((err / scale).max()))
