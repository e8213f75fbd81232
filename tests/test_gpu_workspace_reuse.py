"""GPU tests of one workspace used by calls of other kinds and shapes, one after
another: every call leaves it zeroed, and its result is that of a fresh one."""
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

NODES = [("leaf", -1, -1, 0, 0.0), ("leaf", -1, -1, 1, 0.0), ("mul", 0, 1, -1, 0.0)]
# (kind, rows, cols): few and many counters, before and after few and many partials
CALLS = [("R_ACCU", 1 << 20, 1), ("R_COLSUM", 65536, 128), ("R_ROWSUM", 16384, 300), ("R_NORM", 3000, 1111),
         ("R_ROWSUM", 600, 5000), ("R_COLSUM", 1 << 20, 3), ("R_ROWSUM", 30000, 100), ("R_ACCU", 1 << 24, 1),
         ("R_COLSUM", 20000, 255), ("R_ROWSUM", 20000, 640)]


@pytest.mark.parametrize("dtype", ["float32", "float64", "bfloat16"])
@pytest.mark.parametrize("mode", ["compiled", "tape", "rtc", "static"])
def test_one_workspace_for_all(dtype, mode):
    torch, fx = need_gpu()
    tape = fx.Tape(NODES)
    dt = getattr(torch, dtype)
    g = torch.Generator(device="cuda").manual_seed(5)
    x, y = ((torch.rand(1 << 24, generator=g, device="cuda", dtype=torch.float64) * 2 - 1).to(dt) for _ in range(2))
    code = fx.dtype_code(x)
    shared = torch.zeros(1 << 24, dtype=torch.uint8, device="cuda")
    for name, rows, cols in CALLS:
        kind, n = getattr(fx, name), rows * cols
        ins = [x[:n], y[:n]]
        if mode == "compiled":
            call = {"R_ACCU": lambda o, w: fx.fx_accu_xy(*ins, o, w),
                    "R_NORM": lambda o, w: fx.fx_norm_fro_diff(*ins, o, (rows, cols), w),
                    "R_COLSUM": lambda o, w: fx.fx_colsum_xy(*ins, o, (rows, cols), w),
                    "R_ROWSUM": lambda o, w: fx.fx_c2_rowsum(*ins, ins[0], o, (rows, cols), w)}[name]
        elif mode == "rtc":
            rtc = fx.Rtc(NODES, code, kind)
            call = lambda o, w: rtc.eval(ins, o, (rows, cols), w)
        else:
            call = lambda o, w: fx.fx_tape_eval(tape, ins, o, (rows, cols), kind, w)
        full = name in ("R_ACCU", "R_NORM")
        acc = torch.float64 if full or dtype == "float64" else torch.float32
        size = 1 if full else cols if name == "R_COLSUM" else rows
        got, want = (torch.full((size,), float("nan"), dtype=acc, device="cuda") for _ in range(2))
        call(want, fx.workspace(kind, code, (rows, cols)))
        if mode == "static":
            fx.fx_tape_eval_static(tape, ins, got, (rows, cols), kind)
        else:
            call(got, shared)
        torch.cuda.synchronize()
        assert torch.equal(got, want), (name, rows, cols)
        assert int(shared.count_nonzero()) == 0, (name, rows, cols)
