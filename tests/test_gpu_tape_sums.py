"""GPU tests of the launch that a tape's full reduction takes by default: sizes at
both sides of its lines (one block, small blocks, two blocks per CU), repeated on
one workspace, against FP64 sums; and what needs a workspace."""
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

NODES = [("leaf", -1, -1, 0, 0.0), ("neg", 0, -1, -1, 0.0)]


@pytest.mark.parametrize("dtype", ["float32", "float64", "bfloat16"])
@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 4096, 4097, (1 << 17) - 1, 1 << 17, (1 << 21) + 3])
def test_lines(dtype, n):
    torch, fx = need_gpu()
    g = torch.Generator(device="cuda").manual_seed(5)
    x = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 2 - 1).to(getattr(torch, dtype))
    w = x.to(torch.float64)
    tape = fx.Tape(NODES)
    for kind, want, scale in ((fx.R_ACCU, -w.sum(), w.abs().sum()), (fx.R_NORM, w.square().sum().sqrt(), w.norm())):
        ws = fx.workspace(kind, fx.dtype_code(x), (n, 1))
        out = torch.zeros(1, dtype=torch.float64, device="cuda")
        # sums in FP64 on both sides; squares of FP32 are rounded to it first
        tol = float(scale) * ((n + 8) * 2.0 ** -53 + (2.0 ** -24 if kind == fx.R_NORM and dtype != "float64" else 0))
        for _ in range(3):
            out.fill_(float("nan"))
            fx.fx_tape_eval(tape, [x], out, (n, 1), kind, ws)
            torch.cuda.synchronize()
            assert abs(float(out) - float(want)) <= tol
        with pytest.raises(fx.FxError) as e:
            fx.fx_tape_eval(tape, [x], out, (n, 1), kind)
        assert e.value.code == 4  # FX_E_WORKSPACE


@pytest.mark.parametrize("n,needed", [(2048, False), (2049, True), (8192, True)])
def test_compiled_sum_needs_workspace(n, needed):
    torch, fx = need_gpu()
    x = torch.ones(n, device="cuda")
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    if needed:
        with pytest.raises(fx.FxError) as e:
            fx.fx_accu_xy(x, x, out, None)
        assert e.value.code == 4  # FX_E_WORKSPACE
    else:
        fx.fx_accu_xy(x, x, out, None)
    fx.fx_accu_xy(x, x, out, fx.workspace(fx.R_ACCU, fx.F32, (n, 1)))
    torch.cuda.synchronize()
    assert float(out) == n
