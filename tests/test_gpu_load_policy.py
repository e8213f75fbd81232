"""GPU tests of the element-wise kernel's load policy: ordinary loads while the
inputs and the output together fit the 256 MiB last-level cache, streaming loads
beyond.  Results at both sides of the line equal, bit for bit, those of the same
call made in pieces, also after the inputs have changed and with the output in
place of an input."""
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

LINE = 256 << 20


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
@pytest.mark.parametrize("repeat", [False, True])
@pytest.mark.parametrize("beyond", [0, 1, 4099])
def test_both_sides(dtype, repeat, beyond):
    torch, fx = need_gpu()
    dt = getattr(torch, dtype)
    arrays = 3 if repeat else 4  # distinct inputs and the output
    n = LINE // (arrays * dt.itemsize) + beyond
    g = torch.Generator(device="cuda").manual_seed(3)
    X, Y, W = ((torch.rand(n, generator=g, device="cuda") * 2 - 1).to(dt) for _ in range(3))
    if repeat:
        Y = X
    Z, P = torch.empty_like(X), torch.empty_like(X)
    piece = n // 5 // 8 * 8
    for _ in range(2):
        fx.fx_c1_z(X, Y, W, Z)
        for a in range(0, n, piece):
            fx.fx_c1_z(X[a:a + piece], Y[a:a + piece], W[a:a + piece], P[a:a + piece])
        torch.cuda.synchronize()
        assert torch.equal(Z, P)
        X.mul_(-0.5)  # the next pass must see the new values
    fx.fx_c1_z(X, Y, W, Z)
    fx.fx_c1_z(X, Y, W, W)  # in place
    torch.cuda.synchronize()
    assert torch.equal(Z, W)
