"""The binding enqueues on torch's current stream: the default one, a stream
entered as a context, and back, on whichever is current at the call."""
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def test_calls_follow_the_current_stream():
    torch, fx = need_gpu()
    assert fx._stream(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    n = 1 << 20
    x = torch.rand(n, device="cuda")
    z = torch.empty_like(x)
    with torch.cuda.stream(side):
        assert fx._stream(None) == side.cuda_stream
        side.wait_stream(torch.cuda.default_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):      # captured only if enqueued on `side`
            fx.fx_c1_z(x, x, x, z)
    assert fx._stream(None) == torch.cuda.current_stream().cuda_stream
    for k in range(3):
        x.fill_(float(k))
        z.fill_(-1.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert (z == k * k + 2 * k).all()
    assert fx._stream(side) == side.cuda_stream and fx._stream(0) == 0
