"""GPU tests of the strided views at the sizes where their tiles, vectors and
paired tiles can go wrong, against numpy in FP64: a few rows, remainders of the
vector and of every tile side, odd leading dimensions, misaligned buffers, an
output that is an input read in place, and neighbours of the output that must
stay untouched."""
import numpy as np
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

U = {"f32": 2.0 ** -24, "f64": 2.0 ** -53, "bf16": 2.0 ** -24}
PAD = 16


def _matrices(torch, m, n, dtype, shift):
    g = torch.Generator().manual_seed(m * 1009 + n)
    dt = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16}[dtype]
    dev, host = [], []
    for q in range(4):
        v = torch.rand(m * n, generator=g, dtype=torch.float64)
        v = (v + 1 if q == 3 else 2 * v - 1).to(dt)
        buf = torch.zeros(m * n + 2 * PAD, dtype=dt, device="cuda")
        at = buf[PAD + shift * (q + 1) % 7:][:m * n]
        at.copy_(v)
        dev.append(at)
        host.append(v.to(torch.float64).numpy().reshape(n, m).T)   # rows, columns
    return dev, host, dt


def _want(which, host, m, n):
    A, B, C, D = host
    h, w = m // 2, n // 2
    r, c = (m - h) // 2, (n - w) // 2
    cut = [M[r:r + h, c:c + w] for M in host]
    if which == "addsub2":
        return cut[0] + cut[1], np.abs(cut[0]) + np.abs(cut[1]), 1
    if which == "addsub4":
        return sum(cut), sum(np.abs(x) for x in cut), 3
    if which == "expr1":
        return 2 * (A.T + B) + 2 * (A + B.T), 2 * (abs(A.T) + abs(B) + abs(A) + abs(B.T)), 5
    # the logarithm of 1 .. 4: at most 3.25 units of its value, and its argument's rounding
    return (1.5 * A + (B + C).T + np.log(D * D),
            1.5 * abs(A) + abs(B.T) + abs(C.T) + abs(np.log(D * D)) + 1, 8)


@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("m", [1, 2, 3, 7, 9, 31, 33, 63, 65, 127, 129, 131, 257, 514])
def test_square_views(dtype, m):
    torch, fx = need_gpu()
    for shift in (0, 1):
        dev, host, dt = _matrices(torch, m, m, dtype, shift)
        for which, k in (("addsub2", 2), ("addsub4", 4), ("expr1", 2), ("expr2", 4)):
            rows, cols = fx.fx_paper_view_shape(which, (m, m))
            nz = rows * cols
            buf = torch.full((nz + 2 * PAD,), 77.0, dtype=dt, device="cuda")
            Z = buf[PAD + shift:PAD + shift + nz]
            fx.fx_paper_view_expr(which, dev[:k], Z, (m, m), scalars=(1.5,))
            torch.cuda.synchronize()
            assert (buf[:PAD + shift] == 77).all() and (buf[PAD + shift + nz:] == 77).all()
            if nz == 0:
                continue
            got = Z.to(torch.float64).cpu().numpy().reshape(cols, rows).T
            want, mag, ops = _want(which, host, m, m)
            bound = ops * U[dtype] * mag + (2.0 ** -8 * np.abs(want) + 2.0 ** -130 if dtype == "bf16" else 0)
            assert (np.abs(got - want) <= bound).all(), (which, m, shift, np.abs(got - want).max())


@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("shape", [(5, 300), (300, 5), (18, 37), (259, 34), (1030, 70)])
def test_rectangular_submatrices(dtype, shape):
    torch, fx = need_gpu()
    m, n = shape
    dev, host, dt = _matrices(torch, m, n, dtype, 1)
    for which, k in (("addsub2", 2), ("addsub4", 4)):
        rows, cols = fx.fx_paper_view_shape(which, shape)
        Z = torch.empty(rows * cols, dtype=dt, device="cuda")
        fx.fx_paper_view_expr(which, dev[:k], Z, shape)
        torch.cuda.synchronize()
        got = Z.to(torch.float64).cpu().numpy().reshape(cols, rows).T
        want, mag, ops = _want(which, host, m, n)
        bound = ops * U[dtype] * mag + (2.0 ** -8 * np.abs(want) if dtype == "bf16" else 0)
        assert (np.abs(got - want) <= bound).all(), (which, shape)


@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("m", [5, 66, 131, 1027])
def test_in_place(dtype, m):
    """expr2 into its A, and into its D: the rows two threads' vectors share
    are read before their owner writes them, or not used."""
    torch, fx = need_gpu()
    for q in (0, 3):
        dev, host, dt = _matrices(torch, m, m, dtype, 0)
        ref = torch.empty_like(dev[0])
        fx.fx_paper_view_expr("expr2", dev, ref, (m, m), scalars=(1.5,))
        fx.fx_paper_view_expr("expr2", dev, dev[q], (m, m), scalars=(1.5,))
        torch.cuda.synchronize()
        assert torch.equal(dev[q], ref), (q, m)
