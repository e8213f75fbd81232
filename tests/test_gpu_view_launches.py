"""GPU tests of the strided views' launch rules: one case on each side of every
line between element and vector tiles, wide and narrow ones, streaming and
ordinary loads, whole results against torch in FP64."""
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

DT = {"f32": "float32", "f64": "float64", "bf16": "bfloat16"}
ARITY = {"addsub2": 2, "addsub4": 4, "expr1": 2, "expr2": 4}


def _check(which, dtype, m, n):
    torch, fx = need_gpu()
    dt = getattr(torch, DT[dtype])
    dev, wide = [], []
    for q in range(ARITY[which]):
        g = torch.Generator(device="cuda").manual_seed(1000 * q + m)
        v = torch.rand(m * n, generator=g, device="cuda", dtype=torch.float64)
        v = (v + 1 if q == 3 else 2 * v - 1).to(dt)
        dev.append(v)
        wide.append(v.to(torch.float64).view(n, m))     # [column, row]
    rows, cols = fx.fx_paper_view_shape(which, (m, n))
    guard = 64
    buf = torch.full((rows * cols + 2 * guard,), 77.0, dtype=dt, device="cuda")
    Z = buf[guard:guard + rows * cols]
    fx.fx_paper_view_expr(which, dev, Z, (m, n), scalars=(1.5,))
    assert bool((buf[:guard] == 77).all()) and bool((buf[guard + rows * cols:] == 77).all())
    if which.startswith("addsub"):
        r, c = (m - rows) // 2, (n - cols) // 2
        cut = [w[c:c + cols, r:r + rows] for w in wide]
        want, mag, ops = sum(cut), sum(x.abs() for x in cut), len(cut) - 1
    elif which == "expr1":
        A, B = wide
        want = 2 * (A.T + B) + 2 * (A + B.T)
        mag, ops = 2 * (A.abs().T + B.abs() + A.abs() + B.abs().T), 5
    else:
        A, B, C, D = wide
        log = torch.log(D * D)
        want = 1.5 * A + (B + C).T + log
        # the logarithm of 1 .. 4: at most 3.25 units of its value, and its argument's rounding
        mag, ops = 1.5 * A.abs() + B.abs().T + C.abs().T + log.abs() + 1, 8
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    bound = ops * u * mag
    if dtype == "bf16":
        bound += 2.0 ** -8 * want.abs() + 2.0 ** -130
    assert bool(((Z.to(torch.float64).view(cols, rows) - want).abs() <= bound).all())


# element tiles up to 4 MB of the result, vectors from there on
@pytest.mark.parametrize("which", ["expr1", "expr2"])
@pytest.mark.parametrize("dtype,m", [("f32", 1024), ("f32", 1025), ("f64", 724), ("f64", 725),
                                     ("bf16", 1448), ("bf16", 1449), ("bf16", 1607)])
def test_small_results(which, dtype, m):
    _check(which, dtype, m, m)


# submatrices of 1 .. 8 and of 15 .. 17 columns, and of 32 and 33 rows
@pytest.mark.parametrize("which", ["addsub2", "addsub4"])
@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("shape", [(70001, 2), (65536, 4), (65536, 6), (8195, 16), (8192, 30), (8195, 34),
                                   (5, 4099), (64, 3001), (65, 3001), (66, 3001), (67, 30001)])
def test_narrow_and_short(which, dtype, shape):
    _check(which, dtype, *shape)


# ordinary and streaming loads, by size and by whether columns are whole cache
# lines; the wide tile of transposed parts
@pytest.mark.parametrize("which,dtype,m", [
    ("expr1", "f32", 3104), ("expr1", "f32", 5000), ("expr1", "f32", 5856), ("expr1", "f32", 7500),
    ("expr1", "f64", 3001), ("expr1", "f64", 4112), ("expr1", "bf16", 6700),
    ("expr2", "f32", 3104), ("expr2", "f32", 4112), ("expr2", "f32", 8192),
    ("expr2", "f64", 3001), ("expr2", "f64", 4096), ("expr2", "bf16", 5857)])
def test_large_results_with_transposed_parts(which, dtype, m):
    _check(which, dtype, m, m)


@pytest.mark.parametrize("which,dtype,shape", [
    ("addsub2", "f32", (4096, 4097)), ("addsub2", "f32", (8192, 4099)), ("addsub2", "f32", (8192, 8190)),
    ("addsub4", "f32", (4099, 4099)), ("addsub4", "f32", (8200, 8200)), ("addsub2", "bf16", (8192, 4098)),
    ("addsub4", "f64", (6003, 6001)), ("addsub2", "f64", (2048, 9000))])
def test_large_submatrices(which, dtype, shape):
    _check(which, dtype, *shape)
