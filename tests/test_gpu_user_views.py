"""View expressions of a user's own program (tests/native/user_views.hip), which
no entry point instantiates: matrices read both directly and transposed whose
storage is not the output's, and five transposed parts, against numpy in FP64."""
import ctypes
import os

import numpy as np
import pytest

from gpu_util import need_gpu

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "native", "user_views.hip")
LIB = os.path.join(HERE, "native", "libuser_views.so")


def _lib():
    import paper_2604_22242_amd as fx
    from paper_2604_22242_amd import build
    if not os.path.exists(fx.LIB_PATH):
        build.build()
    if not os.path.exists(LIB):
        build.build_user(SRC, LIB)
    fx.lib()
    return ctypes.CDLL(LIB)


def _call(torch, name, z, ins, n):
    L = _lib()
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    args = [ctypes.c_void_p(t.data_ptr()) for t in (z, *ins)]
    assert getattr(L, name)(*args, ctypes.c_int64(n), st) == 0


def _matrix(torch, seed, n, dt):
    g = torch.Generator().manual_seed(seed)
    v = (torch.rand(n * n, generator=g, dtype=torch.float64) * 2 - 1).to(dt)
    return v.cuda(), v.to(torch.float64).numpy().reshape(n, n).T     # rows, columns


def test_program_builds():
    L = _lib()
    assert all(hasattr(L, f) for f in ("user_pair_bf16_of_f32", "user_pair_f32_of_bf16",
                                       "user_pair_f16_of_bf16", "user_five_f32", "user_five_f64"))


def test_pairs_only_of_the_outputs_storage(tmp_path):
    """The paired kernel reads its matrices as the output's storage type: an
    expression with a leaf of another one must not be taken for it."""
    import subprocess
    from paper_2604_22242_amd import build
    src = tmp_path / "pairs.hip"
    src.write_text(
        '#include "fx_views.hpp"\nusing namespace fx;\n'
        "template <class TZ, class T> constexpr bool taken() {\n"
        "  return pairable<decltype(2 * (t(Leaf<T>{}) + Leaf<T>{})), TZ>::value;\n}\n"
        "static_assert(taken<float, float>() && taken<double, double>() && taken<bf16_t, bf16_t>());\n"
        "static_assert(!taken<bf16_t, float>() && !taken<float, bf16_t>() && !taken<f16_t, bf16_t>());\n"
        "static_assert(!pairable<decltype(t(Leaf<float>{}) + Leaf<bf16_t>{}), float>::value);\n")
    subprocess.check_call([build.HIPCC] + build.CFLAGS + ["-fsyntax-only", str(src)])


@pytest.mark.gpu
@pytest.mark.parametrize("out,store", [("bf16", "f32"), ("f32", "bf16"), ("f16", "bf16")])
def test_mixed_storage_pairs(out, store):
    torch, _ = need_gpu()
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
    for n in (7, 64, 131, 514, 1601):
        x, X = _matrix(torch, n, n, dt[store])
        y, Y = _matrix(torch, n + 1, n, dt[store])
        z = torch.full((n * n,), float("nan"), dtype=dt[out], device="cuda")
        _call(torch, "user_pair_%s_of_%s" % (out, store), z, (x, y), n)
        torch.cuda.synchronize()
        got = z.to(torch.float64).cpu().numpy().reshape(n, n).T
        want = 2 * (X.T + Y) + (X + Y.T)
        mag = 2 * (abs(X.T) + abs(Y)) + abs(X) + abs(Y.T)
        # three FP32 additions (the product by 2 is exact), one rounding to the
        # output: half its unit in the last place, or half its smallest step
        u, step = torch.finfo(dt[out]).eps / 2, 2.0 ** -25 if out == "f16" else 0.0
        bound = 3.01 * 2.0 ** -24 * mag + 1.01 * u * abs(want) + step
        assert (abs(got - want) <= bound).all(), (n, abs(got - want).max())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [3, 33, 130, 2048])
def test_five_transposed_parts(dtype, n):
    torch, _ = need_gpu()
    dt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    dev, host = zip(*(_matrix(torch, 100 * n + q, n, dt) for q in range(6)))
    z = torch.full((n * n,), float("nan"), dtype=dt, device="cuda")
    ptrs = (ctypes.c_void_p * 6)(*[t.data_ptr() for t in dev])
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert getattr(_lib(), "user_five_" + dtype)(ctypes.c_void_p(z.data_ptr()), ptrs, ctypes.c_int64(n), st) == 0
    torch.cuda.synchronize()
    got = z.to(torch.float64).cpu().numpy().reshape(n, n).T
    X = host[0]
    want = 2 * X + sum(M.T * X for M in host[1:])
    mag = 2 * abs(X) + sum(abs(M.T * X) for M in host[1:])
    # five products and five additions, the reference's own in FP64
    u = torch.finfo(dt).eps / 2 + (2.0 ** -53 if dtype == "f64" else 0)
    assert (abs(got - want) <= 10.01 * u * mag).all(), (n, abs(got - want).max())
