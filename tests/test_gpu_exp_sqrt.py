"""GPU tests of the FP32 exp and sqrt where their common range ends: the values
at both sides of each limit, zeros, infinities and NaNs, alone and as one odd
lane among ordinary ones, through the compiled, tape and unfused paths.  An
element's value must not depend on its neighbours."""
import numpy as np
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _edge_values():
    f = np.float32
    v = [0.0, -0.0, 1.0, 87.0, np.nextafter(f(87), f(88)), 88.7, 88.73, 89.0, 103.9, 104.1, 1e30, np.inf,
         np.nan, 2.0 ** -96, np.nextafter(f(2.0 ** -96), f(0)), 2.0 ** -126, 2.0 ** -149, 2.0 ** -100,
         3.4028235e38, 4.0, 2.0, 3.0]
    v = np.array(v, np.float32)
    return np.concatenate([v, -v])


def _vectors():
    """Each edge value alone in a run of 512 ordinary ones, at changing lanes."""
    e = _edge_values()
    x = np.random.default_rng(9).uniform(0.01, 2, 512 * len(e)).astype(np.float32)
    x[np.arange(len(e)) * 512 + np.arange(len(e)) * 5 % 512] = e
    return np.concatenate([x, e, x[:13]])


NABS = [("leaf", -1, -1, 0, 0), ("abs", 0, -1, -1, 0), ("neg", 1, -1, -1, 0), ("exp", 2, -1, -1, 0)]
SABS = [("leaf", -1, -1, 0, 0), ("abs", 0, -1, -1, 0), ("sqrt", 1, -1, -1, 0)]
EXP = [("leaf", -1, -1, 0, 0), ("exp", 0, -1, -1, 0)]
SQRT = [("leaf", -1, -1, 0, 0), ("sqrt", 0, -1, -1, 0)]


@pytest.mark.parametrize("op", ["exp", "sqrt", "exp_nabs", "sqrt_abs"])
def test_edges(op):
    torch, fx = need_gpu()
    x = _vectors()
    w = x.astype(np.float64)
    with np.errstate(all="ignore"):
        want = {"exp": np.exp(w), "sqrt": np.sqrt(w), "exp_nabs": np.exp(-np.abs(w)),
                "sqrt_abs": np.sqrt(np.abs(w))}[op]
        rounded = want.astype(np.float32).astype(np.float64)
    X = torch.from_numpy(x).cuda()
    n = len(x)
    outs = []
    tape = fx.Tape({"exp": EXP, "sqrt": SQRT, "exp_nabs": NABS, "sqrt_abs": SABS}[op])
    for cfg in (None, (64, 1, 16, 0), (64, 1, 4, 0), (256, 4, 16, 0)):
        Z = torch.empty_like(X)
        fx.fx_tape_eval(tape, [X], Z, (n, 1), cfg=cfg)
        outs.append(Z)
    if op in ("exp", "sqrt"):
        for cfg in (None, (64, 1, 4, 0)):
            Z = torch.empty_like(X)
            fx.fx_op_unary(op, X, Z, cfg)
            outs.append(Z)
    torch.cuda.synchronize()
    ref = outs[0].cpu().numpy()
    for Z in outs[1:]:
        assert np.array_equal(ref.view(np.uint32)[~np.isnan(ref)],
                              Z.cpu().numpy().view(np.uint32)[~np.isnan(ref)])
        assert np.array_equal(np.isnan(ref), np.isnan(Z.cpu().numpy()))
    got = ref.astype(np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = ~np.isnan(want)
    if "sqrt" in op:
        assert np.array_equal(got[ok], rounded[ok])          # correctly rounded
        assert np.array_equal(np.signbit(got[ok]), np.signbit(rounded[ok]))
    else:
        fin = ok & np.isfinite(rounded)
        assert np.array_equal(np.isinf(got[ok]), np.isinf(rounded[ok]))
        assert (np.abs(got[fin] - want[fin]) <= 1.5 * U * want[fin] + 2.0 ** -149).all()


def test_fused_neighbours():
    """C2's exp(-|W|) with one infinite W per vector run: the ordinary elements
    keep the bits they have without it."""
    torch, fx = need_gpu()
    n = 4099
    g = torch.Generator(device="cuda").manual_seed(4)
    X, Y, W = (torch.rand(n, generator=g, device="cuda") * 2 - 1 for _ in range(3))
    Z0, Z1 = torch.empty_like(X), torch.empty_like(X)
    fx.fx_c2_z(X, Y, W, Z0, (n, 1))
    odd = torch.arange(5, n, 67, device="cuda")
    W[odd] = float("inf")
    fx.fx_c2_z(X, Y, W, Z1, (n, 1))
    torch.cuda.synchronize()
    keep = torch.ones(n, dtype=torch.bool, device="cuda")
    keep[odd] = False
    assert torch.equal(Z0[keep], Z1[keep])
    assert (Z1[odd] == 0).all()
