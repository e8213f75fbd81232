"""GPU tests of the cost model's kernels over the shapes where their layout
changes: one to four rows per block, weights staged in LDS or read in place,
batches around the 256-row chunk of the gradient sums, tile remainders.  The
reference is numpy in float64."""
import numpy as np
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _case(F, H, heads, B, seed):
    rng = np.random.default_rng(seed)
    C = sum(heads)
    W1 = (rng.uniform(-1, 1, (H, F)) / np.sqrt(F)).astype(np.float32)
    b1 = rng.uniform(-0.5, 0.5, H).astype(np.float32)
    W2 = (rng.uniform(-1, 1, (C, H)) / np.sqrt(H)).astype(np.float32)
    b2 = rng.uniform(-0.5, 0.5, C).astype(np.float32)
    mean = rng.normal(size=F).astype(np.float32)
    std = rng.uniform(0.5, 2, F).astype(np.float32)
    X = (rng.normal(size=(2 * B + 64, F)) * 2 + 1).astype(np.float32)
    pre = ((X.astype(np.float64) - mean) / std) @ W1.T.astype(np.float64) + b1
    X = X[np.abs(pre).min(axis=1) > 1e-5][:B]   # no hidden unit at the edge of its ReLU
    assert len(X) == B
    y = np.stack([rng.integers(0, k, B) for k in heads], axis=1).astype(np.int32)
    return (W1, b1, W2, b2), mean, std, X, y


def _reference(params, mean, std, X, y, heads):
    """logits, loss and gradient in float64, and the magnitudes that bound the
    rounding errors of the FP32 logits and gradient."""
    W1, b1, W2, b2 = [p.astype(np.float64) for p in params]
    B = len(X)
    xn = (X.astype(np.float64) - mean) / std
    pre = xn @ W1.T + b1
    h = np.maximum(pre, 0)
    logits = h @ W2.T + b2
    hm = np.abs(xn) @ np.abs(W1).T + np.abs(b1)
    lm = hm @ np.abs(W2).T + np.abs(b2)
    dl, loss, o = np.zeros_like(logits), 0.0, 0
    for q, k in enumerate(heads):
        z = logits[:, o:o + k]
        e = np.exp(z - z.max(axis=1, keepdims=True))
        p = e / e.sum(axis=1, keepdims=True)
        loss -= np.mean(np.log(p[np.arange(B), y[:, q]]))
        p[np.arange(B), y[:, q]] -= 1
        dl[:, o:o + k] = p / B
        o += k
    dh = (dl @ W2) * (pre > 0)
    g = np.concatenate([(dh.T @ xn).ravel(), dh.sum(0), (dl.T @ h).ravel(), dl.sum(0)])
    # a dlogit is (softmax - 0/1) / B, at most 1 / B, and moves by at most the
    # logits' error over B
    dlm = np.full_like(dl, 1.0 / B) * (1 + lm.max())
    dhm = dlm @ np.abs(W2)
    gm = np.concatenate([(dhm.T @ np.abs(xn)).ravel(), dhm.sum(0), (dlm.T @ hm).ravel(), dlm.sum(0)])
    return logits, lm, loss, g, gm


@pytest.mark.parametrize("F,H,heads,B", [
    (1, 1, (2,), 1), (25, 64, (4, 3, 3, 4), 255), (25, 64, (4, 3, 3, 4), 257),
    (26, 65, (2, 5), 513), (7, 200, (3,), 256), (64, 256, (32, 32), 70)])
def test_shapes(F, H, heads, B):
    torch, fx = need_gpu()
    params, mean, std, X, y = _case(F, H, heads, B, 17)
    logits, lm, loss, g, gm = _reference(params, mean, std, X, y, heads)
    m = fx.Model(F, H, heads)
    m.set(np.concatenate([p.ravel() for p in params]), mean, std)
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    out = torch.full((B, sum(heads)), np.nan, device="cuda")
    choice = torch.full((B, len(heads)), -1, dtype=torch.int32, device="cuda")
    m.forward(Xd, out, choice)
    grad = torch.full((m.n_params,), np.nan, device="cuda")
    ls = torch.full((1,), np.nan, device="cuda")
    m.grad(Xd, yd, grad, ls)
    torch.cuda.synchronize()
    # one rounding per operation of each chain; 16 covers the subtraction and
    # division that standardise, expf, logf and the softmax's own operations
    chain = F + H + sum(heads) + 16
    assert (np.abs(out.cpu().numpy() - logits) <= chain * U * lm).all()
    assert (np.abs(grad.cpu().numpy() - g) <= (2 * chain + B) * U * gm).all()
    assert abs(ls.item() - loss) <= (2 * chain + B) * U * len(heads) * (1 + lm.max())
    for b in sorted({0, B // 2, B - 1}):          # the host twin decides identically
        assert m.choose(X[b]) == list(choice[b].cpu().numpy())


def test_train_equals_stepping_on_a_ragged_epoch():
    """An epoch whose last batch is short, visited in a given order: the same
    bits as gathering the rows and stepping."""
    torch, fx = need_gpu()
    F, H, heads, n, batch = 25, 64, (4, 3, 3, 4), 601, 256
    params, mean, std, X, y = _case(F, H, heads, n, 18)
    flat = np.concatenate([p.ravel() for p in params])
    perm = np.random.default_rng(3).permutation(n).astype(np.int32)
    got = []
    for whole in (True, False):
        m = fx.Model(F, H, heads)
        m.set(flat, mean, std)
        Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
        if whole:
            m.train(Xd, yd, 1, batch, 1e-2, perm[None])
        else:
            for s in range(0, n, batch):
                rows = torch.from_numpy(perm[s:s + batch].astype(np.int64)).cuda()
                xb, yb = Xd[rows].contiguous(), yd[rows].contiguous()
                m.train_step(xb, yb, 1e-2)
                torch.cuda.synchronize()
        got.append(m.get()[0])
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("F,H,heads,line", [(25, 64, (4, 3, 3, 4), 4096), (64, 256, (32, 32), 1024),
                                            (25, 200, (3, 60), 4096)])
def test_forward_at_its_lines(F, H, heads, line):
    """Both sides of the batch from which rows share a block: within the bound,
    and the same bits as the rows alone."""
    torch, fx = need_gpu()
    params, mean, std, X, y = _case(F, H, heads, line + 1, 19)
    logits, lm, _, _, _ = _reference(params, mean, std, X, y, heads)
    m = fx.Model(F, H, heads)
    m.set(np.concatenate([p.ravel() for p in params]), mean, std)
    Xd = torch.from_numpy(X).cuda()
    alone = torch.full((8, sum(heads)), np.nan, device="cuda")
    for B in (line, line + 1):
        out = torch.full((B, sum(heads)), np.nan, device="cuda")
        choice = torch.full((B, len(heads)), -1, dtype=torch.int32, device="cuda")
        m.forward(Xd[:B], out, choice)
        torch.cuda.synchronize()
        chain = F + H + sum(heads) + 16
        assert (np.abs(out.cpu().numpy() - logits[:B]) <= chain * U * lm[:B]).all()
        for s in (0, B - 8):
            m.forward(Xd[s:s + 8].contiguous(), alone)
            torch.cuda.synchronize()
            assert torch.equal(alone, out[s:s + 8])
        for b in (0, B - 1):
            assert m.choose(X[b]) == list(choice[b].cpu().numpy())
