"""GPU parity of the deeper nets' 128 x 128 tiles (deep.hip): ragged row counts, an odd
number of K chunks, a short last row chunk, and the batches around those that take them."""
import numpy as np
import pytest
import torch

from tests.parity import rel
from tests.test_gpu_deep import D, _ctx, _gauss_net, _kink_free, _to, mlp  # noqa: F401

pytestmark = pytest.mark.gpu


def _weights(P, h, L):
    P = P.astype(np.float64)
    Ws = [P[:D * h].reshape(D, h)]
    Ws += [P[D * h + l * h * h:D * h + (l + 1) * h * h].reshape(h, h) for l in range(L - 1)]
    return Ws, P[-h:]


def _grad(X, Y, P, h, L):
    """Gradient and loss of the batch in float64 (the oracle's plain loops take minutes here)."""
    Ws, wo = _weights(P, h, L)
    H = [X.astype(np.float64)]
    for W in Ws:
        H.append(np.maximum(H[-1] @ W, 0))
    r = H[-1] @ wo - Y
    g = 2.0 / len(r) * r
    out = [H[-1].T @ g]
    G = np.outer(g, wo) * (H[-1] > 0)
    for l in range(L - 1, -1, -1):
        out.insert(0, (H[l].T @ G).ravel())
        if l:
            G = (G @ Ws[l].T) * (H[l] > 0)
    return np.concatenate(out), float((r * r).mean()), H[-1] @ wo


# (384: nine 32-row chunks of K and a last one of two; 3,967: a row tile of 127 rows;
# 4,097: one row in the last tile, 64 x 64 tiles instead at h = 1024)
@pytest.mark.parametrize("h,L,B", [(1024, 2, 2048), (1024, 2, 3967), (1024, 2, 4097), (512, 3, 4093),
                                   (512, 2, 8192), (384, 2, 4096), (768, 3, 3333)])
def test_gradients_and_forward(mlp, h, L, B):  # noqa: F811
    """Inputs whose masks the device's rounding cannot change: 1e-5 (as the other
    kink-free gradients of this path). Two layers: rows far enough from every kink,
    repeated where they are few. Three, where hardly a row is: small whole numbers
    over powers of two, whose forward pass is exact (every sum below 2^24 units)."""
    rng = np.random.default_rng(h + L + B)
    n = 2 * B
    Y = rng.standard_normal(n).astype(np.float32)
    if L == 2:
        P = _gauss_net(rng, h, L)
        X = rng.standard_normal((n, D)).astype(np.float32)
        idx = _kink_free(X, P, h, L, np.arange(n))
        idx = rng.permutation(np.resize(idx, B))
    else:
        W = [rng.integers(-1, 2, size=s) for s in [(D, h)] + [(h, h)] * (L - 1) + [(h, 1)]]
        Z = rng.integers(-1, 2, size=(n, D))
        X = (Z / 2).astype(np.float32)
        P = np.concatenate([w.ravel() / 16 for w in W]).astype(np.float32)
        for w in W:
            w = w.astype(np.float64)
            assert (np.abs(Z) @ np.abs(w)).max() < 2 ** 24
            Z = np.maximum(Z @ w, 0)
        idx = rng.permutation(n)[:B]
    idx = np.ascontiguousarray(idx.astype(np.int32))
    ctx, _ = _ctx(mlp, P, h, L, B)
    dP, loss = mlp.mlp_deep_backward(ctx, _to(X), _to(Y), _to(idx))
    out = torch.full((B + 40,), 7.0, device="cuda")   # words past B stay untouched
    mlp.mlp_deep_forward(ctx, _to(X), _to(idx), B=B, out=out)
    mlp.mlp_deep_check_errors(ctx)
    ref, rl, y = _grad(X[idx], Y[idx], P, h, L)
    got, o = dP.cpu().numpy(), 0
    for size in [D * h] + [h * h] * (L - 1) + [h]:   # every weight matrix by itself
        assert rel(got[o:o + size], ref[o:o + size]) <= 1e-5
        o += size
    assert abs(float(loss.cpu()[0]) - rl) <= 1e-5 * rl
    yp = out.cpu().numpy()
    assert rel(yp[:B], y) < 1e-5 and np.all(yp[B:] == 7.0)
