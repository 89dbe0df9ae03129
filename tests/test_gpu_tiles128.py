"""GPU parity of the deeper nets' 128 x 128 tiles (deep.hip): ragged row counts, an odd
number of K chunks, a short last row chunk, and the batches around those that take them.
A copy of the library's rule says which products of a case run on them; each case
states it, so that a change of the rule cannot leave the tiles untested."""
import heapq

import numpy as np
import pytest
import torch

from tests.parity import rel
from tests.test_gpu_deep import D, _ctx, _gauss_net, _kink_free, _to, mlp  # noqa: F401


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


CUS, BT, K_MIN = 256, 128, 256


def _row_chunks(h, rows):
    """(rows per chunk, chunks) of dW_2's split over the batch rows."""
    tiles = (h // 64) ** 2
    splits = max(1, min(-(-(256 if h <= 256 else 512) // tiles), -(-rows // 64), 64))
    kc = -(-(-(-rows // splits)) // 32) * 32
    return kc, -(-rows // kc)


def _on_128(h, rows):
    """Whether the hidden forward product of `rows` rows, and the pair of dW_2 and its
    back-propagation, run on 128 x 128 tiles: h a multiple of 128 (and K at least 256),
    and the 256 compute units busy for three quarters of the time (the pair: seven
    eighths) if the tiles go out in order to whichever is free."""
    if h % BT or rows < BT:
        return False, False
    row_tiles, n = -(-rows // BT), h // BT
    rounds = -(-(row_tiles * n) // CUS)
    forward = h >= K_MIN and 4 * row_tiles * n >= 3 * rounds * CUS
    kc, splits = _row_chunks(h, rows)
    if min(kc, rows) < K_MIN or h < K_MIN:
        return forward, False
    done = [0] * CUS
    work = [min(kc, rows)] * (n * n * splits) + [h] * (row_tiles * n)
    for k in work:
        heapq.heappush(done, heapq.heappop(done) + k)
    return forward, 8 * sum(work) >= 7 * max(done) * CUS


# (h, layers, rows, forward and pair on 128 x 128 tiles, K chunks of dW_2's first and last
# row chunk). 3,967: a row tile of 127 rows; 4,000: one of 32; 4,093: a last K chunk of
# 29; 5,000: a last row chunk of 72; 4,097: one row in the last tile.
CASES = [(1024, 2, 2048, False, True, 32, 32), (1024, 2, 3967, True, True, 62, 62),
         (1024, 2, 4000, True, True, 63, 62), (1024, 2, 4097, False, False, 65, 64),
         (512, 3, 4093, False, True, 16, 16), (512, 2, 8192, True, True, 32, 32),
         (384, 2, 5000, False, True, 11, 3), (384, 2, 8192, True, False, 18, 4),
         (768, 2, 4097, True, False, 33, 30), (768, 3, 12003, False, True, 94, 94),
         (640, 2, 12000, True, True, 63, 60)]


@pytest.mark.parametrize("h,L,B,forward,pair,first,last", CASES, ids=lambda v: str(v))
def test_cases_take_the_tiles_they_are_for(h, L, B, forward, pair, first, last):
    assert _on_128(h, B) == (forward, pair)
    kc, chunks = _row_chunks(h, B)
    assert (kc // 32, -(-(B - (chunks - 1) * kc) // 32)) == (first, last)


@pytest.mark.gpu
@pytest.mark.parametrize("h,L,B", [c[:3] for c in CASES])
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
