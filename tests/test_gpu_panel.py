"""GPU parity of the panel path of the deeper nets (widths up to 256, deep_panel.hip)
at the edges of its panels (16, 32 and 64 rows), row chunks (256) and panel choice,
and of the GEMM launches a smaller workspace falls back to."""
import numpy as np
import pytest
import torch

import datagen
import oracle
from tests.parity import rel
from tests.test_gpu_deep import D, _ctx, _dyadic, _gauss_net, _kink_free, _to, _train, mlp  # noqa: F401

pytestmark = pytest.mark.gpu


def _panel_pays(h, L, rows):
    """A copy of the library's rule: whether a step of `rows` rows runs as panels."""
    if L == 1:
        return rows <= 64 or (h >= 128 and 2048 <= rows <= 8192)
    if L == 2:
        return rows >= (4096 if h == 64 else 512)
    return h <= 192 or rows >= 256


EDGES = [(64, 4, b) for b in (17, 255, 257, 513, 4097, 8193)]
EDGES += [(192, 3, b) for b in (17, 255, 257, 513, 4097, 8193)]
EDGES += [(256, 3, b) for b in (256, 257, 513, 4095)]
EDGES += [(h, 2, b) for h in (128, 256) for b in (512, 513, 769, 4096, 4097, 8192, 8193)]
EDGES += [(64, 2, b) for b in (4096, 4097, 8193)]
EDGES += [(256, 1, b) for b in (17, 64, 2048, 2049, 4097, 8192)] + [(128, 1, 33), (64, 1, 63)]


@pytest.mark.parametrize("h,L,B", EDGES)
def test_gradients_at_panel_edges(mlp, h, L, B):  # noqa: F811
    """Rows whose masks the device's rounding cannot change, repeated where a deep net
    has few: 1e-5 (as the other kink-free gradients of this path). Panels of 16 rows up
    to 4,096, of 32 up to 8,192, then of 64 (one round of 256 workgroups)."""
    assert _panel_pays(h, L, B)
    rng = np.random.default_rng(h + L + B)
    P = _gauss_net(rng, h, L)
    d = datagen.make_data(3 * B, 32, seed=900 + h + B, with_perm=False)
    idx = _kink_free(d.X, P, h, L, np.arange(3 * B))
    assert len(idx) > 0
    idx = np.ascontiguousarray(rng.permutation(np.resize(idx, B)).astype(np.int32))
    ctx, _ = _ctx(mlp, P, h, L, B)
    dP, loss = mlp.mlp_deep_backward(ctx, _to(d.X), _to(d.Y), _to(idx))
    mlp.mlp_deep_check_errors(ctx)
    ref, rl = oracle.deep_grad(d.X, d.Y, P, D, h, L, idx=idx)[:2]
    assert rel(dP.cpu().numpy(), ref) <= 1e-5
    assert abs(float(loss.cpu()[0]) - rl) <= 1e-5 * rl


@pytest.mark.parametrize("h,L", [(64, 3), (192, 2), (256, 2)])
@pytest.mark.parametrize("B", [1, 16, 4097, 8193, 20000])
def test_forward_at_panel_edges(mlp, h, L, B):  # noqa: F811
    rng = np.random.default_rng(h + B)
    P = _gauss_net(rng, h, L)
    X = rng.standard_normal((2000, D)).astype(np.float32)
    idx = rng.integers(0, 2000, size=B).astype(np.int32)
    ctx, _ = _ctx(mlp, P, h, L, 64)
    out = torch.full((B + 70,), 7.0, device="cuda")   # words past B stay untouched
    mlp.mlp_deep_forward(ctx, _to(X), _to(idx), B=B, out=out)
    mlp.mlp_deep_check_errors(ctx)
    got = out.cpu().numpy()
    assert rel(got[:B], oracle.deep_forward(X, P, D, h, L, idx=idx)) < 1e-5
    assert np.all(got[B:] == 7.0)


def test_workspace_without_the_panel_part(mlp):  # noqa: F811
    """One byte short of mlp_deep_workspace_bytes: the GEMM launches serve every
    call. Dyadic inputs make both paths' forward exact, hence equal bitwise."""
    h, L, n = 128, 3, 300
    X, Y, P = _dyadic(np.random.default_rng(5), n, h, L)
    need = mlp.load().mlp_deep_workspace_bytes(D, h, L, n)
    p, q = _to(P), _to(P)
    full = mlp.mlp_deep_init(p, h, L, n)
    part = mlp.mlp_deep_init(q, h, L, n, workspace=torch.empty(need - 1, dtype=torch.uint8, device="cuda"))
    assert torch.equal(mlp.mlp_deep_forward(full, _to(X)), mlp.mlp_deep_forward(part, _to(X)))
    a, la = mlp.mlp_deep_backward(full, _to(X), _to(Y))
    b, lb = mlp.mlp_deep_backward(part, _to(X), _to(Y))
    assert rel(a.cpu().numpy(), b.cpu().numpy()) <= 1e-5
    assert abs(float(la) - float(lb)) <= 1e-5 * float(lb)
    mlp.mlp_deep_train_epochs(full, _to(X), _to(Y), 64, 0.01, 2)
    mlp.mlp_deep_train_epochs(part, _to(X), _to(Y), 64, 0.01, 2)
    assert rel((p.cpu().numpy() - P), (q.cpu().numpy() - P)) <= 1e-3
    with pytest.raises(ValueError):
        mlp.mlp_deep_init(q, h, L, n, workspace=torch.empty(4096, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("h,L,B,E", [(192, 3, 300, 2), (256, 2, 5000, 1), (192, 2, 8200, 1), (256, 3, 1000, 2)])
def test_steps_hand_over_weights_and_rows(mlp, h, L, B, E):  # noqa: F811
    """Several steps with a ragged last one, on panels of 16, 32 and 64 rows: each step's
    update splits the next step's weights and gathers its rows."""
    assert _panel_pays(h, L, B)
    n, lr = 2 * B + B // 3, 0.002
    d = datagen.make_data(n, 32, epochs=E, seed=h + B)
    P = _gauss_net(np.random.default_rng(h + B), h, L)
    gP, gsl, gel = _train(mlp, d.X, d.Y, P, h, L, B, lr, E, perm=d.perm)
    ref = oracle.deep_train(d.X, d.Y, P, D, h, L, B, lr, E, perm=d.perm)
    assert ref["steps"] == len(gsl) == 3 * E
    P0 = P.astype(np.float64)
    assert rel(gP - P0, ref["P"] - P0) <= 1e-3
    assert np.all(np.abs(gsl - ref["step_loss"]) <= 1e-4 * ref["step_loss"])
    assert np.all(np.abs(gel - ref["epoch_loss"]) <= 1e-4 * ref["epoch_loss"])
