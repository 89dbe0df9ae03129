"""GPU parity of the one-launch and two-launch gradient path (k_batch, mlp.hip) at
the edges of its passes: 32-row passes (64 at h = 32), one workgroup up to 64 rows,
and more passes than workgroups (256) from 8,193 rows (16,385 at h = 32)."""
import numpy as np
import pytest
import torch

import datagen
import oracle
from tests.parity import rel
from tests.test_gpu_parity import _check_grad, _ctx, _env, _rows, _to, mlp  # noqa: F401

pytestmark = pytest.mark.gpu

H_ALL = (32, 64, 128, 256, 512, 1024)


@pytest.mark.parametrize("h", H_ALL)
@pytest.mark.parametrize("B", [31, 33, 63, 65, 96, 8193, 16385])
def test_gradient_at_pass_edges(mlp, h, B):  # noqa: F811
    _check_grad(mlp, h, B, n=max(3000, 2 * B), seed=h + B)


@pytest.mark.parametrize("h", H_ALL)
@pytest.mark.parametrize("B", [64, 65])
def test_step_applies_the_gradient(mlp, h, B):  # noqa: F811
    """mlp_sgd_step's weights are W - lr dW with mlp_backward's dW: the two differ
    by the rounding of the product and the difference (2 u of the result, 1 u of the
    product), on one workgroup (64 rows) and through the reduction (65)."""
    d = datagen.make_data(500, h, seed=h, with_perm=False)
    idx = _to(_rows(np.random.default_rng(B), 500, B))
    X, Y, lr = _to(d.X), _to(d.Y), 0.125
    ctx, w1, w2 = _ctx(mlp, d.W1, d.W2, B)
    dW1, dW2, loss = mlp.mlp_backward(ctx, X, Y, idx)
    e1, e2 = w1 - lr * dW1, w2 - lr * dW2
    sl = loss.clone().zero_()
    mlp.mlp_sgd_step(ctx, X, Y, lr, idx=idx, loss=sl)
    mlp.mlp_check_errors(ctx)
    assert float(sl) == float(loss)
    u = 2.0 ** -24
    assert bool(((w1 - e1).abs() <= 4 * u * (e1.abs() + lr * dW1.abs())).all())
    assert bool(((w2 - e2).abs() <= 4 * u * (e2.abs() + lr * dW2.abs())).all())


@pytest.mark.parametrize("h", [256, 512, 1024])
@pytest.mark.parametrize("B", [16383, 16384, 16385, 70001])
@pytest.mark.parametrize("gather", [True, False])
def test_forward_of_many_rows(mlp, h, B, gather):  # noqa: F811
    """The forward pass around the row count from which the wider nets take 32-row
    passes, and over several passes a wave with a ragged last one; outputs past B
    stay untouched and an index out of range is flagged."""
    n = 3000 if gather else B
    d = datagen.make_data(n, h, seed=h, with_perm=False)
    ctx, _, _ = _ctx(mlp, d.W1, d.W2, 64)
    idx = _rows(np.random.default_rng(B), n, B) if gather else None
    out = torch.full((B + 40,), 7.0, device="cuda")
    mlp.mlp_forward(ctx, _to(d.X), None if idx is None else _to(idx), B=B, out=out)
    mlp.mlp_check_errors(ctx)
    got = out.cpu().numpy()
    assert rel(got[:B], oracle.forward(d.X, d.W1, d.W2, idx=idx)) < 1e-5
    assert np.all(got[B:] == 7.0)
    if gather:
        idx[B // 2] = n
        mlp.mlp_forward(ctx, _to(d.X), _to(idx), B=B, out=out)
        with pytest.raises(mlp.MLPError) as e:
            mlp.mlp_check_errors(ctx)
        assert e.value.status == -6


def test_phase_sums_are_not_read_past_their_call(mlp):  # noqa: F811
    """A traced training call's phase sums lie where the gradient's partials go: after a
    gradient there are none to copy."""
    d = datagen.make_data(5000, 256, epochs=1, shuffle=False, seed=3)
    ctx, _, _ = _ctx(mlp, d.W1, d.W2, 256)
    X, Y = _to(d.X), _to(d.Y)
    with _env(MLP_TRACE=1):
        mlp.mlp_train_epochs(ctx, X, Y, 256, 0.001, 1)
    c = mlp.mlp_phase_cycles(ctx)
    assert c is not None and np.all(c[:, :, 0].max(axis=0) == 20 - 8)   # steps from the eighth on
    mlp.mlp_backward(ctx, X, Y, B=100)
    assert mlp.mlp_phase_cycles(ctx) is None
