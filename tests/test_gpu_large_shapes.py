"""The fused trainer's shapes for larger batches (up to 4,096 rows at every width up
to 512 and 2,048 at h = 1024): gradients, training with a tail, and the exchange
protocol's host model for their group counts."""
import numpy as np
import pytest

import datagen
import oracle
from tests.parity import check
from tests.test_exchange_protocol import violations
from tests.test_gpu_parity import _check_grad, _ctx, _env, _to, _train_gpu, mlp  # noqa: F401

# (groups PX, workgroups per group PR, rows R, units U), from index 16 of the library's table
LARGE_SHAPES = [(8, 32, 32, 64), (8, 32, 64, 64), (8, 32, 128, 64), (8, 32, 64, 128),
                (4, 32, 32, 32), (4, 32, 64, 32), (4, 32, 128, 32),
                (2, 32, 32, 32), (2, 32, 64, 32), (2, 32, 128, 32),
                (1, 32, 32, 32), (1, 32, 64, 32), (1, 32, 128, 32)]


@pytest.mark.gpu
@pytest.mark.parametrize("k", range(len(LARGE_SHAPES)))
def test_large_shape(mlp, k):  # noqa: F811
    px, pr, r, u = LARGE_SHAPES[k]
    h, cap = px * u, pr * r
    with _env(MLP_INST=16 + k):
        d = datagen.make_data(64, h, seed=4, with_perm=False)
        ctx, _, _ = _ctx(mlp, d.W1, d.W2, cap)
        assert mlp.mlp_launch_info(ctx, cap, cap, 1) == (8 * pr, 1), "shape table out of step"
        for B in (cap, cap // 2 + 3):
            _check_grad(mlp, h, B, n=2 * cap, seed=k * 7 + B)
        n, lr = 3 * cap - 5, 0.005
        d = datagen.make_data(n, h, epochs=2, shuffle=True, seed=400 + k)
        g1, g2, gsl, gel = _train_gpu(mlp, d, cap, lr, 2, perm=d.perm)
    ref = oracle.train(d.X, d.Y, d.W1, d.W2, cap, lr, 2, perm=d.perm)
    check("W1 - W1_0", g1 - d.W1, ref["W1"] - d.W1.astype(np.float64), 1e-3)
    check("W2 - W2_0", g2 - d.W2, ref["W2"] - d.W2.astype(np.float64), 1e-3)
    assert np.all(np.abs(gsl - ref["step_loss"]) <= 1e-3 * ref["step_loss"])
    assert np.all(np.abs(gel - ref["epoch_loss"]) <= 1e-3 * ref["epoch_loss"])


@pytest.mark.parametrize("px", [1, 2, 4])
def test_exchange_protocol_of_32_workgroup_groups(px):
    assert violations(px, 32, steps=4) == []


@pytest.mark.gpu
@pytest.mark.parametrize("h,B", [(64, 1000), (512, 2048), (256, 256)])
def test_fewer_compute_units_than_workgroups(mlp, h, B):  # noqa: F811
    """A partition of 32 compute units cannot hold the trainer's launch: the tile path
    trains instead."""
    n, lr = 3 * B - 5, 0.005
    d = datagen.make_data(n, h, epochs=1, shuffle=True, seed=h + B)
    with _env(MLP_NUM_CU=32):
        ctx, _, _ = _ctx(mlp, d.W1, d.W2, B)
        assert mlp.mlp_launch_info(ctx, n, B, 1)[1] == 2 * 3 + 1
        g1, g2, gsl, gel = _train_gpu(mlp, d, B, lr, 1, perm=d.perm)
    ref = oracle.train(d.X, d.Y, d.W1, d.W2, B, lr, 1, perm=d.perm)
    check("W1 - W1_0", g1 - d.W1, ref["W1"] - d.W1.astype(np.float64), 1e-3)
    check("W2 - W2_0", g2 - d.W2, ref["W2"] - d.W2.astype(np.float64), 1e-3)
    assert np.all(np.abs(gsl - ref["step_loss"]) <= 1e-3 * ref["step_loss"])


@pytest.mark.gpu
@pytest.mark.parametrize("h,B,n,E,launches", [
    (64, 1000, 20, 1, 2), (64, 1000, 20, 6, 7), (64, 1000, 20, 7, 1),   # steps of one workgroup
    (64, 1000, 1000, 3, 7), (64, 1000, 1000, 4, 1), (32, 4096, 8192, 1, 5),
    (128, 300, 364, 2, 7), (128, 300, 365, 2, 1),                        # a tail of 64 rows, of 65
    (512, 2048, 6000, 1, 7), (1024, 2048, 2048, 4, 1),
    (256, 1000, 20, 1, 1), (64, 256, 20, 1, 1)])                        # the smaller shapes
def test_short_calls(mlp, h, B, n, E, launches):  # noqa: F811
    """Calls of a few steps of the larger batches run on the tile path (up to six launches
    and the epoch-loss clear), longer ones on the trainer; either trains as the
    oracle does, and the static entry does the same bitwise."""
    lr = 0.005
    d = datagen.make_data(n, h, epochs=E, shuffle=True, seed=h + n)
    ctx, _, _ = _ctx(mlp, d.W1, d.W2, B)
    assert mlp.mlp_launch_info(ctx, n, B, E)[1] == launches
    g1, g2, gsl, gel = _train_gpu(mlp, d, B, lr, E, perm=d.perm)
    ref = oracle.train(d.X, d.Y, d.W1, d.W2, B, lr, E, perm=d.perm)
    check("W1 - W1_0", g1 - d.W1, ref["W1"] - d.W1.astype(np.float64), 1e-3)
    check("W2 - W2_0", g2 - d.W2, ref["W2"] - d.W2.astype(np.float64), 1e-3)
    assert np.all(np.abs(gsl - ref["step_loss"]) <= 1e-3 * ref["step_loss"])
    assert np.all(np.abs(gel - ref["epoch_loss"]) <= 1e-3 * ref["epoch_loss"])
    if h <= 256:
        w1, w2 = _to(d.W1), _to(d.W2)
        mlp.mlp_train_epochs_static(w1, w2, _to(d.X), _to(d.Y), B, lr, E, perm=_to(d.perm))
        assert np.array_equal(w1.cpu().numpy(), g1) and np.array_equal(w2.cpu().numpy(), g2)
