"""A training call whose workgroups cannot all start in time (other work holds part of
the GPU) is done by one workgroup. MLP_START_TICKS=0 gives every launch up at its
start barrier; a limit of 1 (10 ns) runs into it while workgroups still arrive, and
either way of running is right."""
import numpy as np
import pytest

import datagen
import oracle
from tests.parity import check
from tests.test_gpu_parity import _ctx, _env, _to, _train_gpu, mlp  # noqa: F401

pytestmark = pytest.mark.gpu


def _compare(d, B, lr, E, got, max_steps=-1):
    g1, g2, gsl, gel = got
    ref = oracle.train(d.X, d.Y, d.W1, d.W2, B, lr, E, perm=d.perm, max_steps=max_steps)
    check("W1 - W1_0", g1 - d.W1, ref["W1"] - d.W1.astype(np.float64), 1e-3)
    check("W2 - W2_0", g2 - d.W2, ref["W2"] - d.W2.astype(np.float64), 1e-3)
    assert np.all(np.abs(gsl - ref["step_loss"]) <= 1e-3 * ref["step_loss"])
    assert np.all(np.abs(gel - ref["epoch_loss"]) <= 1e-3 * ref["epoch_loss"])


# every width; batches of one to four thousand rows, none a multiple of 64 (the rows
# staged at a time), the last of an epoch shorter
@pytest.mark.parametrize("ticks", [0, 1])
@pytest.mark.parametrize("h,B,n,E", [(32, 1000, 2300, 2), (64, 300, 1000, 2), (128, 4093, 17000, 1),
                                     (256, 1, 3, 2), (256, 4096, 9000, 1), (512, 700, 2900, 1),
                                     (1024, 1030, 4200, 1)])
def test_given_up_launch_trains(mlp, h, B, n, E, ticks):  # noqa: F811
    print("h", h, "B", B, "ticks", ticks, flush=True)
    d = datagen.make_data(n, h, epochs=E, shuffle=True, seed=h + B)
    lr = 0.002
    with _env(MLP_START_TICKS=ticks):
        _compare(d, B, lr, E, _train_gpu(mlp, d, B, lr, E, perm=d.perm))


def test_given_up_launch_in_identity_order_and_short(mlp):  # noqa: F811
    """No permutation; a call cut short in its first epoch, whose later epoch losses
    are zero; the call after it runs as ever."""
    d = datagen.make_data(1000, 256, epochs=3, shuffle=False, seed=5)
    with _env(MLP_START_TICKS=0):
        got = _train_gpu(mlp, d, 300, 0.01, 3, max_steps=2)
    d.perm = None
    _compare(d, 300, 0.01, 3, got, max_steps=2)
    assert got[3][0] > 0 and np.all(got[3][1:] == 0)
    a = _train_gpu(mlp, d, 300, 0.01, 3)
    _compare(d, 300, 0.01, 3, a)


def test_given_up_launch_flags_a_bad_row(mlp):  # noqa: F811
    d = datagen.make_data(1500, 64, epochs=1, shuffle=True, seed=6)
    P = d.perm.copy()
    P[0, 333] = 1500
    with _env(MLP_START_TICKS=0):
        ctx, _, _ = _ctx(mlp, d.W1, d.W2, 300)
        mlp.mlp_train_epochs(ctx, _to(d.X), _to(d.Y), 300, 0.01, 1, perm=_to(P))
        with pytest.raises(mlp.MLPError) as e:
            mlp.mlp_check_errors(ctx)
    assert e.value.status == -6
