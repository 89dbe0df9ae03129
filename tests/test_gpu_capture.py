"""Training calls recorded into a HIP graph: every replay trains one more run from the
weights it finds, bitwise as the call outside a graph does, with calls of the
same context between the replays (the exchange words' step tags are arguments
of the recorded launch, the same at every replay)."""
import numpy as np
import pytest
import torch

import datagen
from tests.test_gpu_parity import _to, mlp  # noqa: F401

pytestmark = pytest.mark.gpu


# the trainer's smaller and larger shapes, and a batch of the tile path
@pytest.mark.parametrize("h,B,n", [(256, 256, 2000), (64, 1000, 12100), (512, 2048, 30000), (256, 6000, 20000)])
@pytest.mark.parametrize("static", [False, True])
def test_replays_train_on(mlp, h, B, n, static):  # noqa: F811
    if static and h > 256:
        pytest.skip("wider than the static entry takes")
    print("h", h, "B", B, "static", static, flush=True)
    d = datagen.make_data(n, h, epochs=1, shuffle=True, seed=h + B)
    X, Y, P, lr = _to(d.X), _to(d.Y), _to(d.perm), 0.002
    steps = -(-n // B)
    s = torch.cuda.Stream()
    runs = []
    for graph in (True, False):
        w1, w2 = _to(d.W1), _to(d.W2)
        sl, el = torch.zeros(steps, device="cuda"), torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            ctx = mlp.mlp_init(w1, w2, B)

            def call():
                if static:
                    mlp.mlp_train_epochs_static(w1, w2, X, Y, B, lr, 1, perm=P, epoch_loss=el, step_loss=sl)
                else:
                    mlp.mlp_train_epochs(ctx, X, Y, B, lr, 1, perm=P, epoch_loss=el, step_loss=sl)

            call()                         # outside any graph first
            torch.cuda.synchronize()
        out = []
        if graph:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                call()
        for k in range(4):
            with torch.cuda.stream(s):
                if graph:
                    g.replay()
                else:
                    call()
                torch.cuda.synchronize()
                out.append([t.cpu().numpy() for t in (w1, w2, sl, el)])
                if k == 1:
                    call()                 # and between the replays
        torch.cuda.synchronize()
        mlp.mlp_check_errors(ctx)
        runs.append(out)
    for a, b in zip(*runs):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
    assert not np.array_equal(runs[0][0][0], runs[0][1][0])   # a replay trains


@pytest.mark.parametrize("h,L,B", [(256, 2, 1024), (64, 3, 100), (384, 2, 700)])
def test_deeper_nets_replay(mlp, h, L, B):  # noqa: F811
    """The panel path and the GEMM launches keep nothing between calls."""
    n = 2 * B + 17
    d = datagen.make_data(n, h, epochs=1, shuffle=True, seed=h + B)
    P0 = (np.random.default_rng(h).standard_normal(mlp.load().mlp_deep_param_count(32, h, L)) / np.sqrt(h))
    X, Y, perm = _to(d.X), _to(d.Y), _to(d.perm)
    s = torch.cuda.Stream()
    runs = []
    for graph in (True, False):
        p = _to(P0.astype(np.float32))
        sl = torch.zeros(3, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            ctx = mlp.mlp_deep_init(p, h, L, B)
            torch.cuda.synchronize()
        if graph:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                mlp.mlp_deep_train_epochs(ctx, X, Y, B, 0.002, 1, perm=perm, step_loss=sl)
        out = []
        for k in range(3):
            with torch.cuda.stream(s):
                if graph:
                    g.replay()
                else:
                    mlp.mlp_deep_train_epochs(ctx, X, Y, B, 0.002, 1, perm=perm, step_loss=sl)
                torch.cuda.synchronize()
                out.append([p.cpu().numpy(), sl.cpu().numpy()])
                mlp.mlp_deep_forward(ctx, X)
        torch.cuda.synchronize()
        mlp.mlp_deep_check_errors(ctx)
        runs.append(out)
    for a, b in zip(*runs):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
