"""Performance cases of the MLP-SGD library, through its public entry points.

Every case is one call that a program makes on resident data: an SGD step, a
gradient, a training run over epochs or a forward pass, on the one-hidden-layer
net (32-h-1) or on the deeper ones (32-h-...-h-1, L hidden layers). A case is a
dict of plain values:

  kind      "step", "grad", "train", "forward" on the one-layer net;
            "deep_step", "deep_grad", "deep_train", "deep_forward" with L layers
  hidden    units per hidden layer
  layers    hidden layers (deep kinds)
  rows      rows of the dataset in device memory
  batch     rows of a step or gradient, the mini-batch of a training run, the
            rows of a forward pass
  gather    rows taken through an index array or per-epoch permutation
  epochs    training kinds
  max_batch deep_forward: the batch the context was created for
  static    train: through mlp_train_epochs_static

Inputs follow the repository's data recipe (Gaussian rows, a smooth noisy target,
He-normal weights), drawn on the GPU from the seed.
"""
import math

import torch

from paper_2606_30497_amd import mlp

D_IN = 32
HIDDEN = (32, 64, 128, 256, 512, 1024)
LR = 0.002   # the paper's learning rate


def _case(name, kind, hidden, rows, batch, gather=True, **more):
    c = {"kind": kind, "hidden": hidden, "rows": rows, "batch": batch, "gather": gather}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # one step on the smallest evaluation batch: online training, where the
        # call's launches and latency are all there is
        _case("step_h256_b64", "step", 256, 1024, 64),
        # the paper's largest dataset and its batch of 256 (Table I), four epochs
        _case("train_h256_n25600_b256", "train", 256, 25_600, 256, epochs=4, static=False),
        # a narrow net (Table II) trained on a medium dataset with a larger batch
        # that leaves a remainder
        _case("train_h64_n100003_b1000", "train", 64, 100_003, 1000, epochs=1, static=False),
        # a wide net (Table II) at a large batch
        _case("train_h512_n200k_b2048", "train", 512, 200_000, 2048, epochs=1, static=False),
        # the 1M-row workload of the 1024-wide net, one epoch
        _case("train_h1024_n1M_b1024", "train", 1024, 1_000_000, 1024, epochs=1, static=False),
        # the 10M-row workload, one epoch: the largest training run
        _case("train_h256_n10M_b4096", "train", 256, 10_000_000, 4096, epochs=1, static=False),
        # the gradient of a large gathered batch, for a caller with its own optimizer
        _case("grad_h256_b20001", "grad", 256, 1_000_000, 20_001),
        # evaluation of the whole 10M-row dataset
        _case("forward_h256_n10M", "forward", 256, 10_000_000, 10_000_000, gather=False),
        # inference on a small gathered request
        _case("forward_h128_b1777", "forward", 128, 100_000, 1777),
        # the deeper nets of the deep suite, one epoch of a smaller dataset with
        # a remainder batch: two layers of 256 and two of 1024
        _case("deep_train_256x2_b4096", "deep_train", 256, 100_000, 4096, layers=2, epochs=1),
        _case("deep_train_1024x2_b4096", "deep_train", 1024, 50_000, 4096, layers=2, epochs=1),
        # evaluation of a 1M-row dataset on the context that trained the net
        _case("deep_forward_256x3_n1M", "deep_forward", 256, 1_000_000, 1_000_000, gather=False,
              layers=3, max_batch=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: every kind, width, batch and option,
    odd sizes included, at most 60 GFLOP and 400 steps."""
    kind = rng.choice(("step", "grad", "train", "train", "forward", "forward",
                       "deep_step", "deep_grad", "deep_train", "deep_forward"))
    gather = rng.random() < 0.75
    if not kind.startswith("deep"):
        h = rng.choice(HIDDEN)
        if kind == "step":
            b = _log(rng, 1, 8192)
            return _case(None, kind, h, b + _log(rng, 1, 100_000), b, gather)
        if kind == "grad":
            b = _log(rng, 64, 65_536)
            return _case(None, kind, h, b + _log(rng, 1, 400_000), b, gather)
        if kind == "forward":
            b = _log(rng, 16, 2_000_000)
            b = min(b, int(60e9 / (66 * h)))
            rows = b if not gather else _log(rng, 1000, 1_000_000)
            return _case(None, kind, h, rows, b, gather)
        b = _log(rng, 32, 8192)
        n = _log(rng, max(64, b // 2), 400 * b)
        n = max(1, min(n, 1_000_000, int(60e9 / (134 * h))))
        steps = -(-n // b)
        epochs = max(1, min(rng.randint(1, 6), 400 // steps, int(60e9 / (134 * h * n))))
        return _case(None, kind, h, n, b, gather, epochs=epochs,
                     static=h <= 256 and rng.random() < 0.2)
    h = 64 * rng.choice((1, 2, 3, 4, 4, 4, 5, 8, 12, 16))
    L = rng.choice((1, 2, 2, 3, 3, 4, 6, 8))
    flop = 6 * (D_IN * h + (L - 1) * h * h)
    top = max(64, int(60e9 / flop))
    if kind in ("deep_step", "deep_grad"):
        b = min(_log(rng, 16, 16_384), top)
        return _case(None, kind, h, b + _log(rng, 1, 100_000), b, gather, layers=L)
    if kind == "deep_forward":
        b = min(_log(rng, 16, 300_000), 2 * top)
        rows = b if not gather else _log(rng, 1000, 300_000)
        return _case(None, kind, h, rows, b, gather, layers=L, max_batch=min(b, _log(rng, 64, 8192)))
    b = min(_log(rng, 64, 8192), top)
    n = min(_log(rng, b, 30 * b), top)
    return _case(None, kind, h, n, b, gather, layers=L, epochs=1)


def _shapes(case):
    """[rows, columns] of each weight matrix of the flat parameter array."""
    h, L = case["hidden"], case.get("layers", 1)
    return [(D_IN, h)] + [(h, h)] * (L - 1) + [(h, 1)]


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(*shape, device="cuda", generator=g)

    n = case["rows"]
    a = normal(D_IN) / math.sqrt(D_IN)
    X = normal(n, D_IN)
    Y = None
    if "forward" not in case["kind"]:
        Y = torch.sin(X @ a) + 0.1 * normal(n)
    weights = [normal(r, c) * math.sqrt(2.0 / r) for r, c in _shapes(case)]
    idx = None
    if "train" in case["kind"]:
        if case["gather"]:
            idx = torch.stack([torch.randperm(n, device="cuda", generator=g, dtype=torch.int32)
                               for _ in range(case["epochs"])])
    elif case["gather"]:
        idx = torch.randint(0, n, (case["batch"],), device="cuda", generator=g, dtype=torch.int32)
    return X, Y, weights, idx


def prepare(case, seed):
    X, Y, weights, idx = _inputs(case, seed)
    s = {"case": case, "X": X, "Y": Y, "idx": idx}
    kind, batch = case["kind"], case["batch"]
    if kind.startswith("deep"):
        s["params"] = torch.cat([w.reshape(-1) for w in weights])
        s["ctx"] = mlp.mlp_deep_init(s["params"], case["hidden"], case["layers"],
                                     case.get("max_batch", batch))
    else:
        s["W1"], s["W2"] = weights[0], weights[1].reshape(-1)
        if not case.get("static"):
            # a forward pass takes any number of rows: the context is a trainer's
            s["ctx"] = mlp.mlp_init(s["W1"], s["W2"], min(batch, 4096) if kind == "forward" else batch)
    if "forward" in kind:
        s["out"] = torch.empty(batch, device="cuda")
    if "step" in kind:
        s["loss"] = torch.empty(1, device="cuda")
    if "train" in kind:
        steps = -(-case["rows"] // batch) * case["epochs"]
        s["epoch_loss"] = torch.empty(case["epochs"], device="cuda")
        s["step_loss"] = torch.empty(steps, device="cuda")
    return s


def run(s):
    c = s["case"]
    kind, X, Y, idx, batch = c["kind"], s["X"], s["Y"], s["idx"], c["batch"]
    if kind == "step":
        mlp.mlp_sgd_step(s["ctx"], X, Y, LR, idx=idx, B=batch, loss=s["loss"])
        return [s["W1"], s["W2"], s["loss"]]
    if kind == "grad":
        return mlp.mlp_backward(s["ctx"], X, Y, idx=idx, B=batch)
    if kind == "forward":
        return mlp.mlp_forward(s["ctx"], X, idx=idx, B=batch, out=s["out"])
    if kind == "train":
        kw = dict(perm=idx, epoch_loss=s["epoch_loss"], step_loss=s["step_loss"])
        if c["static"]:
            mlp.mlp_train_epochs_static(s["W1"], s["W2"], X, Y, batch, LR, c["epochs"], **kw)
        else:
            mlp.mlp_train_epochs(s["ctx"], X, Y, batch, LR, c["epochs"], **kw)
        return [s["W1"], s["W2"], s["epoch_loss"], s["step_loss"]]
    if kind == "deep_step":
        mlp.mlp_deep_sgd_step(s["ctx"], X, Y, LR, idx=idx, B=batch, loss=s["loss"])
        return [s["params"], s["loss"]]
    if kind == "deep_grad":
        return mlp.mlp_deep_backward(s["ctx"], X, Y, idx=idx, B=batch)
    if kind == "deep_forward":
        return mlp.mlp_deep_forward(s["ctx"], X, idx=idx, B=batch, out=s["out"])
    mlp.mlp_deep_train_epochs(s["ctx"], X, Y, batch, LR, c["epochs"], perm=idx,
                              epoch_loss=s["epoch_loss"], step_loss=s["step_loss"])
    return [s["params"], s["epoch_loss"], s["step_loss"]]


def work(case):
    """Each input row, target, index and weight read once, each output written
    once; the contractions of eqs. 11-18 at 2 FLOP per multiply-add (a layer's
    three products, less the one into the inputs)."""
    kind, n, b = case["kind"], case["rows"], case["batch"]
    sizes = [r * c for r, c in _shapes(case)]
    params = sum(sizes)
    if "forward" in kind:
        rows = b
        flops = 2 * params * rows
        moved = rows * (4 * D_IN + 4) + 4 * params
    else:
        visits = n * case["epochs"] if "train" in kind else b
        rows = n if "train" in kind else b
        flops = (6 * params - 2 * sizes[0]) * visits
        moved = rows * (4 * D_IN + 4) + 8 * params
    if case["gather"]:
        moved += 4 * (n * case["epochs"] if "train" in kind else b)
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    """About four times the largest error against exact() seen over 130 cases.

    A gradient's error is rounding (2e-7) unless a pre-activation within rounding
    of zero takes the other ReLU mask, which adds or drops one of the batch's
    terms: 3.1e-5 seen at 20,001 rows, growing as 1 / sqrt(rows). A step's one-row
    loss squares a residual that may be small against its two terms. Training
    carries the masks' differences along (one layer 1.3e-6, up to four 8e-7, eight
    layers 2.5e-5)."""
    kind = case["kind"]
    if kind in ("grad", "deep_grad"):
        return {"rel": min(2e-3, max(1e-4, 1.2e-4 * math.sqrt(20_000 / case["batch"])))}
    if kind == "forward":
        return {"rel": 6e-7}
    if kind == "deep_forward":
        return {"rel": 6e-6}
    if kind == "deep_train" and case["layers"] > 4:
        return {"rel": 1e-4}
    if kind == "train":
        return {"rel": 5e-6}
    return {"rel": 1e-5}


def _exact_step(ws, x, y, lr):
    """Loss, gradients and (lr given) updated weights of one batch, float64."""
    acts = [x]
    for w in ws[:-1]:
        acts.append(torch.relu(acts[-1] @ w))
    res = (acts[-1] @ ws[-1]).reshape(-1) - y
    loss = (res * res).mean()
    g = (2.0 / x.shape[0]) * res[:, None]
    grads = [None] * len(ws)
    for i in range(len(ws) - 1, -1, -1):
        grads[i] = acts[i].T @ g
        if i:
            g = (g @ ws[i].T) * (acts[i] > 0)
    if lr is not None:
        ws = [w - lr * d for w, d in zip(ws, grads)]
    return loss, grads, ws


def exact(case, seed):
    X, Y, weights, idx = _inputs(case, seed)
    kind, n, b = case["kind"], case["rows"], case["batch"]
    ws = [w.double() for w in weights]
    lr = float(torch.tensor(LR, dtype=torch.float32))
    deep = kind.startswith("deep")

    def params(parts):
        if deep:
            return [torch.cat([p.reshape(-1) for p in parts])]
        return [parts[0], parts[1].reshape(-1)]

    if "forward" in kind:
        out = torch.empty(b, dtype=torch.float64, device="cuda")
        for i in range(0, b, 100_000):
            j = min(b, i + 100_000)
            h = (X[idx[i:j].long()] if idx is not None else X[i:j]).double()
            for w in ws[:-1]:
                h = torch.relu(h @ w)
            out[i:j] = (h @ ws[-1]).reshape(-1)
        return out
    if "train" not in kind:
        at = idx.long() if idx is not None else torch.arange(b, device="cuda")
        loss, grads, new = _exact_step(ws, X[at].double(), Y[at].double(),
                                       lr if "step" in kind else None)
        return params(new if "step" in kind else grads) + [loss.reshape(1)]
    epoch_loss, step_loss = [], []
    for e in range(case["epochs"]):
        sse = torch.zeros((), dtype=torch.float64, device="cuda")
        for i in range(0, n, b):
            j = min(n, i + b)
            at = idx[e, i:j].long() if idx is not None else slice(i, j)
            loss, _, ws = _exact_step(ws, X[at].double(), Y[at].double(), lr)
            step_loss.append(loss)
            sse = sse + loss * (j - i)
        epoch_loss.append(sse / n)
    return params(ws) + [torch.stack(epoch_loss), torch.stack(step_loss)]
