"""Performance cases of the library: what a program built on it does, through
the public binding (paper_1902_06714_amd.nf), from the smallest call to the
largest network of the workloads.

A case names one pass:

* ``train``: one or more epochs of consecutive mini-batches (nf_train_epoch)
  or of randomly placed windows (nf_train_windows), after which the program
  reads the updated weights back (nf_get_params);
* ``online``: a loop of single-sample steps (nf_train_single), then the weights;
* ``grads``: one mini-batch step (nf_train_batch), then its tendencies
  (nf_get_grads) and the updated weights, as a program that checks or combines
  gradients reads them;
* ``infer``: batched inference (nf_forward) into the program's own buffer.

Inputs follow the workloads: uniform [0, 1) or N(0, 1) samples, one-hot
targets, N(0,1)/sqrt(fan_in) or He-normal weights, N(0,1) biases.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_1902_06714_amd import nf

DEV = "cuda:0"


# -- the cases ---------------------------------------------------------------
def _case(name, call, dims, acts, batch, **kw):
    c = {"call": call, "dims": "-".join(map(str, dims)), "acts": ",".join(acts), "batch": batch,
         "steps": 1, "epochs": 1, "samples": 0, "windows": False, "shards": 1, "eta": 0.1, "dtype": "f32",
         "dist": "uniform", "init": "fan_in"}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    mnist = (784, 30, 10)
    return [
        # one request to a served digit classifier: pure latency
        _case("serve-784-30-10-n1", "infer", mnist, ("sigmoid",), 1),
        # online training, one sample a step (the paper's train_single)
        _case("online-784-30-10", "online", mnist, ("sigmoid",), 1, steps=100, eta=1.0),
        # the small classifier workload: ten epochs of ten mini-batches of 100
        _case("train-784-30-10-b100", "train", mnist, ("sigmoid",), 100, steps=10, epochs=10,
              eta=3.0),
        # the headline workload: three epochs of 60 mini-batches of 1000 ...
        _case("train-784-30-10-b1000", "train", mnist, ("sigmoid",), 1000, steps=60, epochs=3,
              eta=3.0),
        # ... and the evaluation of its 10000 held-out samples
        _case("infer-784-30-10-n10000", "infer", mnist, ("sigmoid",), 10000),
        # two tanh layers of 100, the batch in 16 shards as 16 images would hold it
        _case("train-784-100-100-10-s16", "train", (784, 100, 100, 10),
              ("tanh", "tanh", "sigmoid"), 10000, steps=6, epochs=5, shards=16, eta=1.0),
        # a small ragged network (odd width, unaligned rows) on random windows
        _case("windows-129-77-33-5-b2049", "train", (129, 77, 33, 5),
              ("gaussian", "tanh", "sigmoid"), 2049, steps=40, samples=20001, windows=True, eta=0.5),
        # an odd-sized wider network, gradients read by the program, 3 shards
        _case("grads-1001-517-259-10-b3003", "grads", (1001, 517, 259, 10),
              ("relu", "tanh", "sigmoid"), 3003, shards=3),
        # three relu layers of 1024 (at the workload's rate of 0.1 sixteen steps amplify
        # the last bit of the weights a hundredfold or more, at 0.03 they don't)
        _case("train-784-1024x3-10", "train", (784, 1024, 1024, 1024, 10),
              ("relu", "relu", "relu", "sigmoid"), 4096, steps=16, eta=0.03, init="he"),
        # inference through the same network
        _case("infer-784-1024x3-10-n10000", "infer", (784, 1024, 1024, 1024, 10),
              ("relu", "relu", "relu", "sigmoid"), 10000, init="he"),
        # the widest workload: three relu layers of 4096, N(0,1) inputs
        _case("train-4096x4-10", "train", (4096, 4096, 4096, 4096, 10),
              ("relu", "relu", "relu", "sigmoid"), 8192, steps=4, eta=0.01, init="he",
              dist="normal"),
        # the 16-shard workload in double precision
        _case("train-784-100-100-10-s16-f64", "train", (784, 100, 100, 10),
              ("tanh", "tanh", "sigmoid"), 10000, steps=6, epochs=3, shards=16, eta=1.0, dtype="f64"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed ones' ranges: networks of 1 to 3 hidden
    layers, narrow (up to 32 units), medium (up to 128) or wide (up to 4096)."""
    while True:
        width = rng.choice(["narrow", "medium", "wide"])
        lo, hi = {"narrow": (4, 32), "medium": (33, 128), "wide": (129, 4096)}[width]
        d0 = 784 if rng.random() < 0.4 else _log_int(rng, 64, 4096 if width == "wide" else 1024)
        dims = [d0] + [_log_int(rng, lo, hi) for _ in range(rng.randint(1, 3))]
        dims.append(10 if rng.random() < 0.6 else rng.randint(1, 32))
        hidden = rng.choice(["sigmoid", "tanh", "relu", "gaussian"])
        acts = [hidden] * (len(dims) - 2) + ["sigmoid"]
        dtype = "f64" if rng.random() < 0.2 else "f32"
        call = rng.choices(["train", "infer", "grads", "online"], [6, 3, 2, 1])[0]
        batch = 1 if call == "online" else _log_int(rng, 1, 10000 if call == "infer" else 8192)
        kw = dict(dtype=dtype, init="he" if hidden == "relu" else "fan_in",
                  dist=rng.choice(["uniform", "normal"]),
                  eta={"narrow": 0.5, "medium": 0.2, "wide": 0.02}[width])
        if hidden == "relu":
            kw["eta"] /= 4
        if call in ("train", "online"):
            kw["steps"] = _log_int(rng, 1, 50)
        if call == "train" and rng.random() < 0.4:
            kw["windows"] = True
            kw["samples"] = batch + rng.randint(0, 3 * batch)
        elif call == "train":
            kw["epochs"] = rng.randint(1, 5)
        if call in ("train", "grads") and batch >= 64 and rng.random() < 0.4:
            kw["shards"] = rng.choice([2, 3, 4, 8, 16])
            batch -= batch % kw["shards"]
        c = _case(None, call, dims, acts, batch, **kw)
        w = work(c)
        cap = 8e12 if dtype == "f32" else 1.5e12
        if w["flops"] <= cap and w["bytes"] <= 2e9:
            return c


def _dims(case):
    return [int(v) for v in case["dims"].split("-")]


def _acts(case):
    a = case["acts"].split(",")
    n = len(_dims(case)) - 1
    return a * n if len(a) == 1 else a


def _n_samples(case):
    if case["call"] in ("infer", "grads"):
        return case["batch"]
    return case["samples"] if case["windows"] else case["batch"] * case["steps"]


def _tdtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


# -- inputs ------------------------------------------------------------------
def _inputs(case, seed):
    """(x, y, canonical parameters as a GPU tensor, window positions)."""
    dims, dt = _dims(case), _tdtype(case)
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    n = _n_samples(case)
    make = torch.rand if case["dist"] == "uniform" else torch.randn
    x = make((n, dims[0]), generator=g, device=DEV, dtype=dt)
    label = torch.randint(dims[-1], (n,), generator=g, device=DEV)
    y = torch.zeros((n, dims[-1]), device=DEV, dtype=dt)
    y[torch.arange(n, device=DEV), label] = 1
    parts = []
    for l in range(1, len(dims)):
        scale = math.sqrt((2.0 if case["init"] == "he" else 1.0) / dims[l - 1])
        parts.append(torch.randn(dims[l] * dims[l - 1], generator=g, device=DEV, dtype=dt) * scale)
        parts.append(torch.randn(dims[l], generator=g, device=DEV, dtype=dt))
    theta = torch.cat(parts)
    pos = np.random.default_rng(int(seed)).random(case["steps"], dtype=np.float32)
    return x, y, theta, pos


class _State:
    """What the program holds: the network, its data and an output buffer."""

    def __init__(self, case, seed):
        self.case = case
        self.x, self.y, theta, self.pos = _inputs(case, seed)
        self.f64 = case["dtype"] == "f64"
        dims = _dims(case)
        self.net = nf.nf_net_create(dims, _acts(case), nf.NF_F64 if self.f64 else nf.NF_F32)
        (nf.nf_set_params_f64 if self.f64 else nf.nf_set_params)(self.net, theta.cpu().numpy())
        self.out = None
        if case["call"] == "infer":
            self.out = torch.empty((case["batch"], dims[-1]), device=DEV, dtype=_tdtype(case))

    def __del__(self):
        net, self.net = getattr(self, "net", None), None
        if net:
            nf.nf_net_destroy(net)


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    c, f64 = s.case, s.f64
    if c["call"] == "infer":
        (nf.nf_forward_f64 if f64 else nf.nf_forward)(s.net, s.x, s.out)
        return s.out
    get_params = nf.nf_get_params_f64 if f64 else nf.nf_get_params
    if c["call"] == "online":
        step = nf.nf_train_single_f64 if f64 else nf.nf_train_single
        for i in range(c["steps"]):
            step(s.net, s.x[i], s.y[i], c["eta"])
        return get_params(s.net)
    if c["call"] == "grads":
        (nf.nf_train_batch_f64 if f64 else nf.nf_train_batch)(s.net, s.x, s.y, c["eta"], c["shards"])
        grads = (nf.nf_get_grads_f64 if f64 else nf.nf_get_grads)(s.net)
        return {"grads": grads, "params": get_params(s.net)}
    if c["windows"]:
        (nf.nf_train_windows_f64 if f64 else nf.nf_train_windows)(
            s.net, s.x, s.y, c["batch"], s.pos, c["eta"], c["shards"])
    else:
        epoch = nf.nf_train_epoch_f64 if f64 else nf.nf_train_epoch
        for _ in range(c["epochs"]):
            epoch(s.net, s.x, s.y, c["batch"], c["eta"], c["shards"])
    return get_params(s.net)


def work(case):
    """Every input, target and parameter read once, every result written once
    (a training pass's weights to the program's memory); flops of the forward
    products, the hidden deltas and the tendencies."""
    dims, es = _dims(case), 8 if case["dtype"] == "f64" else 4
    prod = [a * b for a, b in zip(dims, dims[1:])]
    params = sum(prod) + sum(dims[1:])
    n = case["batch"] * case["steps"] * case["epochs"]
    if case["call"] == "infer":
        return {"bytes": es * (n * (dims[0] + dims[-1]) + params), "flops": 2.0 * n * sum(prod)}
    seen = min(n, _n_samples(case))
    results = 2 if case["call"] == "grads" else 1
    return {"bytes": es * (seen * (dims[0] + dims[-1]) + (1 + results) * params),
            "flops": 2.0 * n * (2 * sum(prod) + sum(prod[1:]))}


def tolerance(case):
    """About four times the largest error against fp64 over some 150 drawn
    cases: fp32 sums in another order 3e-7 (inference) and 7e-7 (schedules); a
    relu schedule's other sides of a kink up to 5e-6 and fp64 2e-15, each with
    a margin for schedules that amplify more."""
    if case["dtype"] == "f64":
        return {"rel": 5e-14}
    if case["call"] == "infer":
        return {"rel": 1.5e-6}
    if "relu" in case["acts"]:
        return {"rel": 2e-5}
    return {"rel": 4e-6}


# -- the same in fp64, plain torch -------------------------------------------
def _act(name, z):
    if name == "sigmoid":
        f = torch.sigmoid(z)
        return f, f * torch.sigmoid(-z)
    if name == "tanh":
        f = torch.tanh(z)
        return f, 1.0 - f * f
    if name == "relu":
        return torch.clamp(z, min=0), (z > 0).to(z.dtype)
    f = torch.exp(-z * z)
    return f, -2.0 * z * f


def exact(case, seed):
    dims, acts = _dims(case), _acts(case)
    x, y, theta, pos = _inputs(case, seed)
    f32 = case["dtype"] == "f32"
    if work(case)["flops"] > 1.2e13:
        return None
    theta = theta.double()
    W, b, o = [], [], 0
    for l in range(1, len(dims)):
        n = dims[l] * dims[l - 1]
        W.append(theta[o:o + n].view(dims[l], dims[l - 1]).clone())
        b.append(theta[o + n:o + n + dims[l]].clone())
        o += n + dims[l]

    def flat(ws, bs):
        return torch.cat([t.reshape(-1) for pair in zip(ws, bs) for t in pair]).cpu().numpy()

    def forward(xs):
        a, fp = [xs.double()], []
        for l in range(len(W)):
            f, d = _act(acts[l], a[-1] @ W[l].t() + b[l])
            a.append(f)
            fp.append(d)
        return a, fp

    if case["call"] == "infer":
        return forward(x)[0][-1]
    batch, steps = case["batch"], case["steps"]
    for t in range(steps * case["epochs"]):
        s = t % steps * batch
        if case["windows"]:
            last = x.shape[0] - batch
            p = pos[t] * np.float32(last + 1) if f32 else float(pos[t]) * (last + 1)
            s = min(int(p), last)
        a, fp = forward(x[s:s + batch])
        d = (a[-1] - y[s:s + batch].double()) * fp[-1]
        gw, gb = [None] * len(W), [None] * len(W)
        for l in reversed(range(len(W))):
            gw[l], gb[l] = d.t() @ a[l], d.sum(0)
            if l:
                d = (d @ W[l]) * fp[l - 1]
        for l in range(len(W)):
            W[l] -= case["eta"] / batch * gw[l]
            b[l] -= case["eta"] / batch * gb[l]
    if case["call"] == "grads":
        return {"grads": flat(gw, gb), "params": flat(W, b)}
    return flat(W, b)
