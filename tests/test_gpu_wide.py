"""The wide fp32 contractions (three-part bf16 products) at the edges of their
tiles, and with operands that the three parts cannot hold."""

import numpy as np
import pytest

from oracle import mlp

from . import parity
from .gpu_run import GpuNet, note, to_dev
from .test_gpu_parity import _compare_trajectory, _problem

pytestmark = pytest.mark.gpu

EDGES = [
    # dims, acts, batch, shards, eta, tile that must appear
    ((129, 193, 66), ("tanh", "sigmoid"), 1, 1, 0.5, "64x64"),        # one row; aligned and not
    ((17, 130, 65, 3), ("sigmoid", "tanh", "sigmoid"), 63, 1, 0.5, "64x64"),
    ((1001, 200, 131), ("tanh", "sigmoid"), 191, 1, 0.5, "64x64"),    # k = 1001: partial last stage
    # k and rows about the stages of 32 and the 8 rows that share a branch
    ((16, 133, 31), ("sigmoid", "tanh"), 7, 1, 0.5, "64x64"),
    ((32, 160, 1), ("gaussian", "sigmoid"), 8, 1, 0.5, "64x64"),
    ((33, 129, 47), ("tanh",), 9, 3, 0.5, "64x64"),
    ((48, 224, 64), ("sigmoid",), 33, 1, 0.5, "64x64"),
    ((95, 193, 65), ("tanh", "gaussian"), 65, 1, 0.2, "64x64"),
    ((97, 131, 7), ("relu", "sigmoid"), 40, 2, 0.2, "64x64"),
    ((515, 1023, 1030), ("gaussian", "sigmoid"), 4095, 1, 0.2, "128x128"),
    ((512, 1024, 1153), ("tanh", "sigmoid"), 3969, 3, 0.2, "128x128"),
    ((31, 4093, 4090), ("tanh", "sigmoid"), 4081, 1, 0.02, "256x256"),
    ((48, 4096, 4090, 5), ("sigmoid", "tanh", "sigmoid"), 4080, 2, 0.02, "256x256"),
]


@pytest.mark.parametrize("dims,acts,batch,shards,eta,tile", EDGES)
def test_wide_edges(dims, acts, batch, shards, eta, tile):
    theta, X, Y = _problem(dims, 3 * sum(dims) + batch, batch)
    note(f"wide edges dims={dims} batch={batch} shards={shards}")
    _compare_trajectory(dims, acts, theta, X, Y, batch, eta, shards, 1)
    with GpuNet(dims, acts, theta) as net:
        net.nf.nf_profile(net.h, 1)
        net.train_batch(to_dev(X), to_dev(Y), eta, shards)
        names = {k["name"] for k in net.nf.nf_profile_read(net.h)}
        net.nf.nf_profile(net.h, 0)
    assert any(n.startswith("wide_") and n.endswith(tile) for n in names), names


def _single_layer(rng, m, k, n):
    w = rng.normal(0, 1 / np.sqrt(k), (n, k)).astype(np.float32)
    b = rng.normal(0, 1, n).astype(np.float32)
    return np.concatenate([w.ravel(), b]), w, b


# each tile of the forward kernels, by the name that must appear: the ones that are
# done again lie among ones that stay ordinary
SHAPES = [(70, 203, 150, "64x64"), (300, 96, 2500, "64x64"), (4352, 64, 4352, "128x128"),
          (4096, 1024, 4096, "256x256")]


@pytest.mark.parametrize("m,k,n,tile", SHAPES)
def test_operands_past_bf16(m, k, n, tile):
    """Infinities, NaN, values that round to infinity in bf16 and a row of values
    near 1e-36 give what fp32 arithmetic gives: relu of the fp64 sums, to the
    bound of an fp32 sum of k products, and the same infinities and NaN.  (The
    full range of small operands is in test_gpu_parts.py.)"""
    rng = np.random.default_rng(m + k + n)
    theta, w, b = _single_layer(rng, m, k, n)
    X = rng.uniform(-1, 1, (m, k)).astype(np.float32)
    big = np.float32(3.4e38)
    X[1, 5] = np.inf
    X[2, 6] = -np.inf
    X[3, 7] = np.nan
    X[4, :] = 0
    X[4, 8] = big                      # finite, but bf16(x) is infinite
    X[5, :] *= np.float32(1e-36)
    X[6, 9], X[6, 10] = np.inf, -np.inf
    note(f"operands past bf16 m={m} k={k} n={n}")
    with GpuNet((k, n), ("relu",), theta) as net:
        net.nf.nf_profile(net.h, 1)
        out = net.forward(to_dev(X)).astype(np.float64)
        names = {q["name"] for q in net.nf.nf_profile_read(net.h)}
        net.nf.nf_profile(net.h, 0)
        assert f"wide_fwd_out_{tile}" in names, names
        # without the biases the tiny row is not absorbed
        theta0 = np.concatenate([w.ravel(), np.zeros(n, np.float32)])
        net.nf.nf_set_params(net.h, theta0)
        out0 = net.forward(to_dev(X[5:6])).astype(np.float64)
    with np.errstate(all="ignore"):
        X64, W64 = X.astype(np.float64), w.astype(np.float64)
        Z = X64 @ W64.T + b
        # 0 * inf terms are NaN in any order
        ref = np.where(Z > 0, Z, 0.0)
        # the library's relu: z > 0 ? z : 0, so NaN pre-activations give 0
        bound = (k + 2) * 2.0 ** -24 * (np.abs(X64) @ np.abs(W64).T + np.abs(b))
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(out), fin)
    assert np.array_equal(out[~fin], ref[~fin])
    ok = fin & np.isfinite(bound)
    assert np.all(np.abs(out[ok] - ref[ok]) <= bound[ok])
    ref0 = np.maximum(X64[5:6] @ W64.T, 0)
    bound0 = (k + 2) * 2.0 ** -24 * (np.abs(X64[5:6]) @ np.abs(W64).T) + 2.0 ** -149
    assert np.all(np.abs(out0 - ref0) <= bound0)


def test_not_finite_in_training():
    """A step on a batch with an infinite input leaves the tendencies the
    reference's infinities and NaN, and no others."""
    dims, acts, batch = (130, 200, 140), ("gaussian", "sigmoid"), 200
    theta, X, Y = _problem(dims, 11, batch)
    X[17, 3] = np.inf                  # gaussian(+-inf) = 0, f' = NaN
    note("training with an infinite input")
    with np.errstate(all="ignore"):
        _, G = mlp.train_batch(theta, dims, list(acts), X, Y, 0.5, 1)
    with GpuNet(dims, acts, theta) as net:
        net.train_batch(to_dev(X), to_dev(Y), 0.5)
        g = net.grads().astype(np.float64)
    assert np.array_equal(np.isnan(g), np.isnan(G))
    k = dims[1] * dims[0] + dims[1]
    assert not parity.check_grads(np.concatenate([np.zeros(k), g[k:]]),
                                  np.concatenate([np.zeros(k), G[k:]]), dims)
