"""The tendencies of several layers in one launch and deltas split over a long
range of units: more layers than a launch holds, layers with and without
pieces side by side, unaligned inputs beside aligned layers, both precisions."""

import numpy as np
import pytest

from oracle import mlp

from . import parity
from .gpu_run import GpuNet, note, to_dev
from .test_gpu_parity import _compare_trajectory, _problem

pytestmark = pytest.mark.gpu

CASES = [
    # dims, acts, batch, kernels that must appear
    ((37, 130, 40, 35, 33, 9, 10, 3), ("tanh",), 5, ("wide_dw_sgd",)),   # seven layers: two launches
    ((300, 400, 700, 260, 5), ("tanh",), 33, ("wide_bwd_piece", "bwd_fold")),
    ((64, 513, 1031, 7), ("sigmoid",), 17, ("wide_bwd_piece", "bwd_fold")),
    ((20, 3000, 2900, 12), ("tanh", "tanh", "sigmoid"), 600, ("wide_dw_sgd", "wide_dw_partial")),   # one piece and several
]


@pytest.mark.parametrize("dims,acts,batch,kernels", CASES)
def test_grouped_steps(dims, acts, batch, kernels):
    theta, X, Y = _problem(dims, sum(dims) + batch, 2 * batch)
    _compare_trajectory(dims, acts, theta, X, Y, batch, 0.2, 1, 2)
    with GpuNet(dims, acts, theta) as net:
        net.nf.nf_profile(net.h, 1)
        net.train_batch(to_dev(X[:batch]), to_dev(Y[:batch]), 0.2)
        names = [k["name"] for k in net.nf.nf_profile_read(net.h)]
        net.nf.nf_profile(net.h, 0)
    for want in kernels:
        assert any(n.startswith(want) for n in names), names


@pytest.mark.parametrize("dims,acts,batch,kernels", CASES[:3])
def test_grouped_steps_f64(dims, acts, batch, kernels):
    import torch
    from paper_1902_06714_amd import nf
    theta, X, Y = _problem(dims, sum(dims) + batch, batch)
    note(f"grouped fp64 dims={dims} batch={batch}")
    net = nf.nf_net_create(dims, list(acts), nf.NF_F64)
    try:
        nf.nf_set_params_f64(net, theta.astype(np.float64))
        nf.nf_train_batch_f64(net, torch.from_numpy(X).double().cuda(),
                              torch.from_numpy(Y).double().cuda(), 0.2)
        p, g = nf.nf_get_params_f64(net), nf.nf_get_grads_f64(net)
    finally:
        nf.nf_net_destroy(net)
    ref, G = mlp.train_batch(theta.astype(np.float64), dims, parity.full_acts(dims, acts),
                             X, Y, 0.2, 1, precision="f64")
    # sums of at most 1100 products, each side within 1100 2^-53 of exact, through every layer
    bound = 2 * len(dims) * 1100 * 2.0 ** -53
    for got, want in ((p, ref), (g, G)):
        rms = np.sqrt(np.mean(np.asarray(want) ** 2))
        assert np.max(np.abs(got - want) / np.maximum(np.abs(want), rms)) < bound
