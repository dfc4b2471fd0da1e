"""Input rows that are not whole 16-byte vectors: odd widths and rows that
start off a 16-byte boundary, through the narrow kernels, the skinny forward
and tendency kernels and the medium inference.  The last row ends at the end of
the tensor, and no value of a row may reach its neighbour."""

import numpy as np
import pytest

from oracle import mlp

from . import parity
from .gpu_run import GpuNet, note, to_dev
from .test_gpu_parity import _compare_trajectory, _problem

pytestmark = pytest.mark.gpu

# dims, acts, batch, shards, kernels of the training step, of inference
CASES = [
    ((5, 3), ("sigmoid",), 7, 1, ("narrow_fwd4_train",), "narrow_fwd4_infer"),
    ((61, 17, 2), ("tanh", "sigmoid"), 33, 1, ("narrow_fwd4_train",), "narrow_fwd4_infer"),
    ((65, 32, 31, 4), ("gaussian", "tanh", "sigmoid"), 129, 1, ("narrow_fwd4_train",), "narrow_fwd4_infer"),
    ((785, 30, 10), ("sigmoid",), 1000, 1, ("narrow_fwd4_train",), "narrow_fwd4_infer"),
    ((1027, 12, 10), ("tanh", "sigmoid"), 2049, 1, ("narrow_fwd16_train",), "narrow_fwd16_infer"),
    ((7, 32, 32, 32, 32), ("sigmoid",), 2065, 1, ("narrow_fwd16_train",), "narrow_fwd16_infer"),
    ((33, 40, 10), ("tanh", "sigmoid"), 1, 1, ("fwd_skinny",), "medium_infer"),
    ((129, 77, 33, 5), ("gaussian", "tanh", "sigmoid"), 2049, 1, ("fwd_skinny", "dw_skinny"), "medium_infer"),
    ((785, 100, 100, 10), ("tanh", "tanh", "sigmoid"), 1600, 16, ("fwd_skinny", "dw_skinny"), "medium_infer"),
    ((111, 128, 16, 7, 3), ("tanh",), 1000, 4, ("fwd_skinny", "dw_skinny"), "medium_infer"),
    ((2050, 113, 9), ("tanh", "sigmoid"), 515, 5, ("fwd_skinny", "dw_skinny"), "medium_infer"),
    ((784, 100, 30), ("sigmoid",), 6001, 1, ("fwd_skinny", "dw_skinny"), "medium_infer"),
    # the last batch of the narrow step and the first past it
    ((29, 26, 16), ("tanh", "sigmoid"), 3000, 1, ("narrow_fwd16_train",), "narrow_fwd16_infer"),
    ((29, 26, 16), ("tanh", "sigmoid"), 3001, 1, ("fwd_skinny", "dw_skinny"), "narrow_fwd16_infer"),
    ((29, 26), ("sigmoid",), 3001, 1, ("dw_skinny",), "narrow_fwd16_infer"),
    # much of more than 96 units: the wide tendencies beside the skinny ones
    ((1961, 97, 5), ("tanh", "sigmoid"), 5265, 5, ("fwd_skinny", "wide_dw_partial_128x128", "dw_skinny"),
     "medium_infer"),
    # inference layer by layer
    ((255, 97, 3), ("tanh", "sigmoid"), 12000, 1, ("fwd_skinny",), "wide_fwd_out_64x64"),
    ((255, 97, 3), ("tanh", "sigmoid"), 11999, 1, ("fwd_skinny",), "medium_infer"),
    ((255, 96, 3), ("tanh", "sigmoid"), 12000, 1, ("fwd_skinny",), "medium_infer"),
    ((31, 65, 3), ("tanh", "sigmoid"), 12000, 1, ("fwd_skinny",), "wide_fwd_out_64x64"),
    ((33, 65, 3), ("tanh", "sigmoid"), 12000, 1, ("fwd_skinny",), "medium_infer"),
    ((1501, 97, 3), ("tanh", "sigmoid"), 256, 1, ("fwd_skinny",), "wide_fwd_out_64x64"),
    ((1501, 97, 3), ("tanh", "sigmoid"), 257, 1, ("fwd_skinny",), "medium_infer"),
    ((1501, 96, 3), ("tanh", "sigmoid"), 256, 1, ("fwd_skinny",), "medium_infer"),
]


@pytest.mark.parametrize("dims,acts,batch,shards,train,infer", CASES)
def test_odd_rows(dims, acts, batch, shards, train, infer):
    theta, X, Y = _problem(dims, 13 * sum(dims) + batch, 2 * batch)
    _compare_trajectory(dims, acts, theta, X, Y, batch, 0.3, shards, 2)
    ref = mlp.output(theta.astype(np.float64), dims, parity.full_acts(dims, acts), X[:batch])
    with GpuNet(dims, acts, theta) as net:
        net.nf.nf_profile(net.h, 1)
        out = net.forward(to_dev(X[:batch]))
        ran = {k["name"] for k in net.nf.nf_profile_read(net.h)}
        # the same rows from an address that is 4 bytes past a 16-byte boundary
        flat = to_dev(np.concatenate([[0.0], X[:batch].ravel()]))
        off = net.forward(flat[1:].view(batch, dims[0]))
        net.nf.nf_profile_read(net.h)
        net.train_batch(to_dev(X[:batch]), to_dev(Y[:batch]), 0.3, shards)
        trained = {k["name"] for k in net.nf.nf_profile_read(net.h)}
        net.nf.nf_profile(net.h, 0)
    # an fp32 sum of at most 2050 products of values below 1, through at most
    # four layers of slope at most 1
    assert np.max(np.abs(out - ref)) < 2e-5
    assert np.max(np.abs(off - ref)) < 2e-5
    assert infer in ran, ran
    assert all(k in trained for k in train), trained


@pytest.mark.parametrize("dims,batch", [((61, 17, 2), 33), ((1027, 12, 10), 2049), ((129, 77, 33, 5), 40),
                                        ((785, 100, 10), 130)])
def test_rows_do_not_leak(dims, batch):
    """A row of NaN leaves the rows before and after it as they were."""
    theta, X, _ = _problem(dims, 7 * sum(dims), batch)
    with GpuNet(dims, ("sigmoid",), theta) as net:
        clean = net.forward(to_dev(X))
        bad = np.arange(1, batch, 5)
        X[bad] = np.nan
        out = net.forward(to_dev(X))
    note(f"row leak dims={dims} batch={batch}")
    rest = np.setdiff1d(np.arange(batch), bad)
    assert np.isnan(out[bad]).all()
    assert np.max(np.abs(out[rest] - clean[rest])) < 2e-5
