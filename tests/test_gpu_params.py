"""Parameters through the pinned slots: every element lands where it came from,
whatever the parts' lengths and wherever the slots and launches are cut."""

import numpy as np
import pytest

from .gpu_run import note

pytestmark = pytest.mark.gpu

NETS = [
    (3, 2),                      # 8 elements
    (1, 1, 1, 1, 1, 1),          # parts of one element
    (5,) * 41,                   # 80 parts: several launches of at most 16
    (784, 30, 10),               # padded layout
    (512, 511, 3),               # one slot and a little (fp32: 262144 elements a slot)
    (511, 513),                  # a slot's end inside a row
    (1023, 1025, 2049, 7),       # more slots than threads
]


@pytest.mark.parametrize("dims", NETS)
@pytest.mark.parametrize("f64", [False, True])
def test_round_trip(dims, f64):
    from paper_1902_06714_amd import nf
    note(f"parameter round trip dims={dims[:4]} f64={f64}")
    net = nf.nf_net_create(dims, "sigmoid", nf.NF_F64 if f64 else nf.NF_F32)
    put, get = ((nf.nf_set_params_f64, nf.nf_get_params_f64) if f64
                else (nf.nf_set_params, nf.nf_get_params))
    try:
        n = nf.nf_param_count(net)
        theta = (np.arange(n) + 1).astype(np.float64 if f64 else np.float32)
        for scale in (1, -3):
            put(net, scale * theta)
            assert np.array_equal(get(net), scale * theta)
    finally:
        nf.nf_net_destroy(net)


def test_shared_slots():
    """Nets share the slots: several threads at a time, more of them than slots,
    and nets that come after the last one has given them back."""
    import threading
    from paper_1902_06714_amd import nf
    wrong = []

    def work(k):
        dims = [(1023, 1025, 7), (33, 5), (2049, 513, 2), (700, 700)][k % 4]
        net = nf.nf_net_create(dims, "sigmoid")
        try:
            n = nf.nf_param_count(net)
            theta = np.random.default_rng(k).normal(size=n).astype(np.float32)
            for i in range(6):
                nf.nf_set_params(net, theta + np.float32(i))
                if not np.array_equal(nf.nf_get_params(net), theta + np.float32(i)):
                    wrong.append((k, i))
        finally:
            nf.nf_net_destroy(net)

    for rounds in range(3):
        note(f"shared slots, round {rounds}")
        threads = [threading.Thread(target=work, args=(k,)) for k in range(12)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    assert not wrong
