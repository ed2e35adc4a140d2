"""Krylov steps on sets with more than a million fibers of the first dimension, whose
pass leaves more partial sums of <x|y> than a sweep has values."""
import os

import numpy as np
import pytest

from oracle.oracle import Oracle
from workloads import random_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "needs a GPU"
    return t


def shape(n):
    D = len(n)
    terms = [{"coef": 0.5, "factors": [{"dim": k, "kind": "power", "p": 2}]} for k in range(D)]
    return {"name": "shape", "D": D, "n": n, "lo": [-4.0] * D, "hi": [4.0] * D, "mass": 1.0, "terms": terms, "basis": "dvr",
            "psi0": {"centre": [0.0] * D, "momentum": [0.0] * D, "width": [0.7] * D},
            "eps": 1e-5, "dt": 0.02, "nsteps": 5, "krylov": 10}


@pytest.mark.parametrize("count", [4096 * 256, 4096 * 256 + 1, 64 * 64 * 64 * 5 + 70000])
def test_step_with_many_partial_sums(count, torch):
    """The 4096 blocks of 256 fibers, one more, and all fibers of the grid with a few
    second members: a step of order 4 within 1e-13 of the oracle's (a few units of
    2^-53 per application of dt H, whose norm is below 100)."""
    import paper_1606_04004_amd as ppq
    cd = shape([2, 64, 64, 64, 5])
    keys = np.arange(count, dtype=np.uint64)
    c = random_complex(count, 3)
    c = c / np.linalg.norm(c)
    os.environ["PPQ_BATCH"] = "0"
    try:
        g = ppq.Propagator(cd, device=0, stream=torch.cuda.current_stream())
    finally:
        del os.environ["PPQ_BATCH"]
    g.set_state(keys, c)
    g.step(dt=0.002, m=4)
    assert g.fiber_counts()[0] == min(count, 64 * 64 * 64 * 5)
    o = Oracle(cd)
    o.set_state(keys, c)
    o.sil_step(dt=0.002, m=4)
    _, cg = g.state()
    _, co = o.state()
    assert np.linalg.norm(cg - co) < 1e-13 * np.linalg.norm(co)
