"""Fiber tables of grids whose last dimensions are short: from rotated bitmaps or by
tiles, as the rule has it for a set's size, and by tiles where memory is refused."""
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


def propagator(n, torch, **env):
    saved = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        import paper_1606_04004_amd as ppq
        return ppq.Propagator(shape(n), device=0, stream=torch.cuda.current_stream())
    finally:
        for k, v in saved.items():
            os.environ.pop(k) if v is None else os.environ.update({k: v})


def some_keys(n, count):
    """Points spread over the grid, a crowd in its middle, both ends of the bitmap."""
    total = int(np.prod(n))
    ends = np.arange(min(70, total // 4))
    rng = np.random.default_rng(count)
    return np.unique(np.concatenate([rng.integers(0, total, count // 2), rng.integers(total // 2, min(total // 2 + 2 * count, total), count // 2),
                                     ends, total - 1 - ends])).astype(np.uint64)


def fibers(n, keys):
    strides = [int(np.prod(n[k + 1:])) for k in range(len(n))]
    k64 = keys.astype(np.int64)
    return [np.unique(k64 - k64 // s % nk * s).size for s, nk in zip(strides, n)]


def product(g, keys, x, torch):
    g.set_state(keys, x)
    xt = torch.from_numpy(x).cuda()
    yt = torch.zeros_like(xt)
    g.apply_h(xt, yt)
    torch.cuda.synchronize()
    return yt.cpu().numpy()


# 17M tiles over 2.4M words; 5.3M over 1.0M; 2.7M over 1.4M, where sets of more than 84K functions go by tiles; 7x5x3x3, by tiles
@pytest.mark.parametrize("n,counts", [([64, 64, 64, 64, 3, 3], (4000, 60, 5000)), ([32, 32, 32, 32, 4, 4, 4], (3000, 4000)),
                                      ([40, 40, 40, 40, 12, 3], (4000, 200000, 3000)), ([7, 5, 3, 3], (100, 40))])
@pytest.mark.parametrize("batch", ["0", "2"])
def test_tables(n, counts, batch, torch):
    """One context's sets in turn: as many fibers of every dimension as the keys have,
    products within 1e-13 of the oracle's largest entry."""
    g = propagator(n, torch, PPQ_GRID="0", PPQ_BATCH=batch)
    for count in counts:
        keys = some_keys(n, count)
        x = random_complex(keys.size, 2)
        print(f"{n}: {keys.size} functions, batch {batch}", flush=True)
        y = product(g, keys, x, torch)
        assert g.fiber_counts().tolist() == fibers(n, keys)
        ref = Oracle(shape(n)).apply_def(keys, x)
        assert np.max(np.abs(y - ref)) < 1e-13 * np.max(np.abs(ref))


def test_refused(torch):
    """Any one allocation refused: the call that needed it fails or does without, and
    the products that follow are the same bits (the tables are the same)."""
    from paper_1606_04004_amd import PPQError
    n = [64, 64, 64, 64, 3, 3]
    keys = some_keys(n, 4000)
    x = random_complex(keys.size, 2)
    ref = product(propagator(n, torch, PPQ_GRID="0", PPQ_BATCH="0"), keys, x, torch)
    done = 0
    for k in range(40):
        g = propagator(n, torch, PPQ_GRID="0", PPQ_BATCH="0", PPQ_ALLOC_FAIL=str(k))
        try:
            y = product(g, keys, x, torch)
            done += 1
        except PPQError:
            y = product(g, keys, x, torch)
        assert np.array_equal(y, ref), f"allocation {k}"
    print(f"{done} of 40 without a failure", flush=True)
