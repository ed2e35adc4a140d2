"""The passes over one dimension at the sizes where a fiber meets the end of a
64-entry word, a 256-entry tile or a wavefront's rank range, against the oracle."""
import os

import numpy as np
import pytest

from oracle.oracle import Oracle
from workloads import card, random_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "needs a GPU"
    return t


def run(cd, keys, x, prec, env, torch):
    import paper_1606_04004_amd as ppq
    env = {"PPQ_GRID": "0", "PPQ_BATCH": "0", **env}
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        g = ppq.Propagator(cd, precision=prec, device=0, stream=torch.cuda.current_stream())
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v
    g.set_state(keys, np.where(np.isfinite(x), x, 0))
    xt = torch.from_numpy(x.astype(np.complex64) if prec else x).cuda()
    yt = torch.full_like(xt, 7.0)
    g.apply_h(xt, yt)
    torch.cuda.synchronize()
    return yt.cpu().numpy()


# fiber lengths that divide a word, that drift through it, that fill the halo; runs cut by gaps
@pytest.mark.parametrize("n,fill", [([9, 64], 1.0), ([13, 63], 1.0), ([40, 33], 1.0), ([33, 32], 1.0), ([75, 31], 1.0),
                                    ([60, 24], 0.6), ([24, 60], 0.9), ([5, 23, 24], 0.5), ([32, 8], 1.0), ([2, 2], 1.0)])
def test_point_and_lane_passes(n, fill, torch):
    """FP64 within 1e-13 of the oracle's largest entry, FP32 within 4e-6 (at most
    130 products per entry); an infinite input reaches the functions coupled to it
    and no others."""
    cd = card("small_2d" if len(n) == 2 else "small_3d", n=n)
    total = int(np.prod(n))
    rng = np.random.default_rng(total)
    keys = np.sort(rng.choice(total, size=max(1, int(fill * total)), replace=False)).astype(np.uint64)
    x = random_complex(keys.size, 3)
    ref = Oracle(cd).apply_def(keys, x)
    print(f"{n}: {keys.size} functions", flush=True)
    for prec, tol in ((0, 1e-13), (1, 4e-6)):
        for env in ({"PPQ_HPSI": "3"}, {"PPQ_HPSI": "3", "PPQ_ACC_STAGE": "0"}, {}):
            assert np.max(np.abs(run(cd, keys, x, prec, env, torch) - ref)) < tol * np.max(np.abs(ref))
    bad = x.copy()
    bad[keys.size // 2] = np.inf
    hit = ~np.isfinite(Oracle(cd).apply_def(keys, bad))
    assert np.array_equal(~np.isfinite(run(cd, keys, bad, 0, {"PPQ_HPSI": "3"}, torch)), hit)


@pytest.mark.parametrize("count", [2 ** 18, 2 ** 18 + 1, 256 * 33 * 35 - 3])
def test_potential_of_large_sets(count, torch):
    """Sets at and past the size where a thread evaluates several functions, with
    digits up to 255 and terms of one to three factors: the product at sampled
    functions within 1e-13 of the largest (FP32: 2e-5, 324 products of 2^-24)."""
    cd = card("small_3d", n=[256, 33, 35])
    cd["terms"] = cd["terms"] + [{"coef": 0.02, "factors": [{"dim": k, "kind": "power", "p": p} for k, p in ((0, 1), (1, 3), (2, 2))]}]
    rng = np.random.default_rng(count)
    keys = np.sort(rng.choice(256 * 33 * 35, size=count, replace=False)).astype(np.uint64)
    x = random_complex(count, 5)
    at = np.unique(np.concatenate([rng.choice(count, size=400), [0, 1, 255, 256, count - 1]])).astype(np.int64)
    ref = Oracle(cd).apply_def_at(keys, x, at)
    for prec, tol in ((0, 1e-13), (1, 2e-5)):
        got = run(cd, keys, x, prec, {}, torch)[at]
        assert np.max(np.abs(got - ref)) < tol * np.max(np.abs(ref))


# the tables' tiles: fibers below a digit in runs of less than, exactly and more than 64, runs that start
# anywhere in a word, dimensions of 2 to 64 digits; a last dimension of 15 takes the other form
@pytest.mark.parametrize("n,count", [([2, 16], 32), ([64, 64], 4096), ([5, 7, 17], 300), ([9, 4, 16], 576), ([3, 40, 31], 1),
                                     ([3, 64, 48], 4000), ([12, 5, 3, 33], 2500), ([12, 5, 3, 33], 7), ([7, 6, 5, 15], 900),
                                     ([2, 3, 2, 4, 3, 20], 1000)])
def test_fiber_tables(n, count, torch):
    """The products on the tables within 1e-13 of the oracle's largest entry, and
    the fibers of every dimension as many as the oracle's."""
    import paper_1606_04004_amd as ppq
    cd = card(f"small_{len(n)}d", n=n)
    total = int(np.prod(n))
    rng = np.random.default_rng(count)
    keys = np.sort(rng.choice(total, size=count, replace=False)).astype(np.uint64)
    x = random_complex(count, 9)
    o = Oracle(cd)
    ref = o.apply_def(keys, x)
    got = run(cd, keys, x, 0, {}, torch)
    assert np.max(np.abs(got - ref)) < 1e-13 * np.max(np.abs(ref))
    os.environ["PPQ_GRID"] = "0"
    try:
        g = ppq.Propagator(cd, precision=0, device=0, stream=torch.cuda.current_stream())
    finally:
        del os.environ["PPQ_GRID"]
    for ks in (keys, keys[::3].copy()):
        g.set_state(ks, random_complex(ks.size, 2))
        assert g.fiber_counts().tolist() == [len(o.fiber_ranges(ks, k)) for k in range(len(n))]


def test_default_stream_is_in_order(torch):
    """A propagator on torch's default stream takes inputs that are still being
    written there (a few milliseconds of work ahead of the product)."""
    import paper_1606_04004_amd as ppq
    cd = card("small_3d")
    keys = np.arange(int(np.prod(cd["n"])), dtype=np.uint64)
    x = random_complex(keys.size, 1)
    with torch.cuda.stream(torch.cuda.default_stream()):
        g = ppq.Propagator(cd, precision=0, device=0, stream=torch.cuda.current_stream())
        g.set_state(keys, x)
        src = torch.from_numpy(x).cuda()
        xt, yt = torch.zeros_like(src), torch.zeros_like(src)
        g.apply_h(xt, yt)
        torch.cuda.synchronize()
        big = torch.ones(4096, 4096, device="cuda")
        torch.cuda.synchronize()
        for _ in range(20):
            big = big @ big * 1e-4
        xt += src
        g.apply_h(xt, yt)
        torch.cuda.synchronize()
    ref = Oracle(cd).apply_def(keys, x)
    assert np.max(np.abs(yt.cpu().numpy() - ref)) < 1e-13 * np.max(np.abs(ref))


@pytest.mark.parametrize("n", [[64, 64, 64, 64], [2, 2, 64, 64, 64, 17]])
def test_bitmaps_at_the_scan_limit(n, torch):
    """Bitmaps of exactly 2^18 words (one word per thread of the scans) and of more:
    the same sets after an adaption as the oracle's, coefficients carried over bit
    for bit, and products on their tables within 1e-13 of the largest entry."""
    import paper_1606_04004_amd as ppq
    cd = card(f"small_{len(n)}d", n=n)
    total = int(np.prod(n))
    rng = np.random.default_rng(3)
    keys = np.unique(np.concatenate([rng.choice(total, size=1500), np.arange(total // 2, total // 2 + 600), [0, 63, 64, total - 1]])).astype(np.uint64)
    x = random_complex(keys.size, 4)
    o = Oracle(cd)
    o.set_state(keys, x)
    g = ppq.Propagator(cd, precision=0, device=0, stream=torch.cuda.current_stream())
    g.set_state(keys, x)
    eps = float(np.median(np.abs(x)))
    for turn in range(2):
        o.prune(eps)
        g.prune(eps)
        (ko, co), (kg, cg) = o.state(), g.state()
        assert np.array_equal(kg, ko) and np.array_equal(cg, co)
        z = random_complex(ko.size, 6)
        got, ref = run(cd, ko, z, 0, {}, torch), o.apply_def(ko, z)
        assert np.max(np.abs(got - ref)) < 1e-13 * np.max(np.abs(ref))
