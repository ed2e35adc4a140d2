"""Products on grid vectors (PPQ_GRID) and batched on fiber tables (PPQ_BATCH)
against the oracle, beside a pass per factor, at the sizes where a tile of points
or digits, a slice of digits or a stage of factors ends, over every kind of factor
the operator has."""
import os

import numpy as np
import pytest

from oracle.oracle import Oracle
from workloads import card, random_active_set, random_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "needs a GPU"
    return t


# (PPQ_GRID, PPQ_BATCH): a pass per factor on fiber tables, batched passes, grid vectors, the default
PASSES, BATCH, GRID, DEFAULT = ("0", "0"), ("0", "2"), ("2", "0"), ("1", "1")


def propagator(cd, torch, form, precision=0):
    import paper_1606_04004_amd as ppq
    names = ("PPQ_GRID", "PPQ_BATCH")
    old = [os.environ.get(k) for k in names]
    os.environ.update(zip(names, form))
    try:
        return ppq.Propagator(cd, precision=precision, device=0, stream=torch.cuda.current_stream())
    finally:
        for k, v in zip(names, old):
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


def product(g, x, torch):
    xt = torch.from_numpy(x).cuda()
    yt = torch.full_like(xt, 7.0)
    g.apply_h(xt, yt)
    torch.cuda.synchronize()
    return yt.cpu().numpy()


def cards():
    many = card("small_3d")
    # more factors than one launch takes: 20 complex-weighted one-factor terms
    rng = np.random.default_rng(5)
    many["terms"] = many["terms"] + [
        {"coef": 0.1, "coef_im": 0.05, "factors": [{"dim": i % 3, "kind": "dense",
         "re": (0.1 * rng.standard_normal((many["n"][i % 3],) * 2)).tolist()}]} for i in range(20)]
    return {
        "small_2d": card("small_2d"), "small_3d": card("small_3d"), "small_4d": card("small_4d"),
        "small_6d": card("small_6d"), "sop3d": card("sop3d"), "many": many,
        "pvb4d": dict(card("small_4d", n=[12] * 4), basis="pvb", lattice=[3, 4]),
        "pw3d": dict(card("small_3d", n=[12, 12, 12]), basis="pw", lattice=[3, 4]),
        "long": dict(card("small_3d", n=[65, 3, 70])), "two": dict(card("small_2d", n=[2, 3])),
        "max": dict(card("small_2d", n=[256, 17])),
        # window widths of one to four tiles, columns in runs that are no multiples of 16
        "grid48": dict(card("small_2d", n=[48, 47])), "grid64": dict(card("small_3d", n=[64, 5, 33])),
    }


@pytest.mark.parametrize("name,count", [
    ("small_2d", 1), ("small_2d", 63), ("small_2d", 64), ("small_2d", 65), ("small_3d", 129), ("small_3d", 990),
    ("small_4d", 2000), ("small_4d", 10000), ("small_6d", 40000), ("grid48", 2000), ("grid64", 4000), ("sop3d", 500), ("sop3d", 64), ("many", 300), ("pvb4d", 3000),
    ("pw3d", 700), ("long", 5000), ("two", 6), ("max", 3000)])
def test_product_matches_oracle_and_fibers(name, count, torch):
    """FP64 within 1e-13 of the oracle's largest entry (sums of at most a few
    hundred products), the FP32 form within 4e-6 (a few hundred roundings of
    2^-24 of the largest partial sum); NaN and infinite inputs stay on the
    functions coupled to them."""
    cd = cards()[name]
    total = int(np.prod(cd["n"]))
    rng = np.random.default_rng(count)
    keys = np.sort(rng.choice(total, size=count, replace=False)).astype(np.uint64)
    x = random_complex(count, 3)
    ref = Oracle(cd).apply_def(keys, x)
    scale = np.max(np.abs(ref))
    print(f"{name}: {count} functions", flush=True)
    for prec, tol in ((0, 1e-13), (1, 4e-6)):
        xp = x if prec == 0 else x.astype(np.complex64)
        for form in (PASSES, BATCH, GRID):
            g = propagator(cd, torch, form, prec)
            g.set_state(keys, x)
            got = product(g, xp, torch)
            assert np.array_equal(got, product(g, xp, torch))
            assert np.max(np.abs(got - ref)) < tol * scale
            if form != PASSES and count > 2:
                # a second set on the same context: nothing of the first is left
                sub = keys[::2].copy()
                g.set_state(sub, x[::2])
                r2 = Oracle(cd).apply_def(sub, np.ascontiguousarray(x[::2]))
                assert np.max(np.abs(product(g, np.ascontiguousarray(xp[::2]), torch) - r2)) < tol * scale
                assert g.fiber_counts().tolist() == [len(Oracle(cd).fiber_ranges(sub, k)) for k in range(cd["D"])]
    bad = x.copy()
    bad[count // 2] = np.nan
    for form in (BATCH, GRID):
        g = propagator(cd, torch, form)
        g.set_state(keys, x)
        hit = ~np.isfinite(product(g, bad, torch))
        assert np.array_equal(hit, ~np.isfinite(Oracle(cd).apply_def(keys, bad)))
        assert np.all(np.isfinite(product(g, x, torch)))


@pytest.mark.parametrize("name,nsteps", [("hh2d", 12), ("sop3d", 8), ("small_4d", 15), ("pvb4d", 4)])
def test_run_crosses_between_forms(name, nsteps, torch):
    """A run on grid vectors, one on fiber tables and the oracle's: the same sets,
    observables within the trajectory bound of 1e-10."""
    cd = cards().get(name) or card(name)
    if name == "pvb4d":
        cd = dict(cd, eps=1e-4, dt=0.05)
    o = Oracle(cd)
    o.init_state()
    ref, _ = o.propagate(nsteps=nsteps)
    ko, co = o.state()
    for form in (PASSES, BATCH, GRID, DEFAULT):
        g = propagator(cd, torch, form)
        g.init_state()
        tr = g.propagate(nsteps=nsteps)
        kg, cg = g.state()
        print(f"{name} {form}: |A| {kg.size}", flush=True)
        assert np.array_equal(kg, ko)
        assert np.max(np.abs(cg - co)) < 1e-10
        assert np.max(np.abs(tr[:, 1:7] - ref[:, 1:7])) < 1e-10 * max(1.0, np.max(np.abs(ref[:, 1:5])))


def test_sets_growing_past_the_rule(torch):
    """A set above the rule's size runs on fiber tables and a smaller one after it
    on grid vectors again; the blob's product matches the oracle each time."""
    cd = card("morse4d")
    g = propagator(cd, torch, DEFAULT)
    o = Oracle(cd)
    for fill, seed in ((0.01, 1), (0.9, 2), (0.02, 3)):
        keys = random_active_set(cd["n"], fill, seed, blob=fill > 0.5)
        x = random_complex(keys.size, seed)
        g.set_state(keys, x)
        idx = np.unique(np.random.default_rng(seed).integers(0, keys.size, 400))
        ref = o.apply_def_at(keys, x, idx)
        y = product(g, x, torch)
        print(f"|A| {keys.size}", flush=True)
        assert np.max(np.abs(y[idx] - ref)) < 1e-13 * np.max(np.abs(ref))
