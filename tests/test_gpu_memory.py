"""Running out of device memory: any one allocation of a context's work memory may be
refused (PPQ_ALLOC_FAIL makes HIP refuse the k-th), the call that needed it reports
PPQ_E_OOM or does without, and the same call made again gives the same results."""
import os

import numpy as np
import pytest

from workloads import card, random_complex

pytestmark = pytest.mark.gpu

# (PPQ_GRID, PPQ_BATCH): a pass per factor, batched passes, grid vectors
PASSES, BATCH, GRID = ("0", "0"), ("0", "2"), ("2", "0")
E_OOM = -3


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "needs a GPU"
    return t


def propagator(cd, torch, **env):
    import paper_1606_04004_amd as ppq
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        return ppq.Propagator(cd, device=0, stream=torch.cuda.current_stream())
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


class Twice:
    """Calls that are made again, once, when they report that memory ran out."""

    def __init__(self):
        self.failed = []

    def __call__(self, name, f):
        from paper_1606_04004_amd import PPQError
        try:
            return f()
        except PPQError as e:
            assert e.code == E_OOM, f"{name}: {e}"
            self.failed.append(name)
            return f()


def exercise(cd, form, k, torch):
    keys = np.sort(np.random.default_rng(1).choice(int(np.prod(cd["n"])), size=300, replace=False)).astype(np.uint64)
    c = random_complex(keys.size, 2)
    c = c / np.linalg.norm(c)
    g = propagator(cd, torch, PPQ_GRID=form[0], PPQ_BATCH=form[1], PPQ_ALLOC_FAIL=str(k))
    call = Twice()
    call("reserve", lambda: g.reserve(300))
    call("set_state", lambda: g.set_state(keys, c))
    out = []

    def product():
        x = torch.from_numpy(random_complex(g.active_count(), 3)).cuda()
        y = torch.zeros_like(x)
        g.apply_h(x, y)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    out.append(call("product", product))
    call("step", lambda: g.step(dt=0.01, m=6))
    for eps in (1e-4, 1e-3):
        call("prune", lambda: g.prune(eps))
        out.append(call("product", product))
        out.append(call("observables", lambda: np.array([v for v in g.observables().values()])))
        call("step", lambda: g.step(dt=0.01, m=6))
    kg, cg = g.state()
    return out + [kg, cg], call.failed


def terms_card():
    """The small 4D card with two- and three-factor terms: vectors between factors."""
    cd = card("small_4d")
    rng = np.random.default_rng(11)

    def dense(k):
        return {"dim": k, "kind": "dense", "re": (0.1 * rng.standard_normal((cd["n"][k],) * 2)).tolist()}

    cd["terms"] = cd["terms"] + [{"coef": 0.1, "factors": [dense(0), dense(2)]},
                                 {"coef": 0.1, "factors": [dense(0), dense(1), dense(3)]},
                                 {"coef": 0.1, "factors": [dense(1), {"dim": 2, "kind": "power", "p": 1}]}]
    return cd


@pytest.mark.parametrize("name", ["single", "terms"])
@pytest.mark.parametrize("form", [PASSES, BATCH])
def test_any_allocation_may_be_refused(name, form, torch):
    """Against the run that gets all its memory: the same sets, values within 1e-12 of
    the largest (another form of the product, where one was done without, rounds
    differently: 1e-13 a product, two steps of ten).  Growing by adaption is among
    the calls: the state survives a growth that fails."""
    refuse_each(name, form, torch)


def refuse_each(name, form, torch):
    cd = card("small_4d") if name == "single" else terms_card()
    ref, failed = exercise(cd, form, -1, torch)
    assert not failed
    assert ref[-1].size > 1024  # past the smallest capacity: one of the adaptions grows
    seen = set()
    for k in range(110):
        got, failed = exercise(cd, form, k, torch)
        assert len(failed) <= 1
        seen.update(failed)
        assert np.array_equal(got[-2], ref[-2]), f"allocation {k}"
        for a, b in zip(got, ref):
            assert np.max(np.abs(a - b)) < 1e-12 * max(1.0, np.max(np.abs(b))), f"allocation {k}"
    print(f"{name} {form}: refused in {sorted(seen)}", flush=True)
    assert {"reserve", "step", "prune"} <= seen
    return seen


def gradient(k, grid, torch):
    from paper_1606_04004_amd.adjoint import declare_trainable
    cd = card("small_adjoint4d")
    g = propagator(cd, torch, PPQ_GRID=grid, PPQ_ALLOC_FAIL=str(k))
    declare_trainable(g, cd)
    call = Twice()
    j = call("record", lambda: g.adjoint_record(nsteps=3, m=8, every=2))
    return j, call("gradient", g.adjoint_gradient), call.failed


def refuse_each_of_a_gradient(grid, torch):
    j0, g0, failed = gradient(-1, grid, torch)
    assert not failed
    seen = set()
    for k in range(90):
        j, gr, failed = gradient(k, grid, torch)
        seen.update(failed)
        assert abs(j - j0) < 1e-12
        for a, b in zip(gr, g0):
            assert np.max(np.abs(a - b)) < 1e-10 * max(1.0, np.max(np.abs(b)))
    assert seen == {"record", "gradient"}


def test_adjoint_allocations(torch):
    """The recorded run and its gradient likewise (1e-10: the gradient's own bound)."""
    refuse_each_of_a_gradient("0", torch)


@pytest.mark.parametrize("name", ["single", "terms"])
def test_grid_vectors_are_done_without(name, torch):
    """No product fails for want of grid vectors: there the fiber tables serve."""
    assert "product" not in refuse_each(name, GRID, torch)


def test_adjoint_keeps_its_form(torch):
    """A recorded run's steps are recomputed by the form of the product that
    recorded them, with and without its grid vectors."""
    refuse_each_of_a_gradient("2", torch)


def test_adjoint_of_a_higher_order(torch):
    """A gradient of a higher order than the context's first one: the basis of the
    adjoint vectors grows with it, and the gradient is a new context's bit for bit."""
    from paper_1606_04004_amd.adjoint import declare_trainable
    cd = card("small_adjoint4d")

    def gradient(g, m):
        j = g.adjoint_record(nsteps=3, m=m, every=2)
        return [np.array([j]), *g.adjoint_gradient()]

    g, fresh = propagator(cd, torch), propagator(cd, torch)
    for h in (g, fresh):
        declare_trainable(h, cd)
        h.reserve(10 ** 4)
    gradient(g, 8)
    for a, b in zip(gradient(g, 16), gradient(fresh, 16)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("name", ["single", "terms"])
def test_batched_vectors_are_done_without(name, torch):
    """With the fiber tables there, no product fails for want of the batched form's
    vectors: a pass per factor serves, and goes on serving (the same bits)."""
    cd = card("small_4d") if name == "single" else terms_card()
    keys = np.arange(0, 10 ** 4, 3, dtype=np.uint64)
    x = random_complex(keys.size, 3)
    results = []
    for k in [-1, *range(60)]:
        g = propagator(cd, torch, PPQ_GRID="0", PPQ_ALLOC_FAIL=str(k))
        call = Twice()
        call("set_state", lambda: g.set_state(keys, x))
        call("tables", g.fiber_counts)
        xt = torch.from_numpy(x).cuda()
        ys = []
        for _ in range(3):
            yt = torch.zeros_like(xt)
            call("product", lambda: g.apply_h(xt, yt))
            torch.cuda.synchronize()
            ys.append(yt.cpu().numpy())
        assert "product" not in call.failed, f"allocation {k}"
        assert np.array_equal(ys[0], ys[1]) and np.array_equal(ys[0], ys[2]), f"allocation {k}"
        results.append(ys[0])
        assert np.max(np.abs(ys[0] - results[0])) < 1e-12 * np.max(np.abs(results[0]))
    # some of the refusals led to the other form, whose sums round differently
    assert any(not np.array_equal(r, results[0]) for r in results)


def test_batched_vectors_have_the_size_of_the_rule(torch):
    """Fifteen three-factor terms with 30 vectors between their factors, on a context
    that reserves eight million functions: the batched product takes at most 2 GiB."""
    n = [64, 64, 64, 64]
    cd = card("small_4d", n=n)
    rng = np.random.default_rng(2)
    m = [(0.1 * rng.standard_normal((64, 64))).tolist() for _ in range(4)]
    cd["terms"] = cd["terms"] + [{"coef": 0.1 + 0.01 * i, "factors": [{"dim": k, "kind": "dense", "re": m[k]} for k in range(4) if k != i % 4]}
                                 for i in range(15)]
    g = propagator(cd, torch, PPQ_GRID="0")
    g.reserve(8_000_000)
    keys = np.arange(0, 64 ** 4, 9973, dtype=np.uint64)
    x = random_complex(keys.size, 3)
    g.set_state(keys, x)
    g.fiber_counts()
    xt = torch.from_numpy(x).cuda()
    yt = torch.zeros_like(xt)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    g.apply_h(xt, yt)
    torch.cuda.synchronize()
    taken = free - torch.cuda.mem_get_info()[0]
    print(f"{taken / 2 ** 30:.2f} GiB", flush=True)
    assert taken < 2.1 * 2 ** 30
