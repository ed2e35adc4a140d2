"""Complex factors on dimensions of up to 64 points, in which the batched products
contract one to four tiles of 16 digits."""
import os

import numpy as np
import pytest

from oracle.oracle import Oracle
from workloads import card, random_complex

pytestmark = pytest.mark.gpu

# (PPQ_GRID, PPQ_BATCH): a pass per factor, batched passes, grid vectors
PASSES, BATCH, GRID = ("0", "0"), ("0", "2"), ("2", "0")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "needs a GPU"
    return t


def propagator(cd, form, prec, torch):
    import paper_1606_04004_amd as ppq
    names = ("PPQ_GRID", "PPQ_BATCH")
    old = [os.environ.get(k) for k in names]
    os.environ.update(zip(names, form))
    try:
        return ppq.Propagator(cd, precision=prec, device=0, stream=torch.cuda.current_stream())
    finally:
        for k, v in zip(names, old):
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


def dense_card(n):
    """Every kind of term on the dimensions of n: two dense factors (sharing one), one
    with a diagonal factor, three dense, a complex diagonal one."""
    rng = np.random.default_rng(17)

    def dense(k, kind):
        m = 0.2 / np.sqrt(n[k]) * (rng.standard_normal((n[k], n[k])) + 1j * rng.standard_normal((n[k], n[k])))
        f = {"dim": k, "kind": "dense", "re": m.real.tolist()}
        return dict(f, im=m.imag.tolist()) if kind == "complex" else f

    d0, d1, d2 = dense(0, "complex"), dense(1, "real"), dense(2, "complex")
    q = {"dim": 1, "kind": "power", "p": 1}
    cd = card("small_3d", n=n)
    cd["terms"] = cd["terms"] + [
        {"coef": 0.3, "coef_im": 0.1, "factors": [d0, d2]}, {"coef": -0.2, "factors": [d1, d2]},
        {"coef": 0.4, "factors": [d0, q]}, {"coef": 0.5, "factors": [d0, d1, d2]},
        {"coef": 0.1, "coef_im": -0.2, "factors": [q]}]
    return cd


def lattice_card(n, lattice):
    base = card(f"small_{len(n)}d", n=n)
    return dict(base, basis="pvb", lattice=lattice, lo=[-9.0] * len(n), hi=[9.0] * len(n))


CARDS = {
    "64x5x33": dense_card([64, 5, 33]), "50x17x9": dense_card([50, 17, 9]), "16x48x49": dense_card([16, 48, 49]),
    "lattice 64x64": lattice_card([64, 64], [8, 8]), "lattice 56x64": lattice_card([56, 64], [[7, 8], [8, 8]]),
}


@pytest.mark.parametrize("name", list(CARDS))
@pytest.mark.parametrize("form", [PASSES, BATCH, GRID])
@pytest.mark.parametrize("fill", [1.0, 0.2])
def test_product(name, form, fill, torch):
    """FP64 within 1e-13 of the oracle's largest entry (1e-12 on the lattices, whose
    factors carry the condition of the lattice's overlap), FP32 within 1e-5 (a few
    hundred roundings of 2^-24 of the largest partial sum); full fibers and sets of a
    fifth of the functions."""
    cd = CARDS[name]
    total = int(np.prod(cd["n"]))
    keys = np.sort(np.random.default_rng(4).choice(total, size=int(fill * total), replace=False)).astype(np.uint64)
    x = random_complex(keys.size, 6)
    ref = Oracle(cd).apply_def(keys, x)
    for prec, tol in ((0, 1e-12 if "lattice" in name else 1e-13), (1, 1e-5)):
        print(f"{name} {form} precision {prec}: {keys.size} functions", flush=True)
        g = propagator(cd, form, prec, torch)
        g.set_state(keys, x)
        xt = torch.from_numpy(x.astype(np.complex64) if prec else x).cuda()
        yt = torch.full_like(xt, 7.0)
        g.apply_h(xt, yt)
        torch.cuda.synchronize()
        assert np.max(np.abs(yt.cpu().numpy() - ref)) < tol * np.max(np.abs(ref))


@pytest.mark.parametrize("name", ["64x5x33", "lattice 64x64"])
@pytest.mark.parametrize("form", [BATCH, GRID])
def test_arnoldi_step(name, form, torch):
    """One Arnoldi step of order 6 on a third of the functions: within 1e-12 of the
    oracle's (1e-11 on the lattice), relative to the state's norm."""
    cd = CARDS[name]
    total = int(np.prod(cd["n"]))
    keys = np.sort(np.random.default_rng(8).choice(total, size=total // 3, replace=False)).astype(np.uint64)
    c = random_complex(keys.size, 9)
    c = c / np.linalg.norm(c)
    o = Oracle(cd)
    o.set_state(keys, c)
    g = propagator(cd, form, 0, torch)
    g.set_state(keys, c)
    g.step(dt=0.002, m=6)
    o.sil_step(dt=0.002, m=6)
    _, cg = g.state()
    _, co = o.state()
    err = np.linalg.norm(cg - co) / np.linalg.norm(co)
    print(f"{name} {form}: {err:.1e}", flush=True)
    assert err < (1e-11 if "lattice" in name else 1e-12)
