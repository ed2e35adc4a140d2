"""Product terms of the single-precision form: coefficients and diagonal factors act
in FP64 in every form of the product, and a result is rounded once."""
import os

import numpy as np
import pytest

from workloads import card, random_complex

pytestmark = pytest.mark.gpu

# (PPQ_GRID, PPQ_BATCH): batched passes, grid vectors, the default
BATCH, GRID, DEFAULT = ("0", "2"), ("2", "0"), ("1", "1")
HALF_ULP = 2.0 ** -24


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "needs a GPU"
    return t


def apply32(cd, form, keys, x, torch):
    import paper_1606_04004_amd as ppq
    names = ("PPQ_GRID", "PPQ_BATCH")
    old = [os.environ.get(k) for k in names]
    os.environ.update(zip(names, form))
    try:
        g = ppq.Propagator(cd, precision=1, device=0, stream=torch.cuda.current_stream())
    finally:
        for k, v in zip(names, old):
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v
    g.set_state(keys, x.astype(np.complex128))
    xt = torch.from_numpy(x).cuda()
    yt = torch.zeros_like(xt)
    g.apply_h(xt, yt)
    torch.cuda.synchronize()
    return yt.cpu().numpy()


def bare(n, term):
    """A card whose only operator is the term: zero kinetic matrices, no potential."""
    D = len(n)
    return dict(card(f"small_{D}d", n=n), terms=[term], dim_factors={k: np.zeros((n[k], n[k])).tolist() for k in range(D)})


def identity(k, n):
    return {"dim": k, "kind": "dense", "re": np.eye(n[k]).tolist()}


@pytest.mark.parametrize("form", [BATCH, GRID, DEFAULT])
@pytest.mark.parametrize("kind", ["diagonal", "constant", "one dense", "one dense, real", "two dense", "three dense"])
@pytest.mark.parametrize("n", [[9, 11, 10], [64, 5, 33]])
def test_a_term_is_rounded_once(n, kind, form, torch):
    """A term whose dense factors are identities: coefficient times D(I) times x_I.
    With x exact in FP32, one rounding of the FP64 product leaves each part of the
    result within 2^-24 of its exact value, relative to itself (and a few roundings
    of 2^-53 of the larger part, of the reference and of the FP64 product)."""
    q = [{"dim": 0, "kind": "power", "p": 3}, {"dim": 1, "kind": "power", "p": 1}]
    coef = 0.1 + 1.0 / 3.0 * 1j
    factors = {"diagonal": q, "constant": [], "one dense": [q[0], identity(1, n)], "one dense, real": [q[0], identity(1, n)],
               "two dense": [identity(0, n), identity(2, n)],
               "three dense": [identity(0, n), identity(1, n), identity(2, n)]}[kind]
    if kind == "one dense, real":
        coef = complex(coef.real)
    cd = bare(n, {"coef": coef.real, "coef_im": coef.imag, "factors": factors})
    total = int(np.prod(n))
    keys = np.sort(np.random.default_rng(1).choice(total, size=total * 2 // 3, replace=False)).astype(np.uint64)
    x = random_complex(keys.size, 3).astype(np.complex64)
    digit = np.unravel_index(keys.astype(np.int64), n)
    d = np.ones(keys.size)
    for f in factors:
        if f["kind"] == "power":
            k = f["dim"]
            lo, hi = cd["lo"][k], cd["hi"][k]
            d = d * (lo + (digit[k] + 1) * (hi - lo) / (n[k] + 1)) ** f["p"]
    ref = coef * d * x.astype(np.complex128)
    got = apply32(cd, form, keys, x, torch).astype(np.complex128)
    slack = 2.0 ** -48 * np.abs(ref)
    print(f"{kind} {n} {form}: {np.max(np.abs(got - ref) / np.maximum(np.abs(ref), 1e-300)) / HALF_ULP:.2f} x 2^-24", flush=True)
    assert np.all(np.abs(got.real - ref.real) <= HALF_ULP * np.abs(ref.real) + slack)
    assert np.all(np.abs(got.imag - ref.imag) <= HALF_ULP * np.abs(ref.imag) + slack)
