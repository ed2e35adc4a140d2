"""Single Krylov steps against the oracle at the sizes where the reductions
change shape: sets around one block's 256 points, around the 512 blocks after
which blocks take more than one round, and at every parity of the order."""
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


def unit_state(total, count, seed):
    rng = np.random.default_rng(seed)
    keys = np.sort(rng.choice(total, size=count, replace=False)).astype(np.uint64)
    c = random_complex(count, seed + 1)
    return keys, c / np.linalg.norm(c)


CASES = [("dvr", 1, 1), ("dvr", 255, 4), ("dvr", 256, 5), ("dvr", 257, 16), ("dvr", 513, 15),
         ("lattice", 255, 5), ("lattice", 256, 16), ("lattice", 257, 2), ("lattice", 4097, 7),
         ("large", 131071, 3), ("large", 131073, 4)]


@pytest.mark.parametrize("kind,count,m", CASES)
def test_step_at_reduction_edges(kind, count, m, torch):
    """The step is unitary or a similarity of one and its rounding errors are a
    few units of 2^-53 per application of dt H (norm below 100 on these sets), so
    the unit-norm states agree to 1e-13 (1e-12 on the lattice, whose basis is not
    orthogonal)."""
    import paper_1606_04004_amd as ppq
    if kind == "dvr":
        cd = card("small_4d")
    elif kind == "lattice":
        cd = dict(card("small_4d", n=[12] * 4), basis="pvb", lattice=[3, 4])
    else:
        cd = card("small_3d", n=[61, 60, 59])
    keys, c = unit_state(int(np.prod(cd["n"])), count, 10 * count + m)
    print(f"{kind}: {count} functions, order {m}", flush=True)
    o = Oracle(cd)
    o.set_state(keys, c)
    g = ppq.Propagator(cd, device=0, stream=torch.cuda.current_stream())
    g.set_state(keys, c)
    for _ in range(2):  # the second step starts from the first one's scalars
        g.step(dt=0.02, m=m)
        o.sil_step(dt=0.02, m=m)
    _, cg = g.state()
    _, co = o.state()
    assert np.linalg.norm(cg - co) < (1e-12 if kind == "lattice" else 1e-13) * np.linalg.norm(co)
