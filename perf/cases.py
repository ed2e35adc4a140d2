"""What users of this framework have it do, as cases to be timed.

A case is one of four tasks on one of the framework's models:

  product    y = P H P x on a given active set (Propagator.apply_h)
  step       one short-iterative Lanczos/Arnoldi step of a given state
  propagate  steps with adaption and observables, from a given state or from
             the model's Gaussian packet (Propagator.propagate)
  gradient   the survival probability and its gradient (SurvivalProbability)

The sizes are those of the repository's own cards and benchmark, or odd and
ragged ones around them.  The states are thresholded sums of Gaussian packets
with their neighbours, as adaption leaves them.  exact() restates every task
in plain torch on the full grid, in 64 bits.
"""
import functools
import math
import random

import numpy as np
import torch
import torch.utils.checkpoint

import paper_1606_04004_amd as ppq
from paper_1606_04004_amd.adjoint import SurvivalProbability, declare_trainable

DEV = "cuda"


# ---- the models ----------------------------------------------------------------
def power(k, p):
    return {"dim": k, "kind": "power", "p": p}


def morse(k, a, q0):
    return {"dim": k, "kind": "morse", "a": a, "q0": q0}


def pairs(D):
    return [(k, l) for k in range(D) for l in range(k + 1, D)]


def dense(k, rng, n, scale, kind):
    a = scale * rng.standard_normal((n, n))
    f = {"dim": k, "kind": "dense", "re": (0.5 * (a + a.T) if kind == "sym" else a).tolist()}
    if kind == "complex":
        f["im"] = (scale * rng.standard_normal((n, n))).tolist()
    return f


def card_of(case):
    """The model card of a case: operator, grid, packet and integrator."""
    model, D = case["model"], case["D"]
    n = [int(v) for v in str(case["n"]).split("x")]
    n = n * D if len(n) == 1 else n
    c = {"name": model, "D": D, "n": n, "mass": 1.0, "basis": case.get("basis", "dvr"), "eps": case["eps"],
         "dt": case.get("dt", 0.05), "krylov": case.get("m", 10), "nsteps": case.get("steps", 1)}
    if model == "henon_heiles":
        terms = [{"coef": 0.5, "factors": [power(0, 2)]}, {"coef": 0.5, "factors": [power(1, 2)]},
                 {"coef": 0.111, "factors": [power(0, 2), power(1, 1)]},
                 {"coef": -0.037, "factors": [power(1, 3)]}]
        c.update(lo=[-8.0] * 2, hi=[8.0] * 2, psi0={"centre": [2.0, 1.0], "momentum": [0.0, 0.5], "width": [1.0] * 2})
    elif model in ("anharmonic", "general_terms"):
        terms = [{"coef": v, "factors": [power(k, 2)]} for k, v in enumerate((0.5, 0.7, 0.45))]
        terms += [{"coef": 0.05, "factors": [power(0, 1), power(1, 1)]},
                  {"coef": -0.02, "factors": [power(1, 2), power(2, 1)]}, {"coef": 0.01, "factors": [power(0, 4)]}]
        if model == "general_terms":
            # dense factors and complex coefficients: products applied factor by factor
            rng = np.random.default_rng(77)
            s = 0.1 / math.sqrt(max(n))
            terms += [{"coef": 0.3, "factors": [dense(0, rng, n[0], s, "sym"), power(2, 1)]},
                      {"coef": 0.05, "coef_im": 0.02, "factors": [dense(1, rng, n[1], s, "complex"),
                                                                  dense(2, rng, n[2], s, "real")]},
                      {"coef": 0.02, "factors": [dense(k, rng, n[k], s, "real") for k in range(3)]},
                      {"coef": 0.01, "coef_im": -0.003, "factors": [power(0, 2)]}]
        c.update(mass=1.3, lo=[-5.0, -4.5, -5.5], hi=[5.0, 4.0, 5.0],
                 psi0={"centre": [0.8, -0.3, 0.2], "momentum": [0.3, 0.0, -0.4], "width": [1.0, 0.9, 1.1]})
    elif model == "morse":
        lam = np.random.default_rng(1606).uniform(-0.01, 0.01, size=6)
        terms = [{"coef": 0.2, "factors": [morse(k, 1.0, 0.0)]} for k in range(4)]
        if case["task"] == "gradient":
            # ordered couplings, every one of them trainable
            order = [(k, l) for k in range(4) for l in range(4) if k != l]
            half = {p: 0.5 * v for p, v in zip(pairs(4), lam)}
            terms += [{"coef": half[min(k, l), max(k, l)], "factors": [power(k, 1), power(l, 1)]} for k, l in order]
            c["trainable"] = ([{"name": f"D{k}", "term": k, "what": "coef"} for k in range(4)]
                              + [{"name": f"a{k}", "term": k, "what": "a", "factor": 0} for k in range(4)]
                              + [{"name": f"lam{i}", "term": 4 + i, "what": "coef"} for i in range(12)])
            c["checkpoint_every"] = case["every"]
        else:
            terms += [{"coef": float(v), "factors": [power(k, 1), power(l, 1)]} for (k, l), v in zip(pairs(4), lam)]
        c.update(lo=[-3.0] * 4, hi=[9.0] * 4,
                 psi0={"centre": [0.5, 0.0, 0.0, 0.0], "momentum": [0.0] * 4, "width": [0.5] * 4})
    elif model == "quartic":
        rng = np.random.default_rng(4004)
        w, cc, d = rng.uniform(0.8, 1.2, size=6), rng.normal(0.0, 0.005, size=15), rng.normal(0.0, 0.002, size=20)
        triples = [(k, l, m) for k in range(6) for l in range(k + 1, 6) for m in range(l + 1, 6)]
        terms = [{"coef": float(0.5 * v * v), "factors": [power(k, 2)]} for k, v in enumerate(w)]
        terms += [{"coef": float(v), "factors": [power(k, 2), power(l, 2)]} for (k, l), v in zip(pairs(6), cc)]
        terms += [{"coef": float(v), "factors": [power(k, 1) for k in t]} for t, v in zip(triples, d)]
        c.update(lo=[-6.5] * 6, hi=[6.5] * 6, psi0={"centre": [1.5] + [0.0] * 5, "momentum": [0.0] * 6,
                                                    "width": [float(v) ** -0.5 for v in w]})
    elif model == "double_well":
        terms = [{"coef": v, "factors": [power(0, p)]} for v, p in ((6.4, 4), (-38.4, 3), (63.2, 2), (-76.8, 1))]
        terms += [{"coef": 37.5, "factors": [power(1, 2)]}, {"coef": -150.0, "factors": [power(1, 1)]},
                  {"coef": 10.0, "factors": [power(0, 2), power(1, 1)]}, {"coef": 175.6, "factors": []}]
        c.update(mass=200.0, lo=[-0.5, 1.0], hi=[3.7, 2.9], fgh=[0, 1], krylov_tol=1e-10, max_substeps=64,
                 psi0={"centre": [2.1, 2.05], "momentum": [0.0, 0.0], "width": [0.02 ** 0.5, 0.1]})
    else:
        raise KeyError(model)
    c["terms"] = terms
    if c["basis"] != "dvr":
        c["lattice"] = [int(v) for v in case["lattice"].split("x")]
    return c


def packet_of(case, seed):
    """The card with the packet that `seed` moves a little."""
    c, r = card_of(case), random.Random(seed)
    ps = c["psi0"]
    ps["centre"] = [v + 0.1 * w * r.uniform(-1, 1) for v, w in zip(ps["centre"], ps["width"])]
    ps["momentum"] = [v + 0.1 / w * r.uniform(-1, 1) for v, w in zip(ps["momentum"], ps["width"])]
    if case["task"] == "gradient":  # another point of the training
        for t in c["terms"]:
            t["coef"] *= 1 + 0.02 * r.uniform(-1, 1)
            for f in t["factors"]:
                if f["kind"] == "morse":
                    f["a"] *= 1 + 0.02 * r.uniform(-1, 1)
    return c


# ---- the method on the full grid, in plain torch -----------------------------------
class Grid:
    """A card's one-dimensional ingredients and its operator on full-grid tensors."""

    def __init__(self, card):
        self.card, self.D, self.n = card, card["D"], card["n"]
        self.fgh = set(card.get("fgh", []))
        self.q, self.T, self.w, self.G = [], [], [], []
        for k, n in enumerate(self.n):
            lo, L = card["lo"][k], card["hi"][k] - card["lo"][k]
            if k in self.fgh:  # periodic Fourier grid: plane waves |k| <= (n-1) pi / L
                self.q.append(lo + np.arange(n) * L / n)
                self.w.append(L / n)
                kk = 2 * np.pi / L * np.arange(-(n // 2), n // 2 + 1)
                U = np.exp(1j * np.outer(self.q[k] - lo, kk)) / math.sqrt(n)
                self.T.append(((U * (kk ** 2 / (2 * card["mass"]))) @ U.conj().T).real)
            else:  # sine functions of the box
                i = np.arange(1, n + 1)
                self.q.append(lo + i * L / (n + 1))
                self.w.append(L / (n + 1))
                U = math.sqrt(2 / (n + 1)) * np.sin(np.pi * np.outer(i, i) / (n + 1))
                self.T.append((U * ((np.pi * i / L) ** 2 / (2 * card["mass"]))) @ U.T)
            self.G.append(self.lattice(k) if card["basis"] != "dvr" else None)
        self.axes = []
        for n in self.n:
            self.axes += card["lattice"] if card["basis"] != "dvr" else [n]

    def lattice(self, k):
        """Projected von Neumann Gaussians, or the orthogonal projected Weylets."""
        ns, nl = self.card["lattice"]
        pw = self.card["basis"] == "pw"
        dx = (self.card["hi"][k] - self.card["lo"][k]) / ns
        dp = (np.pi if pw else 2 * np.pi) / dx
        a = dp / (2 * dx)
        d = self.q[k][:, None, None] - (self.card["lo"][k] + (np.arange(ns) + 0.5) * dx)[:, None]
        if pw:
            p = (np.arange(nl) + 0.5) * dp
            F = (8 * a / np.pi) ** 0.25 * np.exp(-a * d * d) * np.sin(p * (d - math.sqrt(np.pi / (8 * a))))
            F = math.sqrt(self.w[k]) * F.reshape(self.n[k], -1)
            w, V = np.linalg.eigh(F.T @ F)
            return (F @ (V * w ** -0.5) @ V.T).astype(complex)
        p = (np.arange(nl) - 0.5 * (nl - 1)) * dp
        return math.sqrt(self.w[k]) * ((2 * a / np.pi) ** 0.25 * np.exp(-a * d * d + 1j * p * d)).reshape(self.n[k], -1)

    def acting(self, k, h):
        return h if self.G[k] is None else self.G[k].conj().T @ h @ np.linalg.inv(self.G[k].conj().T)

    def values(self, f):
        q = self.q[f["dim"]]
        return q ** f["p"] if f["kind"] == "power" else (1 - np.exp(-f["a"] * (q - f["q0"]))) ** 2

    def packet(self, ps, dual=False):
        """The packet's one-dimensional coefficient vectors."""
        out = []
        for k, q in enumerate(self.q):
            g = np.exp(-(q - ps["centre"][k]) ** 2 / (2 * ps["width"][k] ** 2) + 1j * ps["momentum"][k] * (q - ps["centre"][k]))
            g = g / np.linalg.norm(g)
            if self.G[k] is not None:
                g = np.linalg.solve(self.G[k], g) if dual else self.G[k].conj().T @ g
            out.append(torch.from_numpy(g + 0j).to(DEV))
        return out

    def operator(self):
        """One-dimensional matrices, the diagonal potential and the product terms."""
        one = [self.T[k] + 0j for k in range(self.D)]
        self.V, self.prod = torch.zeros(self.n, dtype=torch.float64, device=DEV), []
        for t in self.card["terms"]:
            coef = complex(t["coef"], t.get("coef_im", 0.0))
            mats = {}
            for f in t["factors"]:
                m = np.array(f["re"]) + 1j * np.array(f.get("im", 0.0)) if f["kind"] == "dense" else np.diag(self.values(f)) + 0j
                mats[f["dim"]] = mats[f["dim"]] @ m if f["dim"] in mats else m
            ks = sorted(mats)
            if self.card["basis"] == "dvr" and coef.imag == 0 and not any(f["kind"] == "dense" for f in t["factors"]):
                v = torch.tensor(coef.real, dtype=torch.float64, device=DEV)
                for k in ks:
                    v = v * self.line(k, torch.from_numpy(np.diag(mats[k]).real.copy()).to(DEV))
                self.V += v
            elif self.card["basis"] != "dvr" and len(ks) <= 1:
                k = ks[0] if ks else 0
                one[k] = one[k] + coef * (mats[k] if ks else np.eye(self.n[k]))
            else:
                self.prod.append((coef, [(k, torch.from_numpy(self.acting(k, mats[k])).to(DEV)) for k in ks]))
        one = [self.acting(k, h) for k, h in enumerate(one)]
        self.one = [torch.from_numpy(h if np.abs(h.imag).max() else h.real.copy()).to(DEV) for h in one]
        self.hermitian = self.card["basis"] == "dvr" and not any(
            c.imag or sum(bool((m - torch.diag(torch.diagonal(m))).abs().max()) for _, m in ms) > 1 or
            any(bool((m - m.conj().T).abs().max()) for _, m in ms) for c, ms in self.prod)
        return self

    def line(self, k, v):
        return v.reshape([-1 if j == k else 1 for j in range(self.D)])

    @staticmethod
    def mode(h, x, k):
        X = x.movedim(k, 0)
        Y = X.reshape(X.shape[0], -1)
        if h.is_complex():
            Y = h @ Y
        else:
            Y = (h @ torch.view_as_real(Y).reshape(Y.shape[0], -1)).reshape(*Y.shape, 2)
            Y = torch.view_as_complex(Y)
        return Y.reshape(X.shape).movedim(0, k)

    def apply(self, keys, c, V=None):
        """P H P c for coefficients on the keys."""
        total = math.prod(self.n)
        x = torch.zeros(total, dtype=torch.complex128, device=DEV).index_copy(0, keys, c).reshape(self.n)
        y = (self.V if V is None else V) * x
        for k in range(self.D):
            y = y + self.mode(self.one[k], x, k)
        if self.prod:
            on = torch.zeros(total, dtype=torch.bool, device=DEV).index_fill(0, keys, True).reshape(self.n)
            for coef, ms in self.prod:
                z = x
                for k, m in reversed(ms):
                    z = self.mode(m, z, k) * on
                y = y + coef * z
        return y.reshape(-1)[keys]

    def outer(self, gs):
        v = gs[0]
        for g in gs[1:]:
            v = (v[..., None] * g).reshape(-1)
        return v

    def kept(self, v, eps):
        return v.real ** 2 + v.imag ** 2 >= eps * eps

    def dilate(self, keep):
        keep = keep.reshape(self.axes)
        out = keep.clone()
        for a, n in enumerate(self.axes):
            out.narrow(a, 1, n - 1).logical_or_(keep.narrow(a, 0, n - 1))
            out.narrow(a, 0, n - 1).logical_or_(keep.narrow(a, 1, n - 1))
        return out.reshape(-1).nonzero().reshape(-1)

    def prune(self, keys, c, eps):
        full = torch.zeros(math.prod(self.n), dtype=torch.complex128, device=DEV).index_copy(0, keys, c)
        new = self.dilate(self.kept(full, eps))
        return new, full[new]

    def krylov(self, keys, c, dt, m, tol):
        """One short-iterative step: the new coefficients, its order and alpha_0."""
        n0 = float(torch.linalg.vector_norm(c))
        v, H, est, used = [c / n0], np.zeros((m, m), complex), n0, m
        for j in range(m):
            w = self.apply(keys, v[j])
            for _ in range(2):
                for i in range(j + 1):
                    s = torch.vdot(v[i], w)
                    H[i, j] += complex(s)
                    w = w - s * v[i]
            b = float(torch.linalg.vector_norm(w))
            if j == m - 1:
                break
            H[j + 1, j] = b
            est *= abs(dt) * b / (j + 1)
            if b < 1e-13 or (tol > 0 and est <= tol):
                used = j + 1
                break
            v.append(w / b)
        h = H[:used, :used]
        h = (h + h.conj().T) / 2 if self.hermitian else h
        y = torch.linalg.matrix_exp(torch.from_numpy(-1j * dt * h))[:, 0] * n0
        return sum(complex(y[i]) * v[i] for i in range(used)), used, H[0, 0].real

    def step(self, keys, c, sub):
        """A step under the card's integrator settings; `sub` the substeps to begin with."""
        dt, m, tol, most = self.card["dt"], self.card["krylov"], self.card.get("krylov_tol", 0.0), self.card.get("max_substeps", 1)
        while True:
            x, orders, alpha = c, [], None
            for _ in range(sub):
                x, used, a = self.krylov(keys, x, dt / sub, m, tol)
                orders.append(used)
                alpha = a if alpha is None else alpha
            if most <= 1 or tol <= 0 or max(orders) < m:
                return x, max(orders), alpha, sub, (sub // 2 if most > 1 and max(orders) <= m // 2 and sub > 1 else sub)
            sub *= 2

    def propagate(self, keys, c, steps, eps, bra):
        rows, sub = [], 1
        dual = self.outer(bra)
        for st in range(steps + 1):
            acf = complex(torch.vdot(dual[keys], c))
            rows.append([st * self.card["dt"], float(c.abs().square().sum()), 0.0, acf.real, acf.imag, len(keys),
                         int(self.kept(c, eps).sum()), 0, 0])
            if st:
                rows[st][7:] = order, used
            if st == steps:
                break
            c, order, rows[st][2], used, sub = self.step(keys, c, sub)
            keys, c = self.prune(keys, c, eps)
        rows[-1][2] = float(torch.vdot(c, self.apply(keys, c)).real) / rows[-1][1]
        return np.array(rows), keys, c


# ---- states ----------------------------------------------------------------------
def state_of(case, seed, grid=None):
    """Keys and coefficients of a state as adaption leaves it: a few packets about
    the model's own, spread by the time that has passed and moving against each
    other, thresholded, with their neighbours."""
    card = packet_of(case, seed)
    grid = grid or Grid(card)
    if case["start"] == "packet":
        full = grid.outer(grid.packet(card["psi0"]))
    else:
        r = random.Random(seed + 1)
        full = 0
        for part in (1.0, 0.35, 0.2):
            ps = {"width": [w * case["spread"] * r.uniform(0.95, 1.05) for w in card["psi0"]["width"]],
                  "centre": [v + (1 - part) * 0.5 * case["spread"] * r.uniform(-1, 1) * w for v, w in zip(card["psi0"]["centre"], card["psi0"]["width"])],
                  "momentum": [v + 0.5 * case["spread"] ** 2 * r.uniform(-1, 1) / w for v, w in zip(card["psi0"]["momentum"], card["psi0"]["width"])]}
            full = full + part * np.exp(1j * r.uniform(-np.pi, np.pi)) * grid.outer(grid.packet(ps))
        full /= torch.linalg.vector_norm(full)
    keys = grid.dilate(grid.kept(full, case["eps"]))
    return keys, full[keys].clone()


@functools.lru_cache(maxsize=64)
def room_for(items):
    """Entries of a program's result buffers: what the case's states hold, and for a run what they may grow to."""
    case = dict(items)
    n, total = len(state_of(case, 0)[0]), math.prod(card_of(case)["n"])
    return min(total, 20_000 + (int(1.3 * n) if case["task"] != "propagate" else 2 * n if case["D"] == 6 else 6 * n))


def room_of(case):
    return room_for(tuple(sorted((k, v) for k, v in case.items() if k != "name")))


@functools.lru_cache(maxsize=1)
def stream():
    """The program's stream: every propagator runs on it, between the program's own operations."""
    return torch.cuda.Stream()


def theta_of(card):
    """Trainable parameters: the model's coefficients, the packet's centre and momentum."""
    pot = [card["terms"][t["term"]]["coef"] if t["what"] == "coef" else card["terms"][t["term"]]["factors"][0]["a"]
           for t in card["trainable"]]
    return torch.tensor(pot + card["psi0"]["centre"] + card["psi0"]["momentum"], dtype=torch.float64)


# ---- the cases -------------------------------------------------------------------
def listed():
    six = {"model": "quartic", "D": 6, "n": "24", "eps": 1e-6, "start": "state", "spread": 1.0}
    return [
        # exploring a model interactively: a 2D run where launches and waits are all there is
        {"name": "run_2d", "task": "propagate", "model": "henon_heiles", "D": 2, "n": "48", "eps": 1e-5, "steps": 20,
         "start": "packet", "precision": "f64"},
        # the 2D double well on long Fourier grids, integrated to a tolerance
        {"name": "run_double_well", "task": "propagate", "model": "double_well", "D": 2, "n": "165x81", "eps": 1e-5,
         "dt": 0.1, "m": 16, "steps": 5, "start": "packet", "precision": "f64"},
        # general sum-of-products terms (Arnoldi), ragged 3D grid
        {"name": "run_general_terms", "task": "propagate", "model": "general_terms", "D": 3, "n": "27x33x30", "eps": 1e-5,
         "steps": 4, "start": "packet", "precision": "f64"},
        # a 4D run in the middle of its course
        {"name": "run_4d", "task": "propagate", "model": "morse", "D": 4, "n": "32", "eps": 1e-6, "dt": 0.1, "steps": 3,
         "start": "state", "spread": 2.0, "precision": "f64"},
        # one unpruned step of a 4D state in the single-precision form
        {"name": "step_4d_f32", "task": "step", "model": "morse", "D": 4, "n": "31", "eps": 1e-6, "dt": 0.1,
         "start": "state", "spread": 2.0, "precision": "f32"},
        # the 4D run in a phase-space lattice basis, from its packet
        {"name": "run_lattice_4d", "task": "propagate", "model": "morse", "D": 4, "n": "48", "basis": "pvb",
         "lattice": "6x8", "eps": 1e-6, "dt": 0.1, "steps": 2, "start": "packet", "precision": "f64"},
        # its operator alone, as an outside integrator or eigensolver calls it, on a spread state
        {"name": "product_lattice_4d", "task": "product", "model": "morse", "D": 4, "n": "48", "basis": "pvb",
         "lattice": "6x8", "eps": 1e-7, "start": "state", "spread": 3.0, "precision": "f64"},
        # training: the survival probability and its gradient
        {"name": "gradient_4d", "task": "gradient", "model": "morse", "D": 4, "n": "24", "eps": 1e-5, "steps": 16, "m": 16,
         "every": 5, "start": "packet", "precision": "f64"},
        # the 6D production run: the operator alone in both precisions, steps of the run, a single-precision step
        {"name": "product_6d", "task": "product", "precision": "f64", **six},
        {"name": "product_6d_f32", "task": "product", "precision": "f32", **six},
        {"name": "run_6d", "task": "propagate", "steps": 3, "precision": "f64", **six},
        {"name": "step_6d_f32", "task": "step", "precision": "f32", **six},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def eps(lo, hi):
        return float("%.2g" % math.exp(rng.uniform(math.log(lo), math.log(hi))))

    prec = rng.choice(["f64", "f64", "f32"])
    kind = rng.randrange(7)
    if kind == 0:
        c = {"model": "henon_heiles", "D": 2, "n": "%dx%d" % (size(24, 64), size(24, 64)), "eps": eps(1e-7, 1e-3)}
        c |= rng.choice([{}, {"basis": "pw", "lattice": "6x8", "n": "48"}])
    elif kind == 1:
        c = {"model": "double_well", "D": 2, "n": "%dx%d" % (2 * size(33, 82) + 1, 2 * size(25, 40) + 1),
             "eps": eps(1e-7, 1e-4), "dt": 0.1, "m": 16}
    elif kind == 2:
        c = {"model": rng.choice(["anharmonic", "general_terms"]), "D": 3,
             "n": "x".join(str(size(18, 48)) for _ in range(3)), "eps": eps(1e-7, 1e-3)}
    elif kind == 3:
        c = {"model": "morse", "D": 4, "n": "x".join(str(size(18, 32)) for _ in range(4)), "eps": eps(1e-6, 1e-4), "dt": 0.1}
    elif kind == 4:
        ns, nl = rng.choice([(5, 6), (6, 6), (5, 8), (6, 8)])
        c = {"model": "morse", "D": 4, "n": str(ns * nl), "basis": rng.choice(["pvb", "pw"]),
             "lattice": "%dx%d" % (ns, nl), "eps": eps(1e-6, 1e-4), "dt": 0.1}
    elif kind == 5:
        return {"task": "gradient", "model": "morse", "D": 4, "n": str(size(16, 24)), "eps": eps(1e-5, 1e-4),
                "steps": rng.randint(6, 16), "m": 16, "every": rng.randint(2, 8), "start": "packet", "precision": "f64"}
    else:
        c = {"model": "quartic", "D": 6, "n": "x".join(str(rng.randint(16, 24)) for _ in range(6)), "eps": eps(1e-6, 1e-4)}
    c["task"] = rng.choice(["product", "step"] if prec == "f32" else ["product", "propagate", "propagate"])
    if kind == 1 and c["task"] == "step":
        c["task"] = "product"
    if c["task"] == "propagate":
        c["steps"] = rng.randint(1, 3) if c["D"] > 3 else rng.randint(3, 12) if kind != 1 else rng.randint(2, 5)
    c["start"] = rng.choice(["packet", "state"])
    if c["start"] == "state":
        c["spread"] = round(rng.uniform(1.0, 2.0) if c["D"] == 4 else rng.uniform(0.9, 1.0), 2)
    c["precision"] = prec
    return c


def prepare(case, seed):
    card = packet_of(case, seed)
    prec = ppq.PPQ_FP32 if case["precision"] == "f32" else ppq.PPQ_FP64
    p = ppq.Propagator(card, precision=prec, stream=stream())
    total = math.prod(card["n"])
    s = {"task": case["task"], "p": p, "start": case["start"]}
    if case["task"] == "gradient":
        declare_trainable(p, card)
        p.reserve(total)
        s["theta"] = theta_of(card).requires_grad_(True)
        return s
    grid = Grid(card)
    keys, c = state_of(case, seed, grid)
    n, room = len(keys), room_of(case)
    p.reserve(room)  # programs reserve up front what a run may grow to
    p.set_reference()
    s.update(keys=keys, c=c, n=n)
    single = torch.complex64 if case["precision"] == "f32" else torch.complex128
    if case["task"] == "product":
        p.set_state_device(keys, c)
        s["x"] = torch.zeros(room, dtype=single, device=DEV)
        s["x"][:n] = c
        s["y"] = torch.zeros_like(s["x"])
        p.apply_h(s["x"], s["y"])  # the set's tables are built once
        torch.cuda.synchronize()
        return s
    s["keys_out"] = torch.zeros(room, dtype=torch.int64, device=DEV)
    s["c_out"] = torch.zeros(room, dtype=torch.complex128, device=DEV)
    if case["task"] == "step":
        s["single_out"] = torch.zeros(room, dtype=single, device=DEV)
    torch.cuda.synchronize()
    return s


def run(s):
    p = s["p"]
    if s["task"] == "product":
        p.apply_h(s["x"], s["y"])
        return s["y"]
    if s["task"] == "gradient":
        J = SurvivalProbability.apply(s["theta"], p)
        return {"J": J.detach(), "grad": torch.autograd.grad(J, s["theta"])[0]}
    if s["start"] == "packet" and s["task"] == "propagate":
        p.init_state()
    else:
        p.set_state_device(s["keys"], s["c"])
    if s["task"] == "step":
        p.step()
        n = p.state_device(s["keys_out"], s["c_out"])
        # a single-precision program keeps its states in single precision
        with torch.cuda.stream(stream()):
            s["single_out"][:n] = s["c_out"][:n]
        return s["single_out"]
    trace = p.propagate()
    n = p.state_device(s["keys_out"], s["c_out"])
    return {"trace": trace, "n": n, "keys": s["keys_out"], "c": s["c_out"]}


def work(case):
    """Bytes: the given state (or vector) in, the result out.  Flops: the fibers'
    contractions, the Krylov projections and recombination."""
    card = packet_of(case, 0)
    grid = Grid(card)
    keys, _ = state_of(case, 0, grid)
    n, total = len(keys), math.prod(card["n"])
    on = torch.zeros(total, dtype=torch.float64, device=DEV).index_fill(0, keys, 1.0).reshape(card["n"])
    sq = [float(on.sum(k).square().sum()) for k in range(card["D"])]
    cplx = case.get("basis", "dvr") != "dvr"
    prod = (8 if cplx else 4) * sum(sq) + (0 if cplx else 4 * n)
    for t in card["terms"]:
        ds = sorted({f["dim"] for f in t["factors"] if cplx or f["kind"] == "dense"})
        prod += 8 * sum(sq[k] for k in ds) if len(ds) > cplx else 0
    if case["task"] == "product":
        return {"bytes": (8 if case["precision"] == "f32" else 16) * 2 * n, "flops": prod}
    m, steps = card["krylov"], card["nsteps"]
    step = m * prod + 16 * n * m * (m + 1) / 2 + 8 * n * m
    if case["task"] == "gradient":
        return {"bytes": 24 * n, "flops": 3 * steps * step}
    return {"bytes": (48 if case["task"] == "propagate" else 40) * n, "flops": steps * step}


# ---- what run() returns, in 64 bits -------------------------------------------------
def exact_gradient(case, seed):
    """J and its gradient with the sets of the run held fixed and exact exponentials."""
    card = packet_of(case, seed)
    D, npot = card["D"], len(card["trainable"])
    th = theta_of(card).to(DEV).requires_grad_(True)
    grid = Grid(card).operator()
    q = [torch.from_numpy(v).to(DEV) for v in grid.q]
    at = {}
    for i, t in enumerate(card["trainable"]):
        at[t["term"], t["what"]] = th[i]
    V = 0
    for i, t in enumerate(card["terms"]):
        v = at.get((i, "coef"), t["coef"])
        for f in t["factors"]:
            k = f["dim"]
            v = v * grid.line(k, q[k] if f["kind"] == "power" else (1 - torch.exp(-at[i, "a"] * (q[k] - f["q0"]))) ** 2)
        V = V + v
    gs = []
    for k in range(D):
        d = q[k] - th[npot + k]
        g = torch.exp(-d * d / (2 * card["psi0"]["width"][k] ** 2)) * torch.exp(1j * th[npot + D + k] * d)
        gs.append(g / torch.linalg.vector_norm(g))
    psi0 = grid.outer(gs)
    norm = sum(float(torch.linalg.matrix_norm(h, 2)) for h in grid.one)
    with torch.no_grad():
        keys = grid.dilate(grid.kept(psi0, case["eps"]))

    def move(c, V, keys):
        sub = max(1, math.ceil(card["dt"] * (norm + float(V.detach().reshape(-1)[keys].abs().max())) / 2))
        for _ in range(sub):
            term, out = c, c
            for j in range(1, 27):
                term = grid.apply(keys, term, V) * (-1j * card["dt"] / sub / j)
                out = out + term
            c = out
        return c

    c = psi0[keys]
    for _ in range(card["nsteps"]):
        c = torch.utils.checkpoint.checkpoint(move, c, V, keys, use_reentrant=False)
        with torch.no_grad():
            new, _ = grid.prune(keys, c, case["eps"])
        c = torch.zeros_like(psi0).index_copy(0, keys, c)[new]
        keys = new
    J = torch.vdot(psi0[keys], c).abs().square()
    return {"J": J.detach().cpu(), "grad": torch.autograd.grad(J, th)[0].cpu()}


def exact(case, seed):
    if case["task"] == "gradient":
        return exact_gradient(case, seed)
    card = packet_of(case, seed)
    grid = Grid(card).operator()
    keys, c = state_of(case, seed, grid)
    room = room_of(case)

    def whole(v):
        return torch.cat([v, torch.zeros(room - len(v), dtype=v.dtype, device=DEV)])

    if case["task"] == "product":
        return whole(grid.apply(keys, c.to(torch.complex64).to(torch.complex128) if case["precision"] == "f32" else c))
    if case["task"] == "step":
        return whole(grid.step(keys, c, 1)[0])
    trace, keys, c = grid.propagate(keys, c, card["nsteps"], case["eps"], grid.packet(card["psi0"], dual=True))
    return {"trace": trace, "n": len(keys), "keys": whole(keys), "c": whole(c)}
