"""The work that programs do with this framework, as timed cases.

A case is a lattice and one pass through a public entry point: H x (c128, c64) on chains, rings, the square
lattice and spin-boson models, H x in a digit-sum sector, the autograd function (forward and backward), Lanczos,
time propagation, the batched form and a sweep of couplings.  listed() holds the lattices of the benchmark and of
the tests next to them, from the 12-site chain (a launch-bound call) to the 20-site ring (60 million rows);
draw() spreads sizes, local dimensions, element types and options over the same ranges.

A case's plain values: "kind" (the entry point), "lattice" ("chain" / "ring": sites 2s from "spins"; "ferri": ring
of alternating 1/2 and 1; "square": L x L spin-1; "tavis": spins and one boson mode), "couplings" ("uniform": shared
by all bonds; "bond": one pair per bond) and the sizes and options of the entry point.  Everything random comes
from the seed: the state vectors (complex normal, unit norm) and the couplings.
"""
import math

import numpy as np
import torch

from paper_2606_02169_amd.plan import Batch, MatvecFn, Plan, Sector, Sweep
from workloads import configs as W
from workloads.model import (OP_LOWER, OP_LOWER2, OP_RAISE, OP_RAISE2, OP_Z, OP_Z2, SPIN, Model, Term, spin_site,
                             xxz_bond_terms)

DEV = "cuda"


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    ferri = {"lattice": "ferri", "couplings": "uniform"}
    return [
        # the smallest call: one H x of the 12-site Heisenberg chain, all latency
        {"name": "matvec_chain12", "kind": "matvec", "lattice": "chain", "spins": "1" * 12, "couplings": "one",
         "dtype": "c128", "tuned": True},
        # an ordinary chain of mixed spins with its own couplings on every bond, nothing tuned for it
        {"name": "matvec_mixed13", "kind": "matvec", "lattice": "chain", "spins": "1323122313212",
         "couplings": "bond", "dtype": "c128", "tuned": False},
        # the headline: FP64 H x on the 20-site ferrimagnetic ring
        {"name": "matvec_ring20", "kind": "matvec", **ferri, "n": 20, "dtype": "c128", "tuned": True},
        # the FP32 form on the 4 x 4 periodic spin-1 lattice
        {"name": "matvec_square4x4_c64", "kind": "matvec", "lattice": "square", "n": 4, "couplings": "bond",
         "dtype": "c64", "tuned": True},
        # H x inside the S_z = 0 sector of the ring
        {"name": "sector_ring20", "kind": "sector", **ferri, "n": 20, "dtype": "c128"},
        # a training step's forward and backward through the Tavis-Cummings Hamiltonian
        {"name": "autograd_tavis12", "kind": "autograd", "lattice": "tavis", "n": 12, "n_max": 64,
         "couplings": "bond"},
        # ground state of the small chain: 50 Lanczos steps, launch bound
        {"name": "lanczos_chain12", "kind": "lanczos", "lattice": "chain", "spins": "1" * 12, "couplings": "one",
         "m": 50, "reorth": "cgs2"},
        # ground state of a ten-million-row ring with the default reorthogonalisation
        {"name": "lanczos_ring18", "kind": "lanczos", **ferri, "n": 18, "m": 40, "reorth": "cgs2"},
        # ground state inside a sector, the cheap reorthogonalisation
        {"name": "lanczos_sector_ring18", "kind": "lanczos", **ferri, "n": 18, "m": 40, "reorth": "partial",
         "sector": True},
        # four steps of a driven ring
        {"name": "propagate_ring18", "kind": "propagate", **ferri, "n": 18, "steps": 4, "dt": 0.05,
         "drive": True},
        # many uneven lattices in one launch, blocks of eight c64 vectors
        {"name": "batch_chains64", "kind": "batch", "n": 64, "lattices": 4, "nvec": 8},
        # a sweep of 64 coupling vectors of one ring over eight vectors
        {"name": "sweep_ring14", "kind": "sweep", **ferri, "n": 14, "points": 64, "nvec": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _spins(rng, dmin, dmax):
    """Random 2s in 1..3 per site until the dimension reaches a log-uniform target."""
    target = math.exp(rng.uniform(math.log(dmin), math.log(dmax)))
    kinds = rng.choice(["1", "2", "12", "123", "23"])
    s, D = "", 1
    while True:
        k = rng.choice(kinds)
        if len(s) >= 3 and D * (int(k) + 1) > target:
            return s
        s, D = s + k, D * (int(k) + 1)


def draw(rng):
    kind = rng.choice(["matvec", "matvec", "matvec", "matvec", "sector", "sector", "autograd", "lanczos",
                       "lanczos", "propagate", "batch", "sweep"])
    lattice = rng.choice(["chain", "ring"])
    couplings = rng.choice(["uniform", "bond"])
    if kind == "matvec":
        if rng.random() < 0.15:
            return {"kind": kind, "lattice": "tavis", "n": rng.randint(6, 16), "n_max": _log(rng, 7, 130),
                    "couplings": "bond", "dtype": rng.choice(["c128", "c64"]), "tuned": False}
        return {"kind": kind, "lattice": lattice, "spins": _spins(rng, 2 ** 10, 5e7), "couplings": couplings,
                "dtype": rng.choice(["c128", "c128", "c64"]), "tuned": False}
    if kind == "sector":
        return {"kind": kind, "lattice": lattice, "spins": _spins(rng, 2 ** 12, 5e7), "couplings": couplings,
                "dtype": rng.choice(["c128", "c128", "c64"])}
    if kind == "autograd":
        if rng.random() < 0.5:
            return {"kind": kind, "lattice": "tavis", "n": rng.randint(4, 14), "n_max": _log(rng, 7, 100),
                    "couplings": "bond"}
        return {"kind": kind, "lattice": lattice, "spins": _spins(rng, 2 ** 10, 4e6), "couplings": couplings}
    if kind == "lanczos":
        return {"kind": kind, "lattice": lattice, "spins": _spins(rng, 2 ** 12, 2e7), "couplings": couplings,
                "m": rng.randint(20, 40), "reorth": rng.choice(["cgs2", "cgs2", "cgs2_cond", "partial"]),
                "sector": rng.random() < 0.4}
    if kind == "propagate":
        return {"kind": kind, "lattice": lattice, "spins": _spins(rng, 2 ** 12, 1e7), "couplings": couplings,
                "steps": rng.randint(1, 8), "dt": round(rng.uniform(0.02, 0.1), 4), "drive": rng.random() < 0.5}
    if kind == "batch":
        return {"kind": kind, "n": _log(rng, 8, 64), "lattices": rng.randint(5, 1000),
                "nvec": rng.choice([1, 2, 4, 8, 8])}
    return {"kind": "sweep", "lattice": lattice, "spins": _spins(rng, 2 ** 10, 2.5e5), "couplings": "uniform",
            "points": _log(rng, 8, 64), "nvec": rng.choice([1, 2, 4, 8])}


# ------------------------------------------------------------------------------------------------ the lattices
def _model(case):
    """Sites, terms and the centre of the couplings; theta has one or a few entries ("one", "uniform") or a
    (J_xy, J_z) pair per bond ("bond")."""
    kind = case["lattice"]
    if kind == "ferri":
        return W.ferrimagnetic_ring(case["n"])
    if kind == "square":
        return W.square_lattice_spin1(case["n"], np.random.default_rng(3))
    if kind == "tavis":
        return W.tavis_cummings(case["n"], case["n_max"], 1.0, 1.0, np.random.default_rng(5))
    two_s = [int(c) for c in case["spins"]]
    N = len(two_s)
    if case["couplings"] == "one":
        return W.heisenberg_chain(N, two_s=two_s[0])
    bonds = [(i, i + 1) for i in range(N - 1)] + ([(N - 1, 0)] if kind == "ring" else [])
    terms, theta = [], []
    if case["couplings"] == "bond":
        for b, (i, j) in enumerate(bonds):
            terms += xxz_bond_terms(i, j, 2 * b, 2 * b + 1)
            theta += [1.0, 0.8]
    else:
        for i in range(N):
            terms.append(Term(i, OP_Z, -1, OP_Z, 2, 1.0 if i % 2 == 0 else -1.0))
        for i, j in bonds:
            terms += xxz_bond_terms(i, j, 0, 1)
        theta = [1.0, 1.0, 0.2]
    return Model([spin_site(k) for k in two_s], terms, np.array(theta))


def _models(case):
    """The lattices of a batch: open mixed-spin chains of 8 to 16 sites, as in the benchmark."""
    return W.batched_chains(case["n"], np.random.default_rng(case["lattices"]))


def _digit_sum(model):
    """The largest sector: half of the highest digit sum."""
    return sum(s.k for s in model.sites) // 2


def _gen(seed, device=DEV):
    return torch.Generator(device=device).manual_seed(int(seed))


def _couplings(model, seed, rows=0):
    """float64 couplings (CPU): the model's, each scaled by a factor in [0.8, 1.2]; rows > 0: that many sets."""
    th = torch.as_tensor(model.theta, dtype=torch.float64)
    shape = (rows, th.numel()) if rows else (th.numel(),)
    f = 0.8 + 0.4 * torch.rand(shape, dtype=torch.float64, generator=_gen(7919 * seed + 1, "cpu"))
    return (th * f).contiguous()


def _state(shape, dtype, seed):
    """Complex normal vector(s) of unit norm: one of D entries, or a [D, nvec] block of columns."""
    real = torch.float64 if dtype == "c128" else torch.float32
    x = torch.view_as_complex(torch.randn(tuple(shape) + (2,), dtype=real, device=DEV, generator=_gen(seed)))
    x /= torch.linalg.vector_norm(x, dim=0)
    return x


def _blocks(offsets, total, dims, nvec, seed):
    """The flat tensor of a batch: lattice b's [D_b, nvec] block at offsets[b]."""
    X = torch.zeros(total, dtype=torch.complex64, device=DEV)
    for b, (o, D) in enumerate(zip(offsets, dims)):
        X[o: o + D * nvec] = _state((D, nvec), "c64", seed * 1009 + b).reshape(-1)
    return X


def _inputs(case, seed, model):
    """(couplings on the CPU, vectors on the GPU) of the kinds that work on one vector; exact() uses them too."""
    rows = case["steps"] if case["kind"] == "propagate" and case["drive"] else 0
    theta = _couplings(model, seed, rows)
    n = model.dim
    if case["kind"] == "sector" or case.get("sector"):
        n = _sector_rows(model, _digit_sum(model)).numel()
    vecs = [_state((n,), case.get("dtype", "c128"), seed * 11 + 3)]
    if case["kind"] == "autograd":
        vecs.append(_state((n,), "c128", seed * 11 + 4))
    return theta, vecs


# ------------------------------------------------------------------------------------------------ a program's pass
def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        models = _models(case)
        batch = Batch([Plan.from_model(m) for m in models], case["nvec"])
        theta = torch.cat([_couplings(m, seed * 1013 + b) for b, m in enumerate(models)]).float().to(DEV)
        X = _blocks(batch.offsets, batch.total_elems, [m.dim for m in models], case["nvec"], seed)
        Y = torch.zeros_like(X)
        batch.autotune(theta, X, Y)
        return {"kind": kind, "batch": batch, "theta": theta, "X": X, "Y": Y}
    model = _model(case)
    plan = Plan.from_model(model)
    if kind == "sweep":
        sweep = Sweep(plan, case["nvec"])
        theta = _couplings(model, seed, case["points"]).float().to(DEV)
        X = torch.zeros(sweep.input_elems, dtype=torch.complex64, device=DEV)
        X[: sweep.n] = _state((model.dim, case["nvec"]), "c64", seed * 11 + 3).reshape(-1)
        return {"kind": kind, "sweep": sweep, "theta": theta, "X": X}
    theta, vecs = _inputs(case, seed, model)
    theta = theta.to(DEV)
    if case.get("dtype") == "c64":
        theta = theta.float()
    space = plan
    if kind == "sector" or case.get("sector"):
        space = Sector(plan, _digit_sum(model))
        space.generated(vecs[0].dtype)
    elif case.get("tuned"):
        plan.autotune(theta, vecs[0])
    else:
        plan.prepare(vecs[0].dtype)
    if kind == "autograd":
        plan.grad_kernel_ready()
        theta.requires_grad_(True)
        vecs[0].requires_grad_(True)
    return {"kind": kind, "space": space, "theta": theta, "x": vecs[0], "g": vecs[-1], "case": dict(case)}


def run(state):
    kind = state["kind"]
    if kind == "batch":
        return state["batch"].matvec(state["theta"], state["X"], state["Y"])
    if kind == "sweep":
        return state["sweep"].run(state["theta"], state["X"])
    space, theta, x, case = state["space"], state["theta"], state["x"], state["case"]
    if kind in ("matvec", "sector"):
        return space.matvec(theta, x)
    if kind == "autograd":
        y = MatvecFn.apply(space, theta, x)
        gt, gx = torch.autograd.grad(y, (theta, x), state["g"])
        return {"y": y, "grad_theta": gt, "grad_x": gx}
    if kind == "lanczos":
        out = space.lanczos(theta, x, case["m"], reorth=case["reorth"])
        return {"alpha": out["alpha"], "beta": out["beta"], "energy": out["result"][:1], "u": out["u"]}
    return space.propagate(theta, x, case["dt"], case["steps"])["x"]


# ------------------------------------------------------------------------------------------------ the least work
def _factors(site, op):
    """(shift q, values <n|O|n - q> for n = 0 .. d - 1) of a local operator."""
    d = site.k + 1
    n = np.arange(d, dtype=np.float64)
    z = n - 0.5 * site.k if site.kind == SPIN else n
    up = np.sqrt(n * (d - n)) if site.kind == SPIN else np.sqrt(n)       # <n|O_+|n - 1>
    down = np.append(up[1:], 0.0)                                        # <n|O_-|n + 1>
    if op == OP_Z:
        return 0, z
    if op == OP_Z2:
        return 0, z * z
    if op == OP_RAISE:
        return 1, up
    if op == OP_LOWER:
        return -1, down
    if op == OP_RAISE2:
        return 2, up * np.append(0.0, up[:-1])
    assert op == OP_LOWER2
    return -2, down * np.append(down[1:], 0.0)


def _matvec_flops(model):
    """Multiply-adds of the diagonal and of the admissible off-diagonal entries (real couplings)."""
    per_row = 2.0
    for t in model.terms:
        qa, fa = _factors(model.sites[t.site_a], t.op_a)
        share = np.count_nonzero(fa) / len(fa)
        q = [qa]
        if t.site_b >= 0:
            qb, fb = _factors(model.sites[t.site_b], t.op_b)
            share *= np.count_nonzero(fb) / len(fb)
            q.append(qb)
        if any(q):
            per_row += 4.0 * share
    return per_row * model.dim


def _sector_dim(model, q):
    c = np.array([1.0])
    for s in model.sites:
        c = np.convolve(c, np.ones(s.k + 1))
    return float(c[q])


def _cheb_terms(model, h, tol=1e-12):
    """Terms of a Chebyshev series of length h over an interval of half-width about the bonds' norms."""
    a = sum(float(model.theta[t.param]) * abs(t.w) * np.abs(_factors(model.sites[t.site_a], t.op_a)[1]).max() *
            (np.abs(_factors(model.sites[t.site_b], t.op_b)[1]).max() if t.site_b >= 0 else 1.0)
            for t in model.terms) * 0.45
    z = abs(a * h)
    k = 1
    while k * math.log(2 * k / (math.e * z + 1e-9)) < -math.log(tol) or k < z:
        k += 1
    return k


def work(case):
    """Each input read once and each output written once.  Lanczos: per step the matvec, the recurrence's last two
    vectors and, for full reorthogonalisation, one read of the basis; the Ritz vector reads the basis once more.
    Propagation: per term of the series the state, the previous term and the accumulator."""
    kind = case["kind"]
    if kind == "batch":
        models = _models(case)
        D = sum(m.dim for m in models)
        return {"bytes": 16.0 * D * case["nvec"], "flops": case["nvec"] * sum(map(_matvec_flops, models))}
    model = _model(case)
    D = float(model.dim)
    share = 1.0
    if kind == "sector" or case.get("sector"):
        share = _sector_dim(model, _digit_sum(model)) / D
    D *= share
    flops = _matvec_flops(model) * share
    if kind == "sweep":
        K, nv = case["points"], case["nvec"]
        return {"bytes": 8.0 * nv * D * (1 + K), "flops": nv * (flops + 4.0 * K * model.n_params * D)}
    if kind in ("matvec", "sector"):
        return {"bytes": (32.0 if case["dtype"] == "c128" else 16.0) * D, "flops": flops}
    if kind == "autograd":
        return {"bytes": (2 + 3) * 16.0 * D, "flops": 3.0 * flops}
    if kind == "lanczos":
        m = case["m"]
        full = case["reorth"] != "partial"
        vectors = m * 4 + (m * (m + 1) / 2 if full else 0) + m + 1
        return {"bytes": 16.0 * D * vectors, "flops": m * flops + 16.0 * D * (m * m / 2 if full else m)}
    steps = case["steps"] if case["drive"] else 1
    terms = steps * _cheb_terms(model, case["dt"] * (1 if case["drive"] else case["steps"]))
    return {"bytes": 16.0 * D * 5 * terms, "flops": terms * (flops + 12.0 * D)}


# ------------------------------------------------------------------------------------------------ in 64 bits
def _apply(model, theta, x, only=None):
    """H(theta) x by slices of the tensor that x is (site 0 first): one slice per entry of a local matrix.
    x: complex128 [D] or [D, nvec]; only: the terms of that parameter, with weight 1."""
    dims = [s.k + 1 for s in model.sites]
    nv = x.numel() // model.dim
    y = torch.zeros_like(x)
    diag = torch.zeros(model.dim, dtype=torch.float64, device=x.device)
    for t in model.terms:
        if only is not None and t.param != only:
            continue
        w = complex(t.w) * (1.0 if only is not None else float(theta[t.param]))
        assert w.imag == 0.0
        w = w.real
        a, oa, b, ob = t.site_a, t.op_a, t.site_b, t.op_b
        if b >= 0 and b < a:
            a, oa, b, ob = b, ob, a, oa
        qa, fa = _factors(model.sites[a], oa)
        qb, fb = _factors(model.sites[b], ob) if b >= 0 else (0, np.ones(1))
        db = dims[b] if b >= 0 else 1
        mid = math.prod(dims[a + 1: b]) if b >= 0 else 1
        low = math.prod(dims[b + 1:]) if b >= 0 else math.prod(dims[a + 1:])
        if qa == 0 and qb == 0:
            c = torch.as_tensor(w * np.outer(fa, fb), device=x.device).view(1, dims[a], 1, db, 1)
            diag.view(-1, dims[a], mid, db, low).add_(c)
            continue
        xv, yv = (v.view(-1, dims[a], mid, db, low * nv) for v in (x, y))
        for na in range(dims[a]):
            for nb in range(db):
                f = fa[na] * fb[nb]
                if f != 0.0 and 0 <= na - qa < dims[a] and 0 <= nb - qb < db:
                    yv[:, na, :, nb].add_(xv[:, na - qa, :, nb - qb], alpha=float(w * f))
    y += diag.view(model.dim, *([1] * (x.dim() - 1))) * x
    return y


def _sector_rows(model, q):
    """Full-basis indices of the states whose digits sum to q, ascending (the packed order)."""
    s = torch.zeros(1, dtype=torch.int16, device=DEV)
    for site in model.sites:
        s = (s.view(-1, 1) + torch.arange(site.k + 1, dtype=torch.int16, device=DEV)).reshape(-1)
    return torch.nonzero(s == q).view(-1)


def _in_space(model, theta, rows):
    """v -> H v, or P H P^T v on packed vectors."""
    if rows is None:
        return lambda v: _apply(model, theta, v)

    def mv(v):
        full = torch.zeros(model.dim, dtype=v.dtype, device=v.device)
        full[rows] = v
        return _apply(model, theta, full)[rows]
    return mv


def _exact_lanczos(mv, v0, m):
    """The recurrence with two Gram-Schmidt passes at every step."""
    V = torch.empty((m + 1, v0.numel()), dtype=torch.complex128, device=v0.device)
    V[0] = v0 / torch.linalg.vector_norm(v0)
    alpha, beta = torch.zeros(m, dtype=torch.float64), torch.zeros(m, dtype=torch.float64)
    for j in range(m):
        w = mv(V[j])
        alpha[j] = torch.vdot(V[j], w).real.item()
        w = w - alpha[j].item() * V[j]
        if j:
            w -= beta[j - 1].item() * V[j - 1]
        for _ in range(2):
            for i in range(j + 1):
                w -= torch.vdot(V[i], w) * V[i]
        beta[j] = torch.linalg.vector_norm(w).item()
        V[j + 1] = w / beta[j].item()
    T = torch.diag(alpha) + torch.diag(beta[:-1], 1) + torch.diag(beta[:-1], -1)
    # the sign of the Ritz vector is free, so it has no one value
    return {"alpha": alpha, "beta": beta, "energy": torch.linalg.eigvalsh(T)[:1], "u": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        models, nv = _models(case), case["nvec"]
        offs, total = [], 0
        for m in models:
            offs.append(total)
            total += (m.dim * nv + 31) // 32 * 32
        X = _blocks(offs, total, [m.dim for m in models], nv, seed)
        Y = torch.zeros(total, dtype=torch.complex128, device=DEV)
        for b, (m, o) in enumerate(zip(models, offs)):
            th = _couplings(m, seed * 1013 + b).float().double()
            x = X[o: o + m.dim * nv].view(m.dim, nv).to(torch.complex128)
            Y[o: o + m.dim * nv] = _apply(m, th, x).reshape(-1)
        return Y
    model = _model(case)
    if kind == "sweep":
        nv, K = case["nvec"], case["points"]
        th = _couplings(model, seed, K).float().double()
        x = _state((model.dim, nv), "c64", seed * 11 + 3).to(torch.complex128)
        n = model.dim * nv
        stride = (n + 31) // 32 * 32
        G = [_apply(model, None, x, only=p).reshape(-1) for p in range(model.n_params)]
        Y = torch.zeros((K, stride), dtype=torch.complex128, device=DEV)
        for k in range(K):
            for p, g in enumerate(G):
                Y[k, :n].add_(g, alpha=float(th[k, p]))
        # entries between the blocks are nobody's: there is a value only where there are none
        return Y.reshape(-1) if stride == n else None
    theta, vecs = _inputs(case, seed, model)
    if case.get("dtype") == "c64":
        theta = theta.float().double()
    x = vecs[0].to(torch.complex128)
    rows = _sector_rows(model, _digit_sum(model)) if kind == "sector" or case.get("sector") else None
    if kind in ("matvec", "sector"):
        return _in_space(model, theta, rows)(x)
    if kind == "autograd":
        g = vecs[1]
        gt = torch.stack([torch.vdot(g, _apply(model, None, x, only=p)).real for p in range(model.n_params)])
        return {"y": _apply(model, theta, x), "grad_theta": gt, "grad_x": _apply(model, theta, g)}
    if kind == "lanczos":
        return _exact_lanczos(_in_space(model, theta, rows), x, case["m"])
    # exp(-i H dt) by its Taylor series, in substeps short enough that it converges without cancellation
    for s in range(case["steps"]):
        th = theta[s] if case["drive"] else theta
        mv, sub = _in_space(model, th, None), 8
        for _ in range(sub):
            term = x.clone()
            for k in range(1, 40):
                term = mv(term) * (-1j * case["dt"] / sub / k)
                x = x + term
                if torch.linalg.vector_norm(term).item() < 1e-17:
                    break
    return x
