"""The performance cases of the library: what a chemistry host model has it do.

One case is one pass through the public binding (paper_2501_00011_amd.mcchem and
.autograd) on inputs made from a seed.  The kinds:

  deriv  f at y                                            Cells.deriv
  fj     f and the sparse Jacobian at y                    Cells.deriv_jac
  vjp    J^T v and d(v.f)/d ln k at y                      Cells.vjp
  solve  rate constants of the new environment, then one
         or several consecutive outer BDF steps            Cells.bind, Cells.step
  multi  the same with all cells as one system             Cells.bind, Cells.step_multicell
  grad   one outer step and its reverse pass               autograd.solve_step

Mechanisms: `synth.make_mechanism` with the sizes of the repository's workloads
(20 / 30, 72 / 156 and 150 / 350 species / reactions) in the listed cases, and
sizes between them (and smaller) in the drawn ones.  Everything is float64, the
library's only type.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2501_00011_amd import autograd, mcchem, synth

DEV = "cuda:0"


def listed():
    return [
        # a handful of cells (a box model): launches and host time
        dict(name="deriv_20x10", kind="deriv", species=20, reactions=30, cells=10, dt=60.0),
        # the right-hand side and Jacobian handed to an outside solver: the usual batch, ...
        dict(name="fj_72x10000", kind="fj", species=72, reactions=156, cells=10000, dt=180.0),
        # ... and a regional domain beyond the caches, an odd count (rows not 16-byte aligned)
        dict(name="fj_72x130001", kind="fj", species=72, reactions=156, cells=130001, dt=180.0),
        # reverse mode of f inside a gradient code
        dict(name="vjp_72x10000", kind="vjp", species=72, reactions=156, cells=10000, dt=180.0),
        # one step of a box model
        dict(name="solve_20x10", kind="solve", species=20, reactions=30, cells=10, dt=60.0, thermal=True),
        # the small mechanism's share of a mixed domain
        dict(name="solve_20x30000", kind="solve", species=20, reactions=30, cells=30000, dt=60.0),
        # the headline batch as the benchmark runs it: the autotuner's dense tail, cells
        # ordered by the counters of an earlier step
        dict(name="solve_72x10000", kind="solve", species=72, reactions=156, cells=10000, dt=180.0, tail=32,
             balanced=True),
        # one column block of a domain with the library's own choices
        dict(name="solve_72x1003", kind="solve", species=72, reactions=156, cells=1003, dt=60.0),
        # a host model's time loop: consecutive outer steps, the state advancing, step sizes kept
        dict(name="loop_72x4000", kind="solve", species=72, reactions=156, cells=4000, dt=60.0, steps=4, tail=32),
        # the large mechanism
        dict(name="solve_150x1000", kind="solve", species=150, reactions=350, cells=1000, dt=60.0),
        # a gradient of one outer step
        dict(name="grad_72x1000", kind="grad", species=72, reactions=156, cells=1000, dt=60.0, tail=32),
        # the shared-step mode
        dict(name="multi_20x500", kind="multi", species=20, reactions=30, cells=500, dt=60.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, species log-uniform from 8 to 160, cells
    log-uniform up to what costs about as much as the largest listed case of
    that kind.  (A mechanism's f/J kernels are compiled on their first call,
    so those kinds stay at 96 species.)"""
    kind = rng.choice(["deriv", "fj", "vjp", "solve", "solve", "solve", "solve", "grad", "multi"])
    top = {"solve": 160, "grad": 96, "multi": 32}.get(kind, 96)
    n = _log_int(rng, 8, top)
    c = dict(kind=kind, species=n, reactions=int(n * rng.uniform(1.6, 2.4)), dt=rng.choice([60.0, 180.0]))
    if kind in ("deriv", "fj", "vjp"):
        c["cells"] = _log_int(rng, 10, 120000 * 72 // max(n, 72))
    elif kind == "solve":
        # a cell's cost grows about with the square of the species, and faster beyond 100
        c["cells"] = _log_int(rng, 10, min(30000, int(6000 * (72.0 / n) ** (2.0 if n <= 100 else 2.6))))
        c["steps"] = rng.choice([1, 1, 2])
        if 33 <= n <= 96 and rng.random() < 0.5:
            c["tail"] = 32
        c["balanced"] = rng.random() < 0.3
    elif kind == "grad":
        c["cells"] = _log_int(rng, 10, min(2000, int(800 * (72.0 / n) ** 2)))
    else:
        c["cells"] = _log_int(rng, 10, 400)
    return c


def _mechanism(case):
    n, r = case["species"], case["reactions"]
    if case.get("thermal"):
        return synth.make_mechanism(n, r, (40, 50, 10), first_order="thermal", seed=n)
    return synth.make_mechanism(n, r, (30, 60, 10), first_order="photolysis", seed=n)


def _cells(m, case, seed):
    return synth.make_cells(m, case["cells"], seed=seed, jscale_log10_range=(-1.0, 0.0))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _cotangent(case, seed, y):
    """A loss gradient with respect to f or y(dt): relative deviations of the
    species, so of the size of 1 / y."""
    g = torch.Generator().manual_seed(seed)
    v = torch.randn(y.shape, generator=g, dtype=torch.float64)
    return (v / (np.abs(y) + 1e3)).to(DEV)


def prepare(case, seed):
    """A compiled mechanism, a batch of cells and device arrays, as a program
    sets them up once and keeps them; the inputs of the pass."""
    m = _mechanism(case)
    c = _cells(m, case, seed)
    mech = mcchem.Mechanism(m, device=0, dense_tail=case.get("tail", -1))
    cells = mcchem.Cells(mech, c.n_cells)
    s = dict(case=case, mech=mech, cells=cells, T=_dev(c.T), P=_dev(c.P), j=_dev(c.jscale), y0=_dev(c.y0))
    cells.bind(s["T"], s["P"], s["j"])
    kind, C = case["kind"], c.n_cells
    if kind in ("deriv", "fj", "vjp"):
        # the mechanism's kernels are compiled by its first such call
        s["f"] = cells.deriv(s["y0"])
        if kind == "fj":
            s["jac"] = torch.empty((mech.nnz, C), dtype=torch.float64, device=DEV)
        if kind == "vjp":
            s["v"] = _cotangent(case, seed, c.y0)
            s["glnk"] = torch.empty((mech.n_reactions, C), dtype=torch.float64, device=DEV)
    elif kind == "grad":
        s["lnk"] = torch.log(cells.rate_constants())
        s["g"] = _cotangent(case, seed, c.y0)
    else:
        s["y"] = s["y0"].clone()
        s["status"] = torch.empty(C, dtype=torch.int32, device=DEV)
        s["stats"] = torch.empty((C, mcchem.STATS_DTYPE.itemsize), dtype=torch.uint8, device=DEV)
        s["cold"] = mcchem.default_opts()
        s["warm"] = mcchem.default_opts(warm_start=1)
        if case.get("balanced"):
            cells.step(s["y"], case["dt"], s["cold"], status=s["status"], stats=s["stats"])
            cells.balance(s["stats"])
    return s


def run(state):
    s = state
    case, cells = s["case"], s["cells"]
    kind = case["kind"]
    if kind == "deriv":
        return {"f": cells.deriv(s["y0"], s["f"])}
    if kind == "fj":
        f, jac = cells.deriv_jac(s["y0"], s["f"], s["jac"])
        return {"f": f, "jac": jac}
    if kind == "vjp":
        gy, glnk = cells.vjp(s["y0"], s["v"], s["f"], s["glnk"])
        return {"gy": gy, "glnk": glnk}
    if kind == "grad":
        y0 = s["y0"].detach().requires_grad_(True)
        lnk = s["lnk"].detach().requires_grad_(True)
        y = autograd.solve_step(cells, y0, lnk, case["dt"])
        gy, glnk = torch.autograd.grad(y, (y0, lnk), s["g"])
        return {"y": y.detach(), "gy": gy, "glnk": glnk}
    y = s["y"]
    y.copy_(s["y0"])
    if kind == "multi":
        cells.bind(s["T"], s["P"], s["j"])
        cells.step_multicell(y, case["dt"], s["cold"], status=s["status"], stats=s["stats"])
        return {"y": y, "status": s["status"]}
    for i in range(case.get("steps", 1)):
        cells.bind(s["T"], s["P"], s["j"])  # the environment of this outer step
        cells.step(y, case["dt"], s["cold"] if i == 0 else s["warm"], status=s["status"], stats=s["stats"])
    return {"y": y, "status": s["status"]}


def work(case):
    """Bytes: every input read and every output written once.  Flops: the
    library's own counts per f, Jacobian, factorisation and solve (no padding);
    for the solver times the step attempts that such cells take (about 700 in
    the first step after a disturbance, 65 in a later one; two Newton
    iterations each), for the shared-step mode three times as many."""
    m = _mechanism(case)
    h = mcchem.Mechanism(m, device=-1)
    oc, C = h.op_counts(), case["cells"]
    N, R, nnz = h.n_species, h.n_reactions, h.nnz
    terms = len(m.reac_idx) + len(m.prod_idx)
    kind = case["kind"]
    if kind == "deriv":
        return {"bytes": C * oc["f_bytes"], "flops": C * oc["deriv_flops"]}
    if kind == "fj":
        return {"bytes": C * oc["fj_bytes"], "flops": C * (oc["deriv_flops"] + oc["newton_matrix_flops"])}
    if kind == "vjp":
        return {"bytes": C * 8 * (3 * N + 2 * R), "flops": C * 6 * terms}
    attempt = 2 * oc["deriv_flops"] + oc["newton_matrix_flops"] + oc["lu_flops"] + 2 * oc["solve_flops"]
    steps = case.get("steps", 1)
    attempts = 700 + 65 * (steps - 1)
    io = C * steps * (8 * (2 * N + 3) + 60)
    if kind == "grad":
        back = oc["newton_matrix_flops"] + oc["lu_flops"] + oc["solve_flops"] + oc["deriv_flops"]
        return {"bytes": C * 8 * (4 * N + 2 * R), "flops": C * attempts * (attempt + back)}
    return {"bytes": io, "flops": C * attempts * attempt * (3 if kind == "multi" else 1)}


# ---------------------------------------------------------------------------
# The same values from the definitions, in plain torch.
# ---------------------------------------------------------------------------

class _Plain:
    """r_j = k_j prod y over the reactant slots, nu = products - reactants."""

    def __init__(self, m, device):
        self.m, N, R = m, m.n_species, m.n_reactions
        self.slots = np.full((3, R), -1)
        self.nu = torch.zeros((N, R), dtype=torch.float64)
        for j in range(R):
            for q, s in enumerate(m.reac_idx[m.reac_ptr[j]:m.reac_ptr[j + 1]]):
                self.slots[q, j] = s
                self.nu[s, j] -= 1.0
            for e in range(m.prod_ptr[j], m.prod_ptr[j + 1]):
                self.nu[m.prod_idx[e], j] += float(m.prod_yield[e])
        self.nu = self.nu.to(device)
        self.idx = torch.from_numpy(np.where(self.slots < 0, N, self.slots)).to(device)  # N: the constant 1
        self.device = device

    def k(self, T, j):
        A, th = (torch.from_numpy(np.ascontiguousarray(a)).to(self.device)[:, None] for a in (self.m.A, self.m.theta))
        photo = torch.from_numpy(self.m.rxn_type == synth.RXN_PHOTOLYSIS).to(self.device)[:, None]
        return torch.where(photo, A * j[None], A * torch.exp(-th / T[None]))

    def factors(self, y):
        e = torch.cat([y, torch.ones_like(y[:1])])
        return e[self.idx[0]], e[self.idx[1]], e[self.idx[2]]

    def rates(self, k, y):
        a, b, c = self.factors(y)
        return k * a * b * c

    def partials(self, k, y):
        """d r_j / d y through each reactant slot, [3][R][cells]; 0 where the slot is empty."""
        a, b, c = self.factors(y)
        p = torch.stack([k * b * c, k * a * c, k * a * b])
        return torch.where((self.idx < self.m.n_species)[:, :, None], p, torch.zeros_like(p))

    def deriv(self, k, y):
        return self.nu @ self.rates(k, y)


def exact(case, seed):
    """f, J and the products from their definitions, in blocks of cells; a
    small batch's solution of the ODE by the three-stage Radau IIA method on a
    fine geometric grid (error far below the solver's tolerance); None for the
    larger solves and for the discrete gradient."""
    m = _mechanism(case)
    kind, N, R, C = case["kind"], case["species"], case["reactions"], case["cells"]
    if kind in ("solve", "multi"):
        if N > 24 or C > 16 or case.get("steps", 1) > 1:
            return None
        c = _cells(m, case, seed)
        p = _Plain(m, "cpu")
        k = p.k(torch.from_numpy(c.T), torch.from_numpy(c.jscale))
        return {"y": _radau(p, k, torch.from_numpy(c.y0), case["dt"]), "status": None}
    if kind == "grad":
        return None
    c = _cells(m, case, seed)
    p = _Plain(m, DEV)
    pat = [set((i,)) for i in range(N)]
    nu_np = p.nu.cpu().numpy()
    for j in range(R):
        touched = set(m.reac_idx[m.reac_ptr[j]:m.reac_ptr[j + 1]]) | set(m.prod_idx[m.prod_ptr[j]:m.prod_ptr[j + 1]])
        for i in touched:
            pat[int(i)].update(int(s) for s in p.slots[:, j] if s >= 0)
    rows = np.concatenate([np.full(len(x), i) for i, x in enumerate(pat)])
    cols = np.concatenate([np.array(sorted(x)) for x in pat])
    f = torch.empty((N, C), dtype=torch.float64, device=DEV)
    jac = torch.empty((len(rows) if kind == "fj" else 0, C), dtype=torch.float64, device=DEV)
    glnk = torch.empty((R if kind == "vjp" else 0, C), dtype=torch.float64, device=DEV)
    v = _cotangent(case, seed, c.y0) if kind == "vjp" else None
    y_all, k_all = _dev(c.y0), p.k(_dev(c.T), _dev(c.jscale))
    if kind == "fj":  # entry e of J: sum over (slot q, reaction j) with slot species cols[e] of nu[rows[e], j] * partial
        at = {(int(r), int(s)): e for e, (r, s) in enumerate(zip(rows, cols))}
        w = np.zeros((len(rows), 3 * R))
        for j in range(R):
            for q in range(3):
                s = int(p.slots[q, j])
                for i in np.flatnonzero(nu_np[:, j]) if s >= 0 else ():
                    w[at[(int(i), s)], q * R + j] += nu_np[i, j]
        w = torch.from_numpy(w).to(DEV)
    for b in range(0, C, 20000):
        y, k = y_all[:, b:b + 20000], k_all[:, b:b + 20000]
        if kind != "vjp":
            f[:, b:b + 20000] = p.deriv(k, y)
        if kind == "fj":
            jac[:, b:b + 20000] = w @ p.partials(k, y).reshape(3 * R, -1)
        if kind == "vjp":
            u = p.nu.T.contiguous() @ v[:, b:b + 20000]  # sum_i nu_ij v_i
            g = torch.zeros((N + 1, y.shape[1]), dtype=torch.float64, device=DEV)
            part = p.partials(k, y)
            for q in range(3):
                g.index_add_(0, p.idx[q], part[q] * u)
            f[:, b:b + 20000] = g[:N]
            glnk[:, b:b + 20000] = p.rates(k, y) * u
    if kind == "deriv":
        return {"f": f}
    return {"f": f, "jac": jac} if kind == "fj" else {"gy": f, "glnk": glnk}


def _radau(p, k, y, dt):
    """y(dt) by Radau IIA of order 5, simplified Newton with the Jacobian of the
    step's start, all cells at once; steps grow by 5 % from 1e-9 s."""
    N, C = y.shape
    r6 = math.sqrt(6.0)
    a = torch.tensor([[(88 - 7 * r6) / 360, (296 - 169 * r6) / 1800, (-2 + 3 * r6) / 225],
                      [(296 + 169 * r6) / 1800, (88 + 7 * r6) / 360, (-2 - 3 * r6) / 225],
                      [(16 - r6) / 36, (16 + r6) / 36, 1 / 9]], dtype=torch.float64)
    t, eye = 0.0, torch.eye(3 * N, dtype=torch.float64)
    while t < dt:
        h = min(1e-9 if t == 0.0 else 0.05 * t, dt - t)
        part = p.partials(k, y)
        jac = torch.zeros((C, N, N + 1), dtype=torch.float64)
        for q in range(3):
            for j in range(p.idx.shape[1]):
                jac[:, :, int(p.idx[q, j])] += part[q, j][:, None] * p.nu[:, j][None]
        big = eye - h * torch.einsum("ab,cij->caibj", a, jac[:, :, :N]).reshape(C, 3 * N, 3 * N)
        lu = torch.linalg.lu_factor(big)
        z = torch.zeros((3, N, C), dtype=torch.float64)
        for _ in range(12):
            fs = torch.stack([p.deriv(k, y + z[i]) for i in range(3)])
            res = h * torch.tensordot(a, fs, 1) - z
            d = torch.linalg.lu_solve(*lu, res.permute(2, 0, 1).reshape(C, 3 * N, 1)).reshape(C, 3, N).permute(1, 2, 0)
            z = z + d
            if float((d.abs() / (y.abs() + 1.0)).max()) < 1e-13:
                break
        y = y + z[2]
        t = dt if t + h >= dt else t + h
    return y
