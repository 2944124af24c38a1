"""Performance cases of the generalized shifted COCG library.

Each case is one piece of work a program gives the library through
``paper_1002_1202_amd.api``: a product with the pair, Green's-function
elements, charges, gradients and forces, on synthetic silicon (4x4 sp3 blocks,
second-shell pattern) and water (6x6 molecule blocks, 6 A cutoff).  Inputs are
made here from a seed: geometries, angular factors and the ASED values of H and
S.  ``exact`` gives the same outputs from a dense generalized eigenproblem in
64 bits wherever that is affordable.

Tolerances are the tight ones in use (1e-10; 1e-12 for gradients): two orders
of summation then agree to 1e-10, where at 1e-6 a shift that freezes one
iteration later moves the outputs by 1e-8.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1002_1202_amd import api

A_SI = 5.431                                       # diamond lattice constant, A
SI_BASIS = np.array([[0, 0, 0], [0, 2, 2], [2, 0, 2], [2, 2, 0],
                     [1, 1, 1], [1, 3, 3], [3, 1, 3], [3, 3, 1]])      # units of A_SI / 4
SI_LEVELS = (-13.6, -6.5, -6.5, -6.5)              # 3s, 3p, eV
WATER_LEVELS = (-32.3, -14.8, -14.8, -14.8, -13.6, -13.6)             # O 2s, 2p, H 1s
WATER_DENSITY = 0.03343                            # molecules per A^3
WATER_CUTOFF = 6.0
WATER_U = (13.5, 11.4, 11.4)                       # on-site hardness O, H, H (eV)
ASED = SimpleNamespace(s0=0.3, r0=2.35, lam=0.8, kappa=1.75, theta=0.5)
EXACT_N = 2600                                     # largest dense eigenproblem of exact()


# ------------------------------------------------------------------ geometries
def _block_csr(nb, i, j, trans, ang, diag):
    """Symmetric block-CSR pattern from unordered pairs (i, j) and the diagonal."""
    rows = np.concatenate([i, j, np.arange(nb)])
    cols = np.concatenate([j, i, np.arange(nb)])
    t = np.concatenate([trans, -trans, np.zeros((nb, 3))])
    a = np.concatenate([ang, ang.transpose(0, 2, 1), diag])
    order = np.argsort(rows * nb + cols, kind="stable")
    rowptr = np.zeros(nb + 1, np.int64)
    np.cumsum(np.bincount(rows, minlength=nb), out=rowptr[1:])
    return rowptr, cols[order].astype(np.int32), t[order], np.ascontiguousarray(a[order])


def _silicon(rng, cells, vacancies):
    """Periodic diamond Si, Gaussian displacements of 0.05 A, random vacancies
    (their places, and so the pattern, belong to the case, not to the seed)."""
    dims = 4 * np.array(cells)
    cell = np.stack(np.meshgrid(*(np.arange(c) for c in cells), indexing="ij"), -1).reshape(-1, 3)
    site = (4 * cell[:, None, :] + SI_BASIS[None]).reshape(-1, 3)
    if vacancies:
        site = np.delete(site, np.random.default_rng(vacancies).choice(len(site), size=vacancies, replace=False), axis=0)
    nb = len(site)
    index = np.full(dims, -1, np.int64)
    index[tuple(site.T)] = np.arange(nb)
    shell1 = np.array([[1, 1, 1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1]])
    shell2 = np.array([[a, b, 0] for a in (2, -2) for b in (2, -2)])
    shell2 = np.concatenate([shell2, shell2[:, [0, 2, 1]], shell2[:, [2, 0, 1]]])
    sign = np.where(site[:, :1] % 2 == 0, 1, -1)       # the two sublattices
    ii, jj, image = [], [], []
    for k, off in enumerate(np.concatenate([shell1, shell2])):
        to = site + (sign * off if k < 4 else off)
        j = index[tuple((to % dims).T)]
        use = j > np.arange(nb)
        ii.append(np.arange(nb)[use])
        jj.append(j[use])
        image.append((to // dims)[use])
    i, j = np.concatenate(ii), np.concatenate(jj)
    trans = np.concatenate(image) * (np.array(cells) * A_SI)
    ang = rng.uniform(-1.0, 1.0, size=(len(i), 4, 4))
    rowptr, colidx, t, a = _block_csr(nb, i, j, trans, ang, np.zeros((nb, 4, 4)))
    pos = site * (A_SI / 4) + rng.normal(0.0, 0.05, size=(nb, 3))
    return SimpleNamespace(block=4, n=4 * nb, n_atoms=nb, positions=pos, orb_atom=np.repeat(np.arange(nb), 4),
                           eps=np.tile(SI_LEVELS, nb), rowptr=rowptr, colidx=colidx, trans=t, ang=a, params=ASED)


def _water(rng, n_mol):
    """Rigid molecules on a jittered grid at 1 g/cm^3 with random orientations.
    The box and its pattern belong to the case; the seed moves the molecules by
    0.05 A inside it, as a step of a trajectory with a frozen pattern does."""
    frame = np.random.default_rng(n_mol)
    box = (n_mol / WATER_DENSITY) ** (1.0 / 3.0)
    g = math.ceil(round(n_mol ** (1.0 / 3.0), 9))
    grid = np.stack(np.meshgrid(*[np.arange(g)] * 3, indexing="ij"), -1).reshape(-1, 3)
    pick = np.sort(frame.choice(len(grid), size=n_mol, replace=False))
    o = (grid[pick] + 0.5) * (box / g) + frame.uniform(-0.3, 0.3, size=(n_mol, 3))
    rot = np.linalg.qr(rng.normal(size=(n_mol, 3, 3)))[0]
    half = math.radians(104.52) / 2
    arm = 0.9572 * np.array([[math.sin(half), 0, math.cos(half)], [-math.sin(half), 0, math.cos(half)]])
    h = o[:, None, :] + np.matmul(arm, rot.transpose(0, 2, 1))
    pos = np.concatenate([o[:, None], h], 1).reshape(-1, 3)
    ii, jj = [], []
    for s in range(0, n_mol, 512):
        d = o[None, :] - o[s:s + 512, None]
        d -= box * np.round(d / box)
        near = (d * d).sum(-1) < WATER_CUTOFF ** 2
        a, b = np.nonzero(near & (np.arange(n_mol)[None, :] > np.arange(s, min(s + 512, n_mol))[:, None]))
        ii.append(a + s)
        jj.append(b)
    i, j = np.concatenate(ii), np.concatenate(jj)
    trans = -np.round((o[j] - o[i]) / box) * box
    pos += np.repeat(rng.normal(0.0, 0.05, size=(n_mol, 3)), 3, axis=0)
    ang = rng.uniform(-1.0, 1.0, size=(len(i), 6, 6))
    own = np.triu(rng.uniform(-1.0, 1.0, size=(n_mol, 6, 6)), 1)
    rowptr, colidx, t, a = _block_csr(n_mol, i, j, trans, ang, own + own.transpose(0, 2, 1))
    orb_atom = (3 * np.arange(n_mol)[:, None] + np.array([0, 0, 0, 0, 1, 2])).reshape(-1)
    return SimpleNamespace(block=6, n=6 * n_mol, n_atoms=3 * n_mol, positions=pos, orb_atom=orb_atom,
                           eps=np.tile(WATER_LEVELS, n_mol), rowptr=rowptr, colidx=colidx, trans=t, ang=a,
                           params=ASED)


def _system(text, rng):
    """"si 4x4x4-5": cells and number of vacancies; "water 64": molecules."""
    kind, size = text.split()
    if kind == "water":
        return _water(rng, int(size))
    cells, vacancies = (size + "-0").split("-")[:2]
    return _silicon(rng, tuple(int(c) for c in cells.split("x")), int(vacancies))


def _orbitals(text):
    """Number of orbitals N of a system text."""
    kind, size = text.split()
    if kind == "water":
        return 6 * int(size)
    cells, vacancies = (size + "-0").split("-")[:2]
    return 4 * (8 * math.prod(int(c) for c in cells.split("x")) - int(vacancies))


def _nonzeros(text):
    """Stored entries of one matrix: 17 blocks a row (Si), about 27 (water)."""
    n = _orbitals(text)
    return n * 6 * min(27, n // 6) if text.startswith("water") else n * 68


def _values(s):
    """ASED values of S and H (eq. Hap-1) on the pattern."""
    B = s.block
    row = np.repeat(np.arange(len(s.rowptr) - 1), np.diff(s.rowptr))
    o1 = row[:, None] * B + np.arange(B)
    o2 = s.colidx[:, None].astype(np.int64) * B + np.arange(B)
    u, v = s.orb_atom[o1], s.orb_atom[o2]
    d = s.positions[v][:, None, :, :] + s.trans[:, None, None, :] - s.positions[u][:, :, None, :]
    r = np.sqrt((d * d).sum(-1))
    own = (u[:, :, None] == v[:, None, :]) & ~s.trans.any(1)[:, None, None]
    S = np.where(own, 0.0, ASED.s0 * np.exp(-(r - ASED.r0) / ASED.lam) * s.ang)
    rows = np.zeros(s.n)
    np.add.at(rows, o1.reshape(-1), np.abs(S).sum(2).reshape(-1))
    S *= ASED.theta / rows.max()
    H = 0.5 * ASED.kappa * (s.eps[o1][:, :, None] + s.eps[o2][:, None, :]) * S
    same = own & (o1[:, :, None] == o2[:, None, :])
    return np.where(same, 1.0, S), np.where(same, s.eps[o1][:, :, None], H)


# ------------------------------------------------------------------ inputs of a case
def _grid(case, lo=None, hi=None):
    """Shifts E_k + i eta on the system's spectrum and their trapezoid weights."""
    wide = (-40.0, 5.0) if case["system"].startswith("water") else (-20.0, 5.0)
    lo, hi = lo or wide[0], hi or wide[1]
    e = np.linspace(lo, hi, case["shifts"])
    w = np.full(case["shifts"], (hi - lo) / max(1, case["shifts"] - 1))
    w[0] *= 0.5
    w[-1] *= 0.5
    return e + 1j * case["eta"], w


def _pick(rng, s, count):
    """All orbitals of random blocks, cut to `count`."""
    blocks = rng.choice(s.n // s.block, size=-(-count // s.block), replace=False)
    return (blocks[:, None] * s.block + np.arange(s.block)).reshape(-1)[:count].astype(np.int64)


def _members(case):
    """Systems of a batch: "system:shifts:rhs" separated by commas."""
    for text in case["members"].split(","):
        system, shifts, rhs = text.split(":")
        yield dict(case, system=system, shifts=int(shifts), rhs=int(rhs))


def _inputs(case, seed):
    """Host inputs of one case (every member of a batch), from the seed alone."""
    rng = np.random.default_rng([seed, 17])
    if case["kind"] == "batch":
        return [_one(c, rng) for c in _members(case)]
    return _one(case, rng)


def _one(case, rng):
    s = _system(case["system"], rng)
    d = SimpleNamespace(s=s, rng=rng)
    d.S, d.H = _values(s)
    rhs = case.get("rhs", 0)
    if case["kind"] == "product":
        d.X = rng.normal(size=(s.n, rhs)) + 1j * rng.normal(size=(s.n, rhs))
        d.alpha = rng.uniform(-20.0, 5.0, rhs) + 0.05j
    elif case["kind"] in ("force", "loss"):
        # up to a Fermi level in the gap, as for a band energy
        d.z, d.w = _grid(case, hi=-12.0 if s.block == 6 else -6.65)
        d.orbs = _pick(rng, s, rhs) if rhs else np.arange(s.n)
        d.qbar = rng.normal(size=len(d.orbs))
    else:
        d.z, d.w = _grid(case)
        d.orbs = _pick(rng, s, rhs) if rhs else np.arange(s.n)
        d.dq = 0.05 * rng.normal(size=s.n_atoms)
    return d


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one product z S X - H X of the smallest workload (64 Si atoms, 8 columns): a call's fixed cost
        dict(name="product_small", kind="product", system="si 2x2x2", rhs=8),
        # the same on 8,192 atoms with a ragged block of columns: a caller's own residual check or Krylov loop
        dict(name="product_large", kind="product", system="si 8x8x16", rhs=250),
        # plain method on 64 Si atoms: 8 columns of G at 64 energies, in host memory
        dict(name="green_si64", kind="green", system="si 2x2x2", shifts=64, rhs=8, eta=0.1, tol=1e-10,
             precision="fp64", relax=False, host=True),
        # the headline: 4,096 atoms, every column of G of 64 atoms at 256 energies, in device memory
        dict(name="green_si4096", kind="green", system="si 8x8x8", shifts=256, rhs=256, eta=0.05, tol=1e-10,
             precision="fp64", relax=False, host=False),
        # local densities of states of a defective mid-size cell, mixed precision, ragged counts
        dict(name="ldos_si_mid", kind="ldos", system="si 4x4x5-7", shifts=101, rhs=100, eta=0.05, tol=1e-10,
             precision="mixed"),
        # one self-consistency iteration of a small water box: H from the charges, then every orbital's charge
        dict(name="scc_water24", kind="scc", system="water 24", shifts=128, eta=0.5, tol=1e-10, precision="fp64"),
        dict(name="scc_water256", kind="scc", system="water 256", shifts=128, eta=0.5, tol=1e-10, precision="fp64"),
        # the charges of 16 molecules of the 3,000-molecule box at 1,024 energies
        dict(name="charges_water3000", kind="charges", system="water 3000", shifts=1024, rhs=96, eta=0.05,
             tol=1e-10, precision="mixed"),
        # an MD step: the pair from positions, band energy, its gradients on every stored entry, forces
        dict(name="force_water64", kind="force", system="water 64", shifts=64, eta=0.1, tol=1e-12,
             precision="fp64"),
        # backward of a loss of the charges of a third of the box's orbitals
        dict(name="loss_water64", kind="loss", system="water 64", shifts=64, rhs=130, eta=0.2, tol=1e-12,
             precision="fp64"),
        # G_jj by the generalized Lanczos process on the headline system
        dict(name="lanczos_si4096", kind="lanczos", system="si 8x8x8", shifts=256, rhs=256, eta=0.05, tol=1e-10,
             precision="fp64"),
        # uneven systems solved together: LDOS and charges in mixed precision
        dict(name="batch_mixed", kind="batch", eta=0.05, tol=1e-10, precision="mixed",
             members="si 4x4x4:128:64,si 4x5x6-9:333:100,si 5x6x6-14:211:172,si 6x7x8-20:480:128,si 8x8x9:150:64"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_si(rng, lo, hi):
    """Silicon of about lo to hi atoms, near-cubic cells, up to 2 % vacancies."""
    atoms = _log(rng, lo, hi)
    a = max(2, round((atoms / 8) ** (1 / 3)))
    b = max(2, round((atoms / 8 / a) ** 0.5) + rng.randint(0, 1))
    c = max(2, min(16, round(atoms / 8 / a / b)))
    return "si %dx%dx%d-%d" % (a, b, c, rng.randint(0, 8 * a * b * c // 50))


def draw(rng):
    kind = rng.choice(["product", "green", "ldos", "scc", "charges", "force", "loss", "lanczos", "batch"])
    water = rng.random() < 0.4
    eta = rng.choice([0.05, 0.1])
    if kind == "product":
        system = "water %d" % _log(rng, 27, 3000) if water else _draw_si(rng, 64, 8192)
        return dict(kind=kind, system=system, rhs=int(_log(rng, 1, 300)))
    if kind in ("green", "ldos", "lanczos"):
        system = "water %d" % _log(rng, 27, 600) if water else _draw_si(rng, 64, 2048)
        c = dict(kind=kind, system=system, shifts=int(_log(rng, 8, 256)), rhs=int(_log(rng, 1, 250)), eta=eta,
                 tol=rng.choice([1e-10, 1e-12]), precision=rng.choice(["fp64", "mixed"]))
        c["rhs"] = min(c["rhs"], _orbitals(system))
        if kind == "green":
            c.update(relax=rng.random() < 0.25, host=rng.random() < 0.3 and _orbitals(system) < 2000)
        return c
    if kind == "scc":
        return dict(kind=kind, system="water %d" % _log(rng, 20, 256), shifts=int(_log(rng, 32, 128)),
                    eta=rng.choice([0.2, 0.5]), tol=1e-10, precision=rng.choice(["fp64", "mixed"]))
    if kind == "charges":
        system = "water %d" % _log(rng, 50, 3000) if water else _draw_si(rng, 100, 4096)
        return dict(kind=kind, system=system, shifts=int(_log(rng, 32, 1024)), rhs=int(_log(rng, 4, 128)), eta=eta,
                    tol=1e-10, precision=rng.choice(["fp64", "mixed"]))
    if kind in ("force", "loss"):
        system = "water %d" % _log(rng, 20, 96) if water else _draw_si(rng, 64, 150)
        c = dict(kind=kind, system=system, shifts=int(_log(rng, 16, 96)), eta=rng.choice([0.1, 0.2]), tol=1e-12,
                 precision=rng.choice(["fp64", "mixed"]))
        if kind == "loss":
            c["rhs"] = int(_log(rng, 8, 140))
        return c
    members = ["%s:%d:%d" % (_draw_si(rng, 200, 4000).replace(",", ""), _log(rng, 100, 500), 4 * int(_log(rng, 10, 40)))
               for _ in range(rng.randint(2, 5))]
    return dict(kind="batch", eta=0.05, tol=1e-10, precision=rng.choice(["fp64", "mixed"]),
                members=",".join(members))


# ------------------------------------------------------------------ prepare and run
_contexts = {}


def _context():
    """The program's one context, on torch's current device and stream."""
    dev = torch.cuda.current_device()
    if dev not in _contexts:
        _contexts[dev] = api.Context(dev)
    return _contexts[dev]


def prepare(case, seed):
    ctx = _context()
    data = _inputs(case, seed)
    st = SimpleNamespace(case=case, ctx=ctx, data=data)
    make = lambda d: api.Pair(ctx, d.s.block, d.s.rowptr, d.s.colidx, H=d.H, S=d.S)  # noqa: E731
    if case["kind"] == "batch":
        st.problems = [dict(pair=make(d), z=d.z, rhs=d.orbs, w=d.w) for d in data]
        return st
    st.pair = make(data)
    if case["kind"] == "product":
        st.X = torch.from_numpy(data.X).to("cuda:%d" % ctx.device)
    elif case["kind"] == "scc":
        st.H0 = torch.from_numpy(data.H).to("cuda:%d" % ctx.device)
        st.dq = torch.from_numpy(data.dq).to("cuda:%d" % ctx.device)
        st.csc = api.Csc(ctx, st.pair, data.s, np.tile(WATER_U, data.s.n_atoms // 3))
    return st


def run(st):
    case, ctx, d = st.case, st.ctx, st.data
    kind = case["kind"]
    if kind == "product":
        return api.spmm(ctx, st.pair, st.X, d.alpha)
    opt = dict(tol=case["tol"], precision=case["precision"])
    if kind == "green":
        return api.solve(ctx, st.pair, d.z, rhs=d.orbs, out="host" if case["host"] else "device",
                         inner_relax=case["relax"], **opt).G_cols
    if kind == "ldos":
        return api.solve(ctx, st.pair, d.z, rhs=d.orbs, carry="projected", proj=d.orbs[:, None], out="device",
                         **opt).G_proj
    if kind == "scc":
        st.csc.hamiltonian(st.pair, st.H0, st.dq)
    if kind in ("scc", "charges"):
        q, e, band, _ = api.mulliken_band(ctx, st.pair, d.z, d.w, d.orbs, carry="projected", **opt)
        return dict(q=q, e=e, band=band)
    if kind == "force":
        scale = api.ased_build(ctx, st.pair, d.s)
        dH, dS, band, _ = api.band_energy_vjp(ctx, st.pair, d.z, d.w, **opt)
        return dict(dH=dH, dS=dS, band=band, forces=api.ased_vjp(ctx, st.pair, d.s, scale, dH, dS))
    if kind == "loss":
        dH, dS, _ = api.charge_vjp(ctx, st.pair, d.z, d.w, d.orbs, d.qbar, **opt)
        return dict(dH=dH, dS=dS)
    if kind == "lanczos":
        return api.lanczos_green(ctx, st.pair, d.z, d.orbs, tol=case["tol"], precision=case["precision"],
                                 out="device").G_diag
    return [dict(G=o["G_jj"], q=o["q"], e=o["e"]) for o in api.solve_batched(ctx, st.problems, **opt)]


def work(case):
    """Bytes of the inputs and outputs once; operations of the Krylov process:
    about 1.2 Re-width / eta steps a column (at most N), each one product with H and
    S and one S-solve of log(200 / tol) / 2.5 products, 2 fma a complex entry."""
    if case["kind"] == "batch":
        parts = [work(dict(c, kind="charges")) for c in _members(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    n, nnz = _orbitals(case["system"]), _nonzeros(case["system"])
    cols = case.get("rhs") or n
    if case["kind"] == "product":
        return {"bytes": 16.0 * nnz + 32.0 * n * cols, "flops": 8.0 * nnz * cols}
    width = 45.0 if case["system"].startswith("water") else 25.0
    steps = min(n, 1.2 * width / case["eta"])
    flops = steps * cols * nnz * 4.0 * (2.0 + math.log(200.0 / case["tol"]) / 2.5)
    out = {"green": 16.0 * case["shifts"] * cols * n, "ldos": 16.0 * case["shifts"] * cols,
           "lanczos": 16.0 * case["shifts"] * cols, "force": 16.0 * nnz, "loss": 16.0 * nnz}
    return {"bytes": 16.0 * nnz + out.get(case["kind"], 16.0 * cols), "flops": flops * (2 if case["kind"] == "loss" else 1)}


# ------------------------------------------------------------------ exact values
def _dense(s, V):
    B, nb = s.block, len(s.rowptr) - 1
    row = np.repeat(np.arange(nb), np.diff(s.rowptr))
    out = np.zeros((nb, B, nb, B))
    out[row, :, s.colidx, :] = V
    return out.reshape(nb * B, nb * B)


def _stored(s, M):
    B, nb = s.block, len(s.rowptr) - 1
    row = np.repeat(np.arange(nb), np.diff(s.rowptr))
    return np.ascontiguousarray(M.reshape(nb, B, nb, B)[row, :, s.colidx, :])


def _modes(d, H=None):
    """Generalized eigenpairs: H C = S C diag(lam), C^T S C = 1."""
    S = _dense(d.s, d.S)
    Li = np.linalg.inv(np.linalg.cholesky(S))
    A = Li @ _dense(d.s, d.H if H is None else H) @ Li.T
    lam, V = np.linalg.eigh(0.5 * (A + A.T))
    return S, lam, Li.T @ V


def _csc_hamiltonian(d):
    """H + S (V_u + V_v) / 2 with V = gamma dq (Klopman-Ohno on coupled atom pairs)."""
    s, e2 = d.s, 14.399645
    U = np.tile(WATER_U, s.n_atoms // 3)
    row = np.repeat(np.arange(len(s.rowptr) - 1), np.diff(s.rowptr))
    V = np.zeros(s.n_atoms)
    for p in range(3):
        for q in range(3):
            u, v = 3 * row + p, 3 * s.colidx.astype(np.int64) + q
            r = s.positions[v] + s.trans - s.positions[u]
            a = 0.5 * e2 * (1.0 / U[u] + 1.0 / U[v])
            own = (u == v) & ~s.trans.any(1)
            np.add.at(V, u, np.where(own, U[u], e2 / np.sqrt((r * r).sum(1) + a * a)) * d.dq[v])
    slot = np.arange(s.block)
    v1 = V[s.orb_atom[row[:, None] * s.block + slot]][:, :, None]
    v2 = V[s.orb_atom[s.colidx[:, None].astype(np.int64) * s.block + slot]][:, None, :]
    return d.H + 0.5 * d.S * (v1 + v2)


def _charges(d, S, lam, C):
    f = (1.0 / (d.z[:, None] - lam[None, :])).imag
    P = ((S @ C) * C)[d.orbs]
    q = -2.0 / math.pi * (P @ (d.w @ f))
    e = -2.0 / math.pi * (P @ ((d.w * d.z.real) @ f))
    return dict(q=q, e=e)


def _elements(d, lam, C):
    """G_jj(z_k), [K][R]."""
    return (1.0 / (d.z[:, None] - lam[None, :])) @ (C[d.orbs].T ** 2)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        if max(_orbitals(c["system"]) for c in _members(case)) > EXACT_N:
            return None
        out = []
        for d in _inputs(case, seed):
            S, lam, C = _modes(d)
            out.append(dict(_charges(d, S, lam, C), G=_elements(d, lam, C)))
        return out
    n = _orbitals(case["system"])
    if kind != "product" and n > EXACT_N:
        return None
    if kind == "green" and 16.0 * case["shifts"] * case["rhs"] * n > 2e9:
        return None
    d = _inputs(case, seed)
    s = d.s
    if kind == "product":
        X = d.X.reshape(-1, s.block, d.X.shape[1])
        Y = np.zeros_like(X)
        row = np.repeat(np.arange(len(s.rowptr) - 1), np.diff(s.rowptr))
        for k in range(int(np.diff(s.rowptr).max())):      # the k-th block of every row that has one
            b = s.rowptr[:-1] + k
            b = b[b < s.rowptr[1:]]
            x = X[s.colidx[b]]
            for c in range(s.block):
                Y[row[b]] += (d.S[b][:, :, c, None] * d.alpha - d.H[b][:, :, c, None]) * x[:, None, c]
        return Y.reshape(d.X.shape)
    if kind == "scc":
        S, lam, C = _modes(d, _csc_hamiltonian(d))
    else:
        S, lam, C = _modes(d)
    if kind in ("scc", "charges"):
        out = _charges(d, S, lam, C)
        return dict(out, band=float(out["e"].sum()))
    if kind == "ldos":
        return _elements(d, lam, C)[:, :, None]
    if kind == "lanczos":
        return _elements(d, lam, C)
    f = 1.0 / (d.z[:, None] - lam[None, :])
    if kind == "green":
        return np.stack([(C[d.orbs] * f[k]) @ C.T for k in range(len(d.z))])
    if kind == "force":
        wE = (d.w * d.z.real)[:, None]
        gH = -2.0 / math.pi * (C * (wE * f * f).imag.sum(0)) @ C.T
        gS = -2.0 / math.pi * (C * (wE * (f - d.z[:, None] * f * f)).imag.sum(0)) @ C.T
        return dict(dH=_stored(s, gH), dS=_stored(s, gS), band=float(-2.0 / math.pi * (wE * f).imag.sum()),
                    forces=None)
    Q = np.zeros(n)
    np.add.at(Q, d.orbs, d.qbar)
    M = C.T @ (S * Q) @ C                                   # modes of S Q
    fH = np.einsum("ki,kj->ij", d.w[:, None] * f, f).imag
    fS = np.einsum("ki,kj->ij", (d.w * d.z)[:, None] * f, f).imag
    G = (C * (d.w[:, None] * f).imag.sum(0)) @ C.T
    gH = -2.0 / math.pi * C @ (M * fH) @ C.T
    gS = -2.0 / math.pi * (Q[:, None] * G - C @ (M * fS) @ C.T)
    return dict(dH=_stored(s, gH), dS=_stored(s, gS))
