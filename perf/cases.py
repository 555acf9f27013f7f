"""Performance cases: what a program does with this package, per call.

Every case is one pass through a public entry point on a seeded synthetic
pencil of `paper_1405_0194_amd.lattice` (1D chains, honeycomb sheets, simple
cubic bulk), at the sizes and pole counts of the package's own workloads
(N 256 to 26,624 orbitals, 40 to 80 poles, 8 to 32 real shifts).  Operations:

  replay    a graph plan replayed with a new pole table (an SCF or chemical
            potential iteration on a pattern that is kept)
  eager     the density matrix in one call on kept buffers, pole table included
  api       the sparse-matrix call of the README on a kept solver
  batch     several uneven systems through the batch runner
  inertia   negative-pivot counts at real shifts (bracketing, cumulative DOS)
  ldos      the local density of states at a few energies
  kpoint    a complex Hermitian pencil: L D U plan replayed

`work` counts floating-point operations on the exact structure of L under
the package's ordering, and the bytes of the inputs and outputs.
"""
import math

import numpy as np
import torch

from paper_1405_0194_amd import api, batch, binding, dos, lattice, tune

BETA = lattice.BETA_300K
DE = 1.0          # the generator keeps the spectrum in [-1, 1]; mu = 0
ETA = 0.02        # broadening of the LDOS cases
EXACT_MAX_N = 2300


def listed():
    return [
        # smallest call: one iteration on a kept 1D pattern, bound by latency
        dict(name="chain_replay", op="replay", kind="chain", nx=64, ny=0, nz=0, orb=4, poles=40, sets=2),
        # a longer 1D system called eagerly: many tiny supernodes
        dict(name="chain_eager", op="eager", kind="chain", nx=500, ny=0, nz=0, orb=4, poles=60, sets=2),
        # a small sheet, replayed as in an SCF cycle
        dict(name="sheet416_replay", op="replay", kind="honeycomb", nx=4, ny=4, nz=0, orb=13, poles=40, sets=2),
        # Newton's iteration for mu: all four weight sets, ragged tiles (N = 2106)
        dict(name="sheet2k_newton", op="replay", kind="honeycomb", nx=9, ny=9, nz=0, orb=13, poles=60, sets=4),
        # a small bulk cell in one eager call
        dict(name="bulk2k_eager", op="eager", kind="cubic", nx=5, ny=5, nz=6, orb=13, poles=40, sets=2),
        # bracketing the chemical potential of a mid-size sheet: real factorizations
        dict(name="sheet8k_inertia", op="inertia", kind="honeycomb", nx=17, ny=18, nz=0, orb=13, poles=16, sets=0),
        # one k-point of a periodic sheet
        dict(name="kpoint2k", op="kpoint", kind="honeycomb", nx=9, ny=8, nz=0, orb=13, poles=40, sets=2),
        # the sparse-matrix call, host conversion included
        dict(name="api_sheet1k", op="api", kind="honeycomb", nx=7, ny=6, nz=0, orb=13, poles=40, sets=2),
        # the uneven batch: systems of all three kinds side by side
        dict(name="batch_mix", op="batch", kind="mix", nx=0, ny=0, nz=0, orb=0, poles=0, sets=2),
        # a mid-size sheet, eager
        dict(name="sheet8k_eager", op="eager", kind="honeycomb", nx=17, ny=18, nz=0, orb=13, poles=60, sets=2),
        # a mid-size bulk cell, eager: wide fronts
        dict(name="bulk7k_eager", op="eager", kind="cubic", nx=8, ny=8, nz=9, orb=13, poles=40, sets=2),
        # the largest sheet (N = 26,624)
        dict(name="sheet26k_eager", op="eager", kind="honeycomb", nx=32, ny=32, nz=0, orb=13, poles=40, sets=2),
    ]


def draw(rng):
    op = rng.choice(["replay", "replay", "eager", "eager", "inertia", "ldos", "kpoint", "api"])
    kind = rng.choice(["chain", "honeycomb", "cubic"])
    hi = {"kpoint": 3000.0, "api": 3000.0, "ldos": 4000.0}.get(op, 8000.0 if kind != "cubic" else 6500.0)
    n = math.exp(rng.uniform(math.log(250.0), math.log(hi)))
    nx = ny = nz = 0
    if kind == "chain":
        orb = 4
        nx = max(8, round(n / orb))
    elif kind == "honeycomb":
        orb = rng.choice([4, 9, 13, 13])
        cells = max(4.0, n / (2 * orb))
        nx = max(2, round(math.sqrt(cells) * rng.uniform(0.7, 1.4)))
        ny = max(2, round(cells / nx))
    else:
        orb = rng.choice([4, 9, 13, 13])
        nx = max(2, round((n / orb) ** (1.0 / 3.0)))
        ny = max(2, nx + rng.choice([-1, 0, 1]))
        nz = max(2, round(n / orb / nx / ny))
    if op == "inertia":
        poles, sets = rng.randint(8, 32), 0
    elif op == "ldos":
        poles, sets = rng.randint(3, 16), 0
    else:
        poles, sets = 2 * rng.randint(20, 40 if n < 6000 else 30), rng.choice([1, 2, 2, 4])
    return dict(op=op, kind=kind, nx=nx, ny=ny, nz=nz, orb=orb, poles=poles, sets=sets)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _system(case, seed):
    kind = case["kind"]
    dims = {"chain": case["nx"], "honeycomb": (case["nx"], case["ny"]),
            "cubic": (case["nx"], case["ny"], case["nz"])}[kind]
    make = lattice.make_hermitian_system if case["op"] == "kpoint" else lattice.make_system
    return make(kind, dims, case["orb"], 3.0 if kind == "honeycomb" else 2.0, seed)


_MIX = [("chain", 150, 44), ("honeycomb", (5, 6), 60), ("cubic", (4, 4, 4), 52),
        ("chain", 480, 74), ("honeycomb", (8, 9), 70), ("cubic", (5, 5, 5), 42)]


def _mix(seed):
    """(system, poles) of the uneven batch."""
    return [(lattice.make_system(kind, dims, 4 if kind == "chain" else 13, 3.0 if kind == "honeycomb" else 2.0,
                                 seed * 10 + i), p) for i, (kind, dims, p) in enumerate(_MIX)]


def _energies(case, seed):
    rng = np.random.default_rng(seed + 77)
    half = 0.1 if case["op"] == "inertia" else 0.3
    return np.sort(rng.uniform(-half, half, case["poles"]))


def _full_coo(s):
    """(rows, cols, hval, sval) of the whole symmetric pencil."""
    r, c = s.rowind.astype(np.int64), s.entry_cols()
    off = r != c
    return (np.concatenate([r, c[off]]), np.concatenate([c, r[off]]),
            np.concatenate([s.hval, s.hval[off]]), np.concatenate([s.sval, s.sval[off]]))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def prepare(case, seed):
    op, P = case["op"], case["poles"]
    if op == "batch":
        jobs = [batch.Job(s, p, nsets=case["sets"], dE=DE) for s, p in _mix(seed)]
        return dict(op=op, runner=batch.BatchRunner(jobs, keep_outputs=True))
    s = _system(case, seed)
    if op == "api":
        r, c, h, v = _full_coo(s)
        idx = torch.from_numpy(np.stack([r, c])).cuda()
        H, S = (torch.sparse_coo_tensor(idx, torch.from_numpy(x).cuda(), (s.n, s.n)).to_sparse_csr() for x in (h, v))
        return dict(op=op, solver=api.Solver(), H=H, S=S, case=case)
    H, S = _dev(s.hval), _dev(s.sval)
    a = tune.tuned_analysis(s, P).bind()
    st = dict(op=op, a=a, H=H, S=S, case=case)
    if op == "replay" or op == "kpoint":
        st["plan"] = binding.Plan(a, H, S, P, nsets=case["sets"])
        st["shifts"], st["weights"] = pole_table(BETA, DE, P, case["sets"])
    elif op == "eager":
        st["L"], st["work"] = a.buffers(P)
    elif op == "inertia":
        st["eps"] = _energies(case, seed)
        st["L"], st["work"] = a.buffers(P, real=True)
    elif op == "ldos":
        st["eps"] = _energies(case, seed)
    return st


def run(st):
    op = st["op"]
    if op in ("replay", "kpoint"):
        out, tr, info = st["plan"].run(st["shifts"], st["weights"])
        return dict(out=out, traces=tr, info=info)
    if op == "eager":
        c = st["case"]
        out, tr, info, sh, wt = binding.density_matrix(st["a"], st["H"], st["S"], BETA, DE, 0.0, c["poles"],
                                                       nsets=c["sets"], L=st["L"], work=st["work"])
        return dict(out=out, traces=tr, info=info, shifts=sh, weights=wt)
    if op == "inertia":
        neg, info = binding.inertia(st["a"], st["H"], st["S"], st["eps"], L=st["L"], work=st["work"])
        return dict(neg=neg, info=info)
    if op == "ldos":
        out, tr, info = dos.ldos(st["a"], st["H"], st["S"], st["eps"], ETA)
        return dict(out=out, traces=tr, info=info)
    if op == "api":
        c = st["case"]
        names = api.SETS[:c["sets"]]
        *mats, tr = st["solver"].density_matrix(st["H"], st["S"], 0.0, BETA, c["poles"], outputs=names, dE=DE)
        return dict(out=[m.values() for m in mats], N=tr["N"], Eband=tr["Eband"], info=tr["info"])
    runner = st["runner"]
    runner.run()
    return dict(out=[j.out for j in runner.jobs], traces=[j.traces for j in runner.jobs],
                info=[j.info for j in runner.jobs])


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _work_of(s, P, sets, op):
    i = tune.tuned_analysis(s, max(2, P)).info
    nnz = i["nnz_lower"]
    if op == "inertia":
        return 16.0 * nnz + 16.0 * P, P * i["flops_factor"] / 4.0
    flops = P * (i["flops_factor"] + i["flops_selinv"])
    outs = P if op == "ldos" else sets
    if op == "kpoint":
        return nnz * (32.0 + 16.0 * outs), 2.0 * flops
    return nnz * (16.0 + 8.0 * outs), flops


def work(case):
    if case["op"] == "batch":
        parts = [_work_of(s, p, case["sets"], "eager") for s, p in _mix(1)]
    else:
        parts = [_work_of(_system(case, 1), case["poles"], case["sets"], case["op"])]
    return dict(bytes=sum(p[0] for p in parts), flops=sum(p[1] for p in parts))


# --------------------------------------------------------------------------
# the same results in plain numpy
# --------------------------------------------------------------------------
def _agm_k(kp):
    a, b = 1.0, kp
    while abs(a - b) > 1e-16 * a:
        a, b = 0.5 * (a + b), math.sqrt(a * b)
    return math.pi / (2.0 * a)


def _jacobi(u, k, kp):
    """sn, cn, dn of a real array (Abramowitz & Stegun 16.4)."""
    a, c, b = [1.0], [k], kp
    while abs(c[-1]) > 1e-17 and len(a) < 60:
        a0 = a[-1]
        a.append(0.5 * (a0 + b))
        c.append(0.5 * (a0 - b))
        b = math.sqrt(a0 * b)
    phi = 2.0 ** (len(a) - 1) * a[-1] * u
    for i in range(len(a) - 1, 0, -1):
        phi = 0.5 * (phi + np.arcsin(np.clip(c[i] * np.sin(phi) / a[i], -1.0, 1.0)))
    sn, cn = np.sin(phi), np.cos(phi)
    return sn, cn, np.sqrt(kp * kp + k * k * cn * cn)


def _occupations(x, beta, mu, sets):
    pos = x.real > 0
    e = np.exp(-np.where(pos, beta * x, -beta * x))
    f = np.where(pos, 2.0 * e / (1.0 + e), 2.0 / (1.0 + e))
    free = -(2.0 / beta) * np.log1p(e) + np.where(pos, 0.0, 2.0 * x)
    return [f, (x + mu) * f, free, 0.5 * beta * f * (2.0 - f)][:sets]


def pole_table(beta, dE, P, sets):
    """Shifts (P,) and weights (sets, P) at mu = 0: contour quadrature in
    xi = z^2 + (pi/beta)^2 on the elliptic map, P / 2 nodes, two poles each."""
    Q, m = P // 2, (math.pi / beta) ** 2
    M = dE * dE + m
    r = math.sqrt(M / m)
    k, kp = (r - 1.0) / (r + 1.0), 2.0 * math.sqrt(r) / (r + 1.0)
    K, Kc = _agm_k(kp), _agm_k(k)
    s, c, d = _jacobi(-K + (np.arange(1, Q + 1) - 0.5) * 2.0 * K / Q, k, kp)
    s1, c1, d1 = _jacobi(np.array([0.5 * Kc]), kp, k)
    den = c1 * c1 + k * k * s * s * s1 * s1
    sn = (s * d1 + 1j * c * d * s1 * c1) / den
    cn = (c * c1 - 1j * s * d * s1 * d1) / den
    dn = (d * c1 * d1 - 1j * k * k * s * c * s1) / den
    q = math.sqrt(m * M)
    xi = q * (1.0 / k + sn) / (1.0 / k - sn)
    dxi = q * (2.0 / k) * cn * dn / (1.0 / k - sn) ** 2
    z = np.sqrt(xi - m)
    coef = -(2.0 * K / (math.pi * Q)) * dxi / (2.0 * z)
    plus, minus = _occupations(z, beta, 0.0, sets), _occupations(-z, beta, 0.0, sets)
    wt = [np.concatenate([-coef * p, -np.conj(coef * n)]) for p, n in zip(plus, minus)]
    return np.concatenate([z, -np.conj(z)]), np.array(wt)


def _eigen(s):
    """Generalized eigenvalues and S-orthonormal eigenvectors, and dense H, S."""
    H, S = s.dense()
    Li = np.linalg.inv(np.linalg.cholesky(S))
    e, U = np.linalg.eigh(Li @ H @ Li.conj().T)
    return e, Li.conj().T @ U, H, S


def _sums(s, eig, rows):
    """Entries on the lower pattern, and the two traces, of C diag(f) C^H."""
    e, C, H, S = eig
    r, c = s.rowind, s.entry_cols()
    out, tr = [], []
    for f in rows:
        G = (C * f) @ C.conj().T
        out.append(G[r, c])
        tr.append([np.sum(G * S.conj()).real, np.sum(G * H.conj()).real])
    return np.array(out), np.array(tr)


def _gamma(s, shifts, weights):
    eig = _eigen(s)
    inv = 1.0 / (eig[0][:, None] - shifts[None, :])
    return _sums(s, eig, [(inv @ w).imag for w in weights])


def exact(case, seed):
    op, P, sets = case["op"], case["poles"], case["sets"]
    if op == "inertia":
        return None
    if op == "batch":
        systems = _mix(seed)
        if max(s.n for s, _ in systems) > EXACT_MAX_N:
            return None
        got = [_gamma(s, *pole_table(BETA, DE, p, sets)) for s, p in systems]
        return dict(out=[g[0] for g in got], traces=[g[1] for g in got], info=[None] * len(got))
    s = _system(case, seed)
    if s.n > EXACT_MAX_N:
        return None
    if op == "ldos":
        eig = _eigen(s)
        rows = [(2.0 / np.pi) * (1.0 / (eig[0] - (x + 1j * ETA))).imag for x in _energies(case, seed)]
        out, tr = _sums(s, eig, rows)
        return dict(out=out, traces=tr, info=None)
    sh, wt = pole_table(BETA, DE, P, sets)
    out, tr = _gamma(s, sh, wt)
    if op == "api":
        return dict(out=list(out), N=float(tr[0, 0]), Eband=float(tr[0, 1]), info=None)
    got = dict(out=out, traces=tr, info=None)
    if op == "eager":
        got.update(shifts=sh, weights=wt)
    return got
