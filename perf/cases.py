"""Cases that time the framework through its public entry points.

A case is a dict of plain values.  ``op`` names the call, ``kind`` and ``n`` the
molecule family and its size, and the rest its options:

* ``jk``    -- Coulomb and exchange matrices of one density on a fitted tensor
               that the program keeps: the inner step of every SCF.
* ``fock``  -- the fitted tensor of a new geometry, then its first J and K: what
               every step of a trajectory or of a scan pays before it iterates.
* ``scf``   -- a whole restricted SCF in FP64 (how many iterations the mixed schedule takes turns on
               the last bits of its FP32 stage, so its parts are timed instead: ``jk`` in FP32).
* ``grad``  -- the nuclear gradient at given orbitals.
* ``mp2``   -- the MP2 correlation energy on a fitted tensor.
* ``train`` -- one optimiser step of the network behind the learned start.

The molecules are the families of the repository's own workloads, with their
even-tempered bases, at any size: hydrogen chains, water clusters on a jittered
lattice, zigzag alkanes, random carbon clusters (the ones with f orbitals and
g auxiliary functions).  Every coordinate is jittered from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1707_03771_amd as dfx

# the exchange matrix of a reduced-precision build has the digits of its type: it is handed on in that type
PRECISIONS = {"fp64": (dfx.FP64, torch.float64), "fp32": (dfx.FP32, torch.float32),
              "bf16": (dfx.BF16, torch.bfloat16)}


def listed():
    return [
        # the smallest Fock build there is: four hydrogens, all of it launches and latency
        {"name": "jk_chain4", "op": "jk", "kind": "chain", "n": 4, "precision": "fp64", "given": "orbitals"},
        # a small cluster, as in a training set or a fragment calculation (192 functions)
        {"name": "jk_water8", "op": "jk", "kind": "water", "n": 8, "precision": "fp64", "given": "orbitals"},
        # a long thin molecule, where distant pairs are screened (730 functions)
        {"name": "jk_alkane30", "op": "jk", "kind": "alkane", "n": 30, "precision": "fp64", "given": "orbitals"},
        # J and K of a density matrix instead of orbitals, as a density-based start needs once
        {"name": "jk_density_alkane10", "op": "jk", "kind": "alkane", "n": 10, "precision": "fp64",
         "given": "density"},
        # the reduced-precision build of the mixed schedule on a big basis with f functions (1200 functions)
        {"name": "jk_carbon40_fp32", "op": "jk", "kind": "carbon", "n": 40, "precision": "fp32",
         "given": "orbitals"},
        # a new geometry of a long molecule (730 functions): integrals, metric, fit, first build
        {"name": "fock_alkane30", "op": "fock", "kind": "alkane", "n": 30, "precision": "fp64"},
        # the same, the largest, with every integral class up to (ff|g) (1200 functions)
        {"name": "fock_carbon40", "op": "fock", "kind": "carbon", "n": 40, "precision": "fp64"},
        # whole SCF runs from the core guess: a small one, where the loop's own overheads count, ...
        {"name": "scf_water8", "op": "scf", "kind": "water", "n": 8},
        # ... and a larger one (394 functions)
        {"name": "scf_alkane16", "op": "scf", "kind": "alkane", "n": 16},
        # forces for one step of a geometry optimisation
        {"name": "grad_water8", "op": "grad", "kind": "water", "n": 8},
        # correlation energy of a middling cluster, cores frozen (648 functions)
        {"name": "mp2_water27", "op": "mp2", "kind": "water", "n": 27, "frozen": True},
        # a minibatch of the water O-H pair network
        {"name": "train_pair", "op": "train", "d_in": 454, "hidden": 256, "depth": 3, "d_out": 70, "batch": 128},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    plain = [{k: v for k, v in c.items() if k != "name"} for c in listed()]
    while True:
        case = _draw(rng)
        if case not in plain:
            return case


def _draw(rng):
    op = rng.choice(["jk", "jk", "jk", "fock", "fock", "scf", "grad", "mp2", "train"])
    if op == "jk":
        kind = rng.choice(["chain", "water", "alkane", "carbon"])
        given = rng.choice(["orbitals", "orbitals", "orbitals", "density"])
        most = ({"chain": 60, "water": 16, "alkane": 30, "carbon": 38} if given == "orbitals" else
                {"chain": 60, "water": 16, "alkane": 14, "carbon": 12})
        n = _log_int(rng, 2, most[kind])
        n += n % 2 if kind == "chain" else 0
        return {"op": op, "kind": kind, "n": n, "precision": rng.choice(["fp64", "fp64", "fp32", "bf16"]),
                "given": given}
    if op == "fock":
        kind = rng.choice(["chain", "water", "alkane", "carbon"])
        n = _log_int(rng, 2, {"chain": 60, "water": 16, "alkane": 30, "carbon": 38}[kind])
        return {"op": op, "kind": kind, "n": n + (n % 2 if kind == "chain" else 0),
                "precision": rng.choice(["fp64", "fp64", "fp32"])}
    if op == "scf":
        kind = rng.choice(["water", "alkane"])
        return {"op": op, "kind": kind, "n": _log_int(rng, 2, {"water": 12, "alkane": 15}[kind])}
    if op == "grad":
        kind = rng.choice(["chain", "water", "alkane", "carbon"])
        n = _log_int(rng, 2, {"chain": 20, "water": 8, "alkane": 5, "carbon": 3}[kind])
        return {"op": op, "kind": kind, "n": n + (n % 2 if kind == "chain" else 0)}
    if op == "mp2":
        kind = rng.choice(["chain", "water", "alkane"])
        n = _log_int(rng, 4, {"chain": 60, "water": 26, "alkane": 20}[kind])
        return {"op": op, "kind": kind, "n": n + (n % 2 if kind == "chain" else 0),
                "frozen": kind != "chain" and rng.random() < 0.5}
    return {"op": op, "d_in": rng.randint(50, 460), "hidden": rng.choice([64, 128, 256]), "depth": rng.randint(1, 4),
            "d_out": rng.randint(1, 196), "batch": _log_int(rng, 16, 512)}


# ---- molecules ----------------------------------------------------------------

CHARGE = {"H": 1, "C": 6, "O": 8}
# even-tempered shells: {family: {element: number of shells per l}}
ORBITAL = {"water": {"O": [3, 2, 1], "H": [2, 1]}, "alkane": {"C": [3, 2, 1], "H": [2, 1]},
           "carbon": {"C": [4, 3, 2, 1]}}
AUXILIARY = {"water": {"O": [8, 6, 4, 2], "H": [4, 3, 2]}, "alkane": {"C": [7, 5, 4, 2], "H": [4, 3, 2]},
             "carbon": {"C": [8, 6, 5, 3, 2]}}
CHAIN_ORBITAL = [(0, 0.1 * 3 ** k) for k in range(3)] + [(1, 0.8)]
CHAIN_AUXILIARY = ([(0, 0.05 * 2.5 ** k) for k in range(6)] + [(1, 0.2 * 2.5 ** k) for k in range(3)]
                   + [(2, 0.5 * 2.5 ** k) for k in range(2)])


def _unit(v):
    return v / np.linalg.norm(v)


def _chain(n, rng):
    return ["H"] * n, np.array([[0.0, 0.0, 1.8 * k] for k in range(n)]) + rng.normal(0.0, 0.02, (n, 3))


def _water(n, rng):
    side = math.ceil(n ** (1 / 3) - 1e-9)
    half = math.radians(104.5) / 2
    mono = 1.81 * np.array([[0, 0, 0], [math.sin(half), 0, math.cos(half)], [-math.sin(half), 0, math.cos(half)]])
    xyz = []
    for k in range(n):
        o = 5.5 * np.array([k // side // side, k // side % side, k % side], float) + rng.normal(0.0, 0.1, 3)
        q, r = np.linalg.qr(rng.normal(size=(3, 3)))
        q = q * np.sign(np.diag(r))
        q[:, 0] *= np.linalg.det(q)
        xyz += [o + q @ m for m in mono]
    return ["O", "H", "H"] * n, np.array(xyz)


def _alkane(n, rng):
    th, cc, ch = math.radians(109.4712206), 2.91, 2.06
    C = [np.array([k * cc * math.sin(th / 2), (k % 2) * cc * math.cos(th / 2), 0.0]) for k in range(n)]
    H = []
    for k in range(1, n - 1):
        u = -_unit(_unit(C[k - 1] - C[k]) + _unit(C[k + 1] - C[k]))
        w = _unit(np.cross(C[k - 1] - C[k], C[k + 1] - C[k]))
        H += [C[k] + ch * (math.cos(th / 2) * u + s * math.sin(th / 2) * w) for s in (1.0, -1.0)]
    for k, m in ((0, 1), (n - 1, n - 2)):
        e = _unit(C[m] - C[k])
        p = _unit(np.cross(np.cross(e, [0.0, 0.0, 1.0]), e))
        q = np.cross(e, p)
        H += [C[k] + ch * (-e / 3 + math.sqrt(8) / 3 * (math.cos(a) * p + math.sin(a) * q))
              for a in (0.0, 2 * math.pi / 3, 4 * math.pi / 3)]
    xyz = np.array(C + H)
    return ["C"] * n + ["H"] * len(H), xyz + rng.uniform(-0.05, 0.05, xyz.shape)


def _carbon(n, rng):
    box, pts = 20.0 * (n / 40) ** (1 / 3), []
    while len(pts) < n:
        c = rng.uniform(0.0, max(box, 6.0), 3)
        if all(np.linalg.norm(c - p) >= 2.5 for p in pts):
            pts.append(c)
    return ["C"] * n, np.array(pts)


def molecule(kind, n, seed):
    """(xyz, Z, orbital shells, auxiliary shells, occupied orbitals)."""
    rng = np.random.default_rng([seed, n])
    elems, xyz = {"chain": _chain, "water": _water, "alkane": _alkane, "carbon": _carbon}[kind](n, rng)

    def shells(shape, base, ratio, chain):
        out = []
        for e, r in zip(elems, xyz):
            each = chain if kind == "chain" else [(l, base * ratio ** k) for l, m in enumerate(shape[kind][e])
                                                  for k in range(m)]
            out += [{"center": np.array(r), "l": l, "exps": [a], "coefs": [1.0]} for l, a in each]
        return out

    Z = np.array([CHARGE[e] for e in elems], np.int32)
    return (xyz, Z, shells(ORBITAL, 0.15, 3.0, CHAIN_ORBITAL), shells(AUXILIARY, 0.1, 2.5, CHAIN_AUXILIARY),
            int(Z.sum()) // 2)


def _nfun(shells):
    return sum(2 * s["l"] + 1 for s in shells)


def _orbitals(nbf, nocc, seed):
    """Orthonormal columns (QR of a normal matrix, positive diagonal): occupied orbitals of a kernel-only run."""
    q, r = np.linalg.qr(np.random.default_rng([seed, nbf, nocc]).normal(size=(nbf, nocc)))
    return q * np.sign(np.diag(r))


def _core_orbitals(sh, xyz, Z):
    """Eigenvectors and levels of the core Hamiltonian in the Loewdin basis (all orbitals)."""
    S, T, V = (m.cpu() for m in dfx.int1e(sh, xyz, Z))
    s, U = torch.linalg.eigh(S)
    X = U @ torch.diag(s.clamp_min(1e-9) ** -0.5) @ U.T
    e, W = torch.linalg.eigh(X @ (T + V) @ X)
    return (X @ W).contiguous(), e


# ---- prepare, run -------------------------------------------------------------

def prepare(case, seed):
    op = case["op"]
    if op == "train":
        g = torch.Generator().manual_seed(seed)
        w = _widths(case)
        theta = torch.cat([torch.cat([torch.randn(a * b, generator=g) * (1.0 / a) ** 0.5, torch.zeros(b)])
                           for a, b in zip(w, w[1:])]).cuda()
        return {"case": case, "w": w, "theta": theta, "m": torch.zeros_like(theta), "v": torch.zeros_like(theta),
                "X": torch.randn(case["batch"], w[0], generator=g).cuda(),
                "T": torch.randn(case["batch"], w[-1], generator=g).cuda()}
    xyz, Z, sh, ax, nocc = molecule(case["kind"], case["n"], seed)
    st = {"case": case, "xyz": xyz, "Z": Z, "sh": sh, "ax": ax, "nocc": nocc}
    if op in ("jk", "fock"):
        C = _orbitals(_nfun(sh), nocc, seed)
        st["C"] = torch.from_numpy(C @ C.T if case.get("given") == "density" else C).cuda()
    if op in ("jk", "mp2"):
        st["B"] = dfx.eri3(sh, ax)
    if op in ("grad", "mp2"):
        C, e = _core_orbitals(sh, xyz, Z)
        if op == "mp2":
            st["C"], st["eps"] = C.cuda(), e.numpy()
            st["frozen"] = int((Z > 1).sum()) if case["frozen"] else 0
        else:
            st["C"], st["eps"] = C[:, :nocc].numpy().copy(), e[:nocc].numpy().copy()
    return st


def run(st):
    case = st["case"]
    op = case["op"]
    if op in ("jk", "fock"):
        precision, dtype = PRECISIONS[case["precision"]]
        B = st["B"] if op == "jk" else dfx.eri3(st["sh"], st["ax"])
        kind = dfx.DENSITY if case.get("given") == "density" else dfx.COCC
        J, K = dfx.jk(B, st["C"], kind=kind, precision=precision)
        return J, K.to(dtype)
    if op == "scf":
        E, _, eps, _ = dfx.scf(st["xyz"], st["Z"], st["sh"], st["ax"], conv_dE=1e-10, conv_err=1e-8)
        return {"E": E, "eps": eps}  # the orbitals' signs are anyone's choice: energy and levels
    if op == "grad":
        return dfx.rhf_grad(st["xyz"], st["Z"], st["sh"], st["ax"], st["C"], st["eps"])[0]
    if op == "mp2":
        return dfx.mp2(st["B"], st["C"], st["eps"], st["nocc"], nfrozen=st["frozen"])
    # one Adam step from the same parameters every time
    theta, m, v = (st[k].clone() for k in ("theta", "m", "v"))
    loss, g = dfx.mlp_loss_grad(st["w"], theta, st["X"], st["T"])
    dfx.mlp_adam(theta, g, m, v, 1)
    return {"loss": loss, "grad": g, "theta": theta, "m": m, "v": v}


def _widths(case):
    return [case["d_in"]] + [case["hidden"]] * case["depth"] + [case["d_out"]]


# ---- work ---------------------------------------------------------------------

def work(case):
    """Bytes and operations of one pass that no method of these equations avoids."""
    op = case["op"]
    if op == "train":
        w = _widths(case)
        par, act = sum(a * b + b for a, b in zip(w, w[1:])), case["batch"] * (w[0] + w[-1])
        mac = sum(a * b for a, b in zip(w, w[1:])) * case["batch"]
        return {"bytes": 4.0 * (8 * par + act), "flops": 2.0 * (3 * mac - case["batch"] * w[0] * w[1])}
    _, _, sh, ax, o = molecule(case["kind"], case["n"], 0)
    n, q = _nfun(sh), _nfun(ax)
    cols = n * (n + 1) / 2
    tensor = 8.0 * q * cols
    jk = 4.0 * q * cols + 2.0 * n * n * o * q + n * (n + 1.0) * o * q
    fit = q * float(q) * cols + q ** 3 / 3.0
    if op == "jk":
        given = 8.0 * n * (n if case["given"] == "density" else o)
        return {"bytes": tensor + given + 16.0 * n * n, "flops": jk}
    if op == "fock":
        return {"bytes": tensor + 8.0 * n * o + 16.0 * n * n, "flops": fit + jk}
    if op == "scf":  # the fit, and ten iterations
        return {"bytes": 11 * tensor, "flops": fit + 10 * (jk + 12.0 * n ** 3)}
    if op == "grad":
        return {"bytes": tensor + 8.0 * n * o, "flops": 2 * fit + (4.0 * n * n * o + 2.0 * n * n * o) * q
                + float(q) * q * (o * o + 2 * q)}
    f = int(round(case["n"])) if case["frozen"] else 0
    o, v = o - f, n - o
    return {"bytes": tensor + 8.0 * n * n, "flops": 2.0 * q * (n * n * o + v * n * o) + float(v) * v * q * o * (o + 1)}


# ---- exact values -------------------------------------------------------------

def exact(case, seed):
    """The outputs in 64 bits by plain torch and numpy: the network's step, and J and K of hydrogen chains
    (McMurchie-Davidson integrals); None where that takes too long or the integrals would."""
    if case["op"] == "train":
        return _exact_train(case, seed)
    if case["op"] not in ("jk", "fock") or case["kind"] != "chain" or case["n"] > 12:
        return None
    _, _, sh, ax, nocc = molecule("chain", case["n"], seed)
    C = _orbitals(_nfun(sh), nocc, seed)
    D = C @ C.T
    raw, one = _integrals(sh, sh, ax), [{"center": np.zeros(3), "l": 0, "exps": [0.0], "coefs": [1.0]}]
    metric = _integrals(ax, one, ax)[:, 0, :]
    L = np.linalg.cholesky((metric + metric.T) / 2)
    B = torch.linalg.solve_triangular(torch.from_numpy(L), torch.from_numpy(raw.reshape(-1, raw.shape[2]).T.copy()),
                                      upper=False).numpy().reshape(raw.shape[2], *raw.shape[:2])
    J = np.einsum("qmn,q->mn", B, np.einsum("qmn,mn->q", B, D))
    X = np.einsum("qmn,ni->qmi", B, C)
    return J, np.einsum("qmi,qni->mn", X, X)


def _exact_train(case, seed):
    st = prepare(case, seed)
    w, X, T = st["w"], st["X"].double().cpu(), st["T"].double().cpu()
    theta = st["theta"].double().cpu().requires_grad_()
    a, at = X, 0
    for i, (p, q) in enumerate(zip(w, w[1:])):
        a = a @ theta[at:at + p * q].reshape(q, p).T + theta[at + p * q:at + p * q + q]
        a = a if i == len(w) - 2 else a * torch.sigmoid(a)
        at += p * q + q
    loss = ((a - T) ** 2).mean()
    g, = torch.autograd.grad(loss, theta)
    m, v = 0.1 * g, 0.001 * g * g
    new = theta.detach() - 1e-3 * (m / 0.1) / ((v / 0.001).sqrt() + 1e-8)
    return {"loss": float(loss), "grad": g, "theta": new, "m": m, "v": v}


# real solid harmonics as Cartesian monomials {(i, j, k): c}, m = -l .. l, any scale
SOLID = {0: [{(0, 0, 0): 1.0}],
         1: [{(0, 1, 0): 1.0}, {(0, 0, 1): 1.0}, {(1, 0, 0): 1.0}],
         2: [{(1, 1, 0): 1.0}, {(0, 1, 1): 1.0}, {(0, 0, 2): 2.0, (2, 0, 0): -1.0, (0, 2, 0): -1.0},
             {(1, 0, 1): 1.0}, {(2, 0, 0): 1.0, (0, 2, 0): -1.0}]}


def _odd(n):
    return math.prod(range(1, n, 2)) if n > 0 else 1


def _norm(poly, a):
    """1 / sqrt(self overlap) of poly(x, y, z) exp(-a r^2)."""
    s = 0.0
    for p, c in poly.items():
        for q, d in poly.items():
            t = [x + y for x, y in zip(p, q)]
            if all(x % 2 == 0 for x in t):
                s += c * d * math.prod(_odd(x) / (4 * a) ** (x // 2) for x in t)
    return (s * (math.pi / (2 * a)) ** 1.5) ** -0.5


def _boys(nmax, T):
    """F_0 .. F_nmax of an array T: a series below 25, upward recursion from erf above."""
    F = np.zeros((nmax + 1,) + T.shape)
    small = T < 25.0
    t = np.where(small, T, 0.0)
    term = np.full(T.shape, 1.0 / (2 * nmax + 1))
    for k in range(1, 120):
        F[nmax] += term
        term = term * 2 * t / (2 * nmax + 2 * k + 1)
    F[nmax] *= np.exp(-t)
    for n in range(nmax - 1, -1, -1):
        F[n] = (2 * t * F[n + 1] + np.exp(-t)) / (2 * n + 1)
    t = np.where(small, 25.0, T)
    up = 0.5 * np.sqrt(np.pi / t) * torch.erf(torch.from_numpy(np.sqrt(t))).numpy()
    for n in range(nmax + 1):
        F[n] = np.where(small, F[n], up)
        up = ((2 * n + 1) * up - np.exp(-t)) / (2 * t)
    return F


def _hermite(i, j, p, PA, PB):
    """E_t of x_A^i x_B^j in Hermite Gaussians (without the pair's exponential), t = 0 .. i + j."""
    E = [np.ones_like(p)]
    for d in [PA] * i + [PB] * j:
        E = [(E[t - 1] / (2 * p) if t > 0 else 0.0) + (d * E[t] if t < len(E) else 0.0)
             + ((t + 1) * E[t + 1] if t + 1 < len(E) else 0.0) for t in range(len(E) + 1)]
    return E


def _integrals(A, B, K):
    """(a b|k) over all functions; an exponent of zero in B stands for the function 1."""
    first = [np.concatenate([[0], np.cumsum([2 * s["l"] + 1 for s in S])]) for S in (A, B, K)]
    out = np.zeros([f[-1] for f in first])
    for la in range(3):
        for lb in range(3):
            for lk in range(3):
                ia, ib, ik = ([x for x, s in enumerate(S) if s["l"] == l] for S, l in ((A, la), (B, lb), (K, lk)))
                if ia and ib and ik:
                    _block(A, B, K, ia, ib, ik, la, lb, lk, first, out)
    return out


def _block(A, B, K, ia, ib, ik, la, lb, lk, first, out):
    def take(S, idx, shape):
        return (np.array([S[x]["exps"][0] for x in idx]).reshape(shape),
                np.array([S[x]["center"] for x in idx]).T.reshape((3,) + shape))

    (a, ra), (b, rb), (k, rk) = take(A, ia, (-1, 1, 1)), take(B, ib, (1, -1, 1)), take(K, ik, (1, 1, -1))
    p = a + b
    PA, PB = -b / p * (ra - rb), a / p * (ra - rb)
    R = PA + (ra - rk)
    rho = p * k / (p + k)
    nmax = la + lb + lk
    F = _boys(nmax, rho * (R ** 2).sum(0))
    pref = 2 * math.pi ** 2.5 / (p * k * np.sqrt(p + k)) * np.exp(-a * b / p * ((ra - rb) ** 2).sum(0))
    memo = {(n, 0, 0, 0): (-2 * rho) ** n * F[n] * pref for n in range(nmax + 1)}

    def r(n, t):
        key = (n,) + t
        if key not in memo:
            x = next(x for x in range(3) if t[x])
            less = tuple(t[y] - (y == x) for y in range(3))
            v = R[x] * r(n + 1, less)
            if less[x]:
                v = v + less[x] * r(n + 1, tuple(less[y] - (y == x) for y in range(3)))
            memo[key] = v
        return memo[key]

    for ma, pa in enumerate(SOLID[la]):
        for mb, pb in enumerate(SOLID[lb]):
            for mk, pk in enumerate(SOLID[lk]):
                v = 0.0
                for ea, ca in pa.items():
                    for eb, cb in pb.items():
                        E = [_hermite(ea[x], eb[x], p, PA[x], PB[x]) for x in range(3)]
                        for ek, ck in pk.items():
                            H = [_hermite(ek[x], 0, k, 0.0 * k, 0.0 * k) for x in range(3)]
                            for t in np.ndindex(*[len(e) for e in E]):
                                for u in np.ndindex(*[len(h) for h in H]):
                                    c = H[0][u[0]] * H[1][u[1]] * H[2][u[2]] * (-1.0) ** sum(u)
                                    if np.any(c):
                                        v = v + (ca * cb * ck * c * E[0][t[0]] * E[1][t[1]] * E[2][t[2]]
                                                 * r(0, tuple(x + y for x, y in zip(t, u))))
                na = np.array([_norm(pa, x) for x in a.ravel()]).reshape(-1, 1, 1)
                nb = np.array([_norm(pb, x) if x > 0 else 1.0 for x in b.ravel()]).reshape(1, -1, 1)
                nk = np.array([_norm(pk, x) for x in k.ravel()]).reshape(1, 1, -1)
                rows = [first[0][x] + ma for x in ia], [first[1][x] + mb for x in ib], [first[2][x] + mk for x in ik]
                out[np.ix_(*rows)] = v * na * nb * nk
