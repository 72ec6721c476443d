"""Timed workloads of the library, through its Python entry points.

Every case is one molecule (or one batch of molecules) and one thing that an
electronic-structure program asks of the library for it: the stored integral
matrix B, the Coulomb matrix J of a density (full, contracted, screened,
compressed, over adaptive boxes, in an orbital basis) or the exchange matrix.
The sizes are those of the package's own workloads (inputs.py: 8, 64, 400 and
1000 functions, batches of 20 to 120) and sizes between them that are no
multiple of any tile.
"""
import math

import numpy as np
import torch

from paper_2210_13069_amd import inputs as I
from paper_2210_13069_amd import tai

F64 = torch.float64
ESIZE = {"fp64": 8, "fp32": 4, "f16x3": 4, "bf16x3": 4, "bf16x6": 4}
# components per atom and the range of the log-uniform exponents, as inputs.py has them
SHELLS = {"s": (1, 0.2, 20.0), "sp": (4, 0.1, 50.0), "spd": (10, 0.1, 100.0)}
BOX_TAU = 1e-20    # support threshold of the adaptive boxes
SCREEN_TAU = 1e-12


def listed():
    return [
        # the smallest molecule, everything for its B in FP64: launches and latency count
        dict(name="B tiny fp64", kind="B", prec="fp64", atoms=4, shells="ss", n=24, nq=16, omega=0.5, degree_tol=0.0),
        # a small molecule's reference B, formed once per geometry
        dict(name="B sp64 fp64", kind="B", prec="fp64", atoms=16, shells="sp", n=32, nq=24, omega=0.5, degree_tol=0.0),
        # a medium molecule in single precision with a degree per quadrature node; no size fits a tile
        dict(name="B spd130 fp32 degrees", kind="B", prec="fp32", atoms=13, shells="spd", n=37, nq=29, omega=0.7,
             degree_tol=1e-8),
        # the package's headline: 400 functions, 6.4e9 entries of B on the 16-bit matrix cores
        dict(name="B spd400 f16x3", kind="B", prec="f16x3", atoms=40, shells="spd", n=40, nq=32, omega=0.3,
             degree_tol=0.0),
        # many small molecules in one call (a screening campaign, a data set)
        dict(name="B batch64 f16x3", kind="batch", prec="f16x3", mols=64, lo=5, hi=30, shells="sp", n=32, nq=24,
             sizes=1),
        # one SCF iteration of a small molecule in a contracted basis: the moments are in hand, D is new
        dict(name="J contracted sp96 fp64", kind="J", prec="fp64", atoms=24, shells="sp", prims=2, n=32, nq=24,
             omega=0.5),
        # one SCF iteration of a large molecule
        dict(name="J spd1000 fp64", kind="J", prec="fp64", atoms=100, shells="spd", prims=1, n=48, nq=32, omega=0.4),
        # a new geometry of a large molecule with screening: kept pairs, their moments, J
        dict(name="J screened spd500 fp32", kind="screened", prec="fp32", atoms=50, shells="spd", n=40, nq=32,
             omega=0.3),
        # a new geometry with compressed moments that serve the iterations after it
        dict(name="J compressed spd610 fp64", kind="compressed", prec="fp64", atoms=61, shells="spd", n=48, nq=32,
             omega=0.4, rank_tol=1e-5, builds=3),
        # a new geometry over adaptive boxes, in split BF16
        dict(name="J boxes spd250 bf16x6", kind="boxes", prec="bf16x6", atoms=25, shells="spd", n=40, nq=32,
             omega=0.3, parts=4),
        # exchange of a small molecule's occupied orbitals, the moments in hand
        dict(name="exchange sp92 fp64", kind="exchange", prec="fp64", atoms=23, shells="sp", n=32, nq=24, omega=0.5,
             orbitals=8),
        # Coulomb integrals between the orbitals of a medium molecule, the moments in hand
        dict(name="orbital J spd200 fp32", kind="orbital", prec="fp32", atoms=20, shells="spd", n=40, nq=32,
             omega=0.3, orbitals=12),
    ]


# atoms and precisions that each kind of call is used with
RANGES = {
    "B": (2, 40, ["fp64", "fp64", "fp32", "f16x3", "f16x3", "bf16x6", "bf16x3"]),
    "batch": (2, 30, ["f16x3", "f16x3", "fp64", "fp32"]),
    "J": (4, 100, ["fp64", "fp64", "fp32", "bf16x6"]),
    "screened": (10, 100, ["fp64", "fp32", "bf16x6"]),
    "compressed": (10, 100, ["fp64", "fp32"]),
    "boxes": (10, 100, ["fp64", "bf16x6", "bf16x3"]),
    "exchange": (4, 40, ["fp64", "fp32"]),
    "orbital": (8, 100, ["fp64", "fp32"]),
}
RATE = {"fp64": 6e13, "fp32": 1.2e14, "bf16x6": 2.2e14, "f16x3": 4.8e14, "bf16x3": 4.8e14}
MOST_S = 0.045     # what a drawn case may take by its work; the largest listed one takes about 0.05 s


def draw(rng):
    while True:
        kind = rng.choice(sorted(RANGES))
        lo, hi, precs = RANGES[kind]
        atoms = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        c = dict(kind=kind, prec=rng.choice(precs), shells=rng.choice(["ss", "sp", "spd"] if atoms < 12 else
                                                                     ["sp", "spd", "spd"]),
                 n=rng.choice([24, 32, 40, 48, rng.randint(18, 48)]), nq=rng.choice([16, 24, 32, rng.randint(12, 32)]))
        if kind == "batch":
            c.update(mols=int(round(math.exp(rng.uniform(math.log(3), math.log(64))))), lo=max(2, atoms // 3),
                     hi=max(4, atoms), shells=rng.choice(["ss", "sp"]), sizes=rng.randint(2, 1000))
        else:
            c.update(atoms=atoms, omega=rng.choice([0.3, 0.4, 0.5, round(rng.uniform(0.2, 1.0), 2)]))
        if kind == "B":
            c.update(degree_tol=rng.choice([0.0, 0.0, 1e-8]) if c["prec"] in ("fp64", "fp32") else 0.0)
        elif kind == "J":
            c.update(prims=rng.choice([1, 1, 2, 3]))
            c["atoms"] = max(2, c["atoms"] // c["prims"])
        elif kind == "compressed":
            c.update(rank_tol=rng.choice([1e-5, 1e-6]), builds=rng.randint(1, 8))
        elif kind == "boxes":
            c.update(parts=rng.randint(2, 6))
        elif kind in ("exchange", "orbital"):
            c.update(orbitals=rng.randint(2, 16))
        if _seconds(c) <= MOST_S:
            return c


# ---- the molecules ---------------------------------------------------------------
def _side(c):
    """Half-width of the cube the atoms lie in: 3 bohr for 4 atoms, 5 for 16, 12 for 100."""
    return round(max(3.0, 1.2 * math.sqrt(c["atoms"])), 2)


def _functions(c):
    per = 2 if c["shells"] == "ss" else SHELLS[c["shells"]][0]
    return c["atoms"] * per


def _draw_molecule(rng, atoms, side, shells, prims=1):
    """centre, exponent, powers of every primitive, and the function it belongs to."""
    comps = [I.SHELL_COMPONENTS[s] for s in shells]
    lo, hi = SHELLS["s" if shells == "ss" else shells][1:]
    at = rng.uniform(-side, side, size=(atoms, 3))
    ex = np.exp(rng.uniform(math.log(lo), math.log(hi), size=(atoms, len(comps), prims)))
    cen, alp, pw, fn = [], [], [], []
    f = -1
    for i in range(atoms):
        for s, cs in enumerate(comps):
            for l in cs:
                f += 1
                for k in range(prims):
                    cen.append(at[i])
                    alp.append(ex[i, s, k])
                    pw.append(l)
                    fn.append(f)
    return np.array(cen), np.array(alp), np.array(pw, dtype=np.int32), np.array(fn, dtype=np.int32)


def _norms(alpha, powers):
    """Unit-norm constant of each primitive Cartesian Gaussian."""
    df = np.array([1.0, 1.0, 3.0, 15.0, 105.0])
    a = alpha[:, None]
    return np.sqrt(np.sqrt(2 * a / math.pi) * (4 * a) ** powers / df[powers]).prod(axis=1)


def _inputs(c, seed):
    """Host-side inputs of a case from the seed alone."""
    rng = np.random.default_rng(seed)
    g = {}
    if c["kind"] == "batch":
        sz = np.random.default_rng(c["sizes"])
        g["mols"] = []
        for _ in range(c["mols"]):
            atoms, omega = int(sz.integers(c["lo"], c["hi"] + 1)), float(sz.choice([0.3, 0.5, 1.0]))
            cen, alp, pw, _f = _draw_molecule(rng, atoms, 5.0, c["shells"])
            g["mols"].append((cen, alp, pw, I.Params(omega, c["nq"], c["n"], 12.0)))
        return g
    side, prims = _side(c), c.get("prims", 1)
    g["cen"], g["alp"], g["pw"], g["fn"] = _draw_molecule(rng, c["atoms"], side, c["shells"], prims)
    g["params"] = I.Params(c["omega"], c["nq"], c["n"], 2.0 * side + 2.0, degree_tol=c.get("degree_tol", 0.0),
                           rank_tol=c.get("rank_tol", 0.0))
    nb = int(g["fn"][-1]) + 1
    if prims > 1:
        g["coef"] = _norms(g["alp"], g["pw"]) * rng.uniform(0.2, 1.0, len(g["alp"]))
    # densities that decay with the distance of the functions' centres
    cf = g["cen"][::prims]
    decay = np.exp(-np.linalg.norm(cf[:, None] - cf[None], axis=2) / 4.0)
    g["D"] = []
    for _ in range(c.get("builds", 1)):
        d = np.triu(rng.standard_normal((nb, nb)) * decay)
        g["D"].append(d + np.triu(d, 1).T)
    if "orbitals" in c:
        g["Q"] = rng.standard_normal((c["orbitals"], nb)) / math.sqrt(nb)
    return g


def _gpu(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=F64, device="cuda")


def prepare(case, seed):
    g = _inputs(case, seed)
    st = {"case": case, "prec": tai.PREC_BY_NAME[case["prec"]]}
    if case["kind"] == "batch":
        n, prm = case["n"], [m[3] for m in g["mols"]]
        npair = [len(m[1]) * (len(m[1]) + 1) // 2 for m in g["mols"]]
        dt = F64 if case["prec"] == "fp64" else torch.float32
        st["M"] = torch.empty(sum(3 * n * q for q in npair), dtype=F64, device="cuda")
        st["B"] = torch.empty(sum(q * q for q in npair), dtype=dt, device="cuda")
        st["arrays"] = [tai.BasisArrays(I.Basis(m[0], m[1], m[2])) for m in g["mols"]]
        st["mols"], m0, b0 = [], 0, 0
        for ba, p, q in zip(st["arrays"], prm, npair):
            st["mols"].append(tai.tai_mol(ba.struct, tai.make_params(p, st["prec"]), st["M"][m0:].data_ptr(),
                                          st["B"][b0:].data_ptr(), q))
            m0, b0 = m0 + 3 * n * q, b0 + q * q
        return st
    st["basis"], st["params"] = I.Basis(g["cen"], g["alp"], g["pw"]), g["params"]
    st["D"] = [_gpu(d) for d in g["D"]]
    if case["kind"] in ("J", "exchange", "orbital"):   # the moments of the geometry are in hand
        st["M"] = tai.moments(st["basis"], st["params"], coef=g.get("coef"))
    if case.get("prims", 1) > 1:
        st["fmap"] = g["fn"]
    if "Q" in g:
        st["Q"] = _gpu(g["Q"])
    return st


def run(st):
    c, kind, prec, p = st["case"], st["case"]["kind"], st["prec"], st.get("params")
    if kind == "B":
        M = tai.moments(st["basis"], p)
        return {"M": M, "B": tai.assemble_B(M, p, prec=prec)}
    if kind == "batch":
        tai.context().assemble_B_batched(st["mols"])
        return {"M": st["M"], "B": st["B"]}
    if kind == "J":
        if "fmap" in st:
            return tai.apply_J_contracted(st["M"], st["basis"].nb, st["fmap"], st["D"][0], p, prec=prec)
        return tai.apply_J(st["M"], st["D"][0], p, prec=prec)
    if kind == "screened":
        pairs = tai.screen_pairs(st["basis"], SCREEN_TAU)
        M = tai.moments_pairs(st["basis"], p, pairs)
        # the list itself shows in J: the entries of a dropped pair are zero
        return {"kept": pairs.shape[0], "J": tai.apply_J_pairs(M, st["D"][0], pairs, p, prec=prec)}
    if kind == "compressed":
        M = tai.moments(st["basis"], p)
        R, U, Kc = tai.compress_operands(M, p)
        return {"rank": R, "J": [tai.apply_J_compressed(U, Kc, D, p, R, prec=prec) for D in st["D"]]}
    if kind == "boxes":
        pairs, counts, boxes = tai.partition_pairs(st["basis"], BOX_TAU, c["parts"])
        M = tai.moments_partitioned(st["basis"], p, pairs, counts, boxes)
        return {"pairs": pairs, "counts": counts, "boxes": boxes,
                "J": tai.apply_J_partitioned(M, st["D"][0], pairs, counts, boxes, p, prec=prec)}
    if kind == "exchange":
        return tai.exchange(st["M"], st["basis"].nb, st["Q"], p, prec=prec)
    return tai.coulomb_mo(st["M"], st["basis"].nb, st["Q"], p, prec=prec)


# ---- the work of one pass ----------------------------------------------------------
def _pairs(nb):
    return nb * (nb + 1) // 2


def work(case):
    n, nq, kind = case["n"], case["nq"], case["kind"]
    if kind in ("B", "batch"):
        if kind == "B":
            nbs = [_functions(case)]
        else:
            sz = np.random.default_rng(case["sizes"])
            nbs = []
            for _ in range(case["mols"]):
                nbs.append((2 if case["shells"] == "ss" else SHELLS[case["shells"]][0]) *
                           int(sz.integers(case["lo"], case["hi"] + 1)))
                sz.choice([0.3, 0.5, 1.0])
        q = [_pairs(b) for b in nbs]
        return {"bytes": sum(24 * n * x + ESIZE[case["prec"]] * x * x for x in q),
                "flops": sum(nq * (6 * n + 4) * x * (x + 1) / 2 for x in q)}
    nb = _functions(case)
    npair = _pairs(nb * case.get("prims", 1))
    M, phi = 24 * n * npair, 6.0 * nq * n ** 4
    pair_sums = 2.0 * n ** 3 * npair                  # a density on the grid, or the grid onto the pairs
    if kind == "exchange":
        t = case["orbitals"] * nb
        return {"bytes": M + 8 * (t + nb * nb), "flops": t * (2.0 * n ** 3 * nb + phi) + 2.0 * nb * t * n ** 3}
    if kind == "orbital":
        o = case["orbitals"]
        return {"bytes": M + 8 * (o * nb + o * o), "flops": o * (pair_sums + phi) + 2.0 * o * o * n ** 3}
    if kind == "screened":
        kept = 0.2 * npair                            # about a fifth of the pairs are kept at these sizes
        return {"bytes": 48 * n * kept + 20 * nb * nb, "flops": 4.0 * n ** 3 * kept + phi}
    if kind == "compressed":
        b, r = case["builds"], 0.65 * n               # the kept rank is about two thirds of n
        return {"bytes": M + b * (24 * r * npair + 16 * nb * nb),
                "flops": b * (4.0 * r ** 3 * npair + 6.0 * nq * r ** 4) + 12.0 * n * n * npair}
    if kind == "boxes":
        return {"bytes": 2 * M + 20 * nb * nb, "flops": 2 * pair_sums + case["parts"] ** 2 * phi}
    return {"bytes": M + 16 * nb * nb, "flops": 2 * pair_sums + phi}


def _seconds(c):
    w = work(c)
    rate = RATE[c["prec"]] if c["kind"] in ("B", "batch") else 3e13
    return w["flops"] / rate + w["bytes"] / 4e12


# ---- the results in 64 bits ----------------------------------------------------------
def _chebyshev(n):
    """V[a][j] = T_j(u_a) on the Lobatto grid u_a = cos(pi a / (n - 1)), and its inverse."""
    V = np.cos(np.outer(np.pi * np.arange(n) / (n - 1), np.arange(n)))
    return V, np.linalg.inv(V)


def _nodes(p):
    z, w = np.polynomial.legendre.leggauss(p.nq)
    return 0.5 * p.omega * (1 + z), 0.5 * p.omega * w * (2 / math.sqrt(math.pi))


def _grid(n, L):
    return L * np.cos(np.pi * np.arange(n) / (n - 1))


def _tables(p):
    """w [nq] and the node values [nq][n][n] of each factor, cut to its degree with degree_tol > 0."""
    t, w = _nodes(p)
    x = _grid(p.n, p.L)
    K = np.exp(-(t[:, None, None] * (x[:, None] - x[None])) ** 2)
    if p.degree_tol > 0:
        V, Vi = _chebyshev(p.n)
        big = np.maximum.outer(np.arange(p.n), np.arange(p.n))
        for k in range(p.nq):
            C = Vi @ K[k] @ Vi.T
            m = next(m for m in range(1, p.n + 1) if np.abs(C[big >= m]).sum() <= p.degree_tol)
            K[k] = V @ np.where(big < m, C, 0.0) @ V.T
    return _gpu(w), _gpu(K)


def _pair_list(nb):
    return torch.triu_indices(nb, nb, device="cuda")


def _moments(cen, alp, pw, n, L, mu, nu, coef=None):
    """[3][n][pairs]: the pair products against the Lagrange basis, by composite Gauss-Legendre quadrature."""
    cen, alp = _gpu(cen), _gpu(alp)
    pw = torch.as_tensor(pw, device="cuda")
    df = torch.tensor([1.0, 1.0, 3.0, 15.0, 105.0], dtype=F64, device="cuda")
    a = alp[:, None]
    N = torch.sqrt(torch.sqrt(2 * a / math.pi) * (4 * a) ** pw / df[pw.long()])
    if coef is not None:
        N = torch.stack([_gpu(coef)] + 2 * [torch.ones_like(alp)], 1)
    z, zw = (_gpu(v) for v in np.polynomial.legendre.leggauss(48))
    panels = torch.arange(8, dtype=F64, device="cuda")
    Vi = _gpu(_chebyshev(n)[1])
    M = torch.empty((3, n, mu.numel()), dtype=F64, device="cuda")
    for d in range(3):
        for s in range(0, mu.numel(), 32768):
            i, j = mu[s:s + 32768], nu[s:s + 32768]
            p = alp[i] + alp[j]
            A, B = cen[i, d], cen[j, d]
            P = (alp[i] * A + alp[j] * B) / p
            pref = N[i, d] * N[j, d] * torch.exp(-alp[i] * alp[j] / p * (A - B) ** 2)
            lo, hi = torch.clamp(P - 9 / p.sqrt(), min=-L), torch.clamp(P + 9 / p.sqrt(), max=L)
            h = torch.clamp(hi - lo, min=0) / 8
            x = lo[:, None, None] + h[:, None, None] * (panels[:, None] + 0.5 + 0.5 * z[None])
            x = x.reshape(len(i), -1)
            f = (0.5 * h[:, None, None] * zw).expand(-1, 8, -1).reshape(len(i), -1) * pref[:, None]
            f = f * (x - A[:, None]) ** pw[i, d][:, None] * (x - B[:, None]) ** pw[j, d][:, None]
            f = f * torch.exp(-p[:, None] * (x - P[:, None]) ** 2)
            u = x / L
            T0, T1, mom = torch.ones_like(u), u, [f.sum(1), (f * u).sum(1)]
            for _ in range(2, n):
                T0, T1 = T1, 2 * u * T1 - T0
                mom.append((f * T1).sum(1))
            M[d, :, s:s + 32768] = Vi.T @ torch.stack(mom[:n])
    return M


def _exact_B(M, w, K):
    npair = M.shape[2]
    B = torch.empty((npair, npair), dtype=F64, device="cuda")
    step = max(64, min(npair, 200_000_000 // npair))
    KM = [[K[k] @ M[d] for d in range(3)] for k in range(len(w))] if npair < 20000 else None
    for s in range(0, npair, step):
        out = B[s:s + step].zero_()
        rows = [M[d][:, s:s + step].T.contiguous() for d in range(3)]
        for k in range(len(w)):
            f = [rows[d] @ (KM[k][d] if KM else K[k] @ M[d]) for d in range(3)]
            out.addcmul_(f[0].mul_(f[1]), f[2], value=float(w[k]))
    return B


def _density_pairs(D, mu, nu):
    return D[mu, nu] * torch.where(mu == nu, 1.0, 2.0)


def _rho(M, Dt):
    n = M.shape[1]
    r = torch.zeros((n * n, n), dtype=F64, device="cuda")
    for s in range(0, M.shape[2], 16384):
        m = M[:, :, s:s + 16384]
        r += ((Dt[s:s + 16384] * m[0])[:, None] * m[1][None]).reshape(n * n, -1) @ m[2].T.contiguous()
    return r.view(n, n, n)


def _modes(r, K):
    """r x_1 K x_2 K x_3 K for a stack of grid tensors [..., n, n, n]."""
    r = r @ K.T.contiguous()
    r = K @ r
    return (K @ r.reshape(*r.shape[:-2], -1)).reshape(r.shape)


def _phi(rho, w, K):
    out = torch.zeros_like(rho)
    for k in range(len(w)):
        out += w[k] * _modes(rho, K[k])
    return out


def _on_pairs(M, Phi):
    n, out = M.shape[1], []
    for s in range(0, M.shape[2], 16384):
        m = M[:, :, s:s + 16384]
        X = (Phi.reshape(n * n, n) @ m[2].contiguous()).view(n, n, -1)
        out.append(((X * m[1][None]).sum(1) * m[0]).sum(0))
    return torch.cat(out)


def _unpack(v, mu, nu, nb):
    J = torch.zeros((nb, nb), dtype=F64, device="cuda")
    J[mu, nu] = v
    J[nu, mu] = v
    return J


def _exact_J(M, D, mu, nu, w, K):
    return _unpack(_on_pairs(M, _phi(_rho(M, _density_pairs(D, mu, nu)), w, K)), mu, nu, D.shape[0])


def _exact_boxes(g, c, p, D, mu, nu):
    a, cen = _gpu(g["alp"]), _gpu(g["cen"])
    s = a[mu] + a[nu]
    P = (a[mu, None] * cen[mu] + a[nu, None] * cen[nu]) / s[:, None]
    b = P.abs().max(1).values + torch.sqrt(math.log(1 / BOX_TAU) / s)
    srt = b.sort().values
    box = [float(srt[-(-(k + 1) * len(srt) // c["parts"]) - 1]) for k in range(c["parts"])]
    part = torch.bucketize(b, torch.tensor(box, dtype=F64, device="cuda"))
    t, w = _nodes(p)
    sel = [torch.nonzero(part == k).flatten() for k in range(c["parts"])]
    M = [_moments(g["cen"], g["alp"], g["pw"], p.n, v, mu[i], nu[i]) for i, v in zip(sel, box)]
    Dt = _density_pairs(D, mu, nu)
    rho = [_rho(m, Dt[i]) for m, i in zip(M, sel)]
    x = [_grid(p.n, v) for v in box]
    Jp = torch.zeros_like(Dt)
    for k in range(c["parts"]):
        Phi = torch.zeros_like(rho[0])
        for l in range(c["parts"]):
            Phi += _phi(rho[l], _gpu(w), _gpu(np.exp(-(t[:, None, None] * (x[k][:, None] - x[l][None])) ** 2)))
        if len(sel[k]):
            Jp[sel[k]] = _on_pairs(M[k], Phi)
    return {"pairs": torch.cat(sel).int(), "counts": [len(i) for i in sel], "boxes": box,
            "J": _unpack(Jp, mu, nu, D.shape[0])}


def _exact_exchange(M, Q, w, K):
    norb, nb = Q.shape
    n = M.shape[1]
    index = torch.zeros((nb, nb), dtype=torch.long, device="cuda")
    mu, nu = _pair_list(nb)
    index[mu, nu] = index[nu, mu] = torch.arange(len(mu), device="cuda")
    X = torch.empty((nb, norb, n, n, n), dtype=F64, device="cuda")
    for f in range(nb):
        m = M[:, :, index[f]]
        kr = (m[1][:, None] * m[2][None]).reshape(n * n, nb)
        X[f] = ((Q[:, None] * m[0][None]).reshape(norb * n, nb) @ kr.T.contiguous()).view(norb, n, n, n)
    Kx = torch.empty((nb, nb), dtype=F64, device="cuda")
    flat = X.view(nb, -1)
    for s in range(0, nb, 8):
        Kx[:, s:s + 8] = 2 * flat @ _phi(X[s:s + 8], w, K).reshape(-1, flat.shape[1]).T.contiguous()
    return Kx


def exact(case, seed):
    g = _inputs(case, seed)
    kind = case["kind"]
    if kind == "batch":
        Ms, Bs = [], []
        for cen, alp, pw, p in g["mols"]:
            mu, nu = _pair_list(len(alp))
            M = _moments(cen, alp, pw, p.n, p.L, mu, nu)
            w, K = _tables(p)
            Ms.append(M.reshape(-1))
            Bs.append(_exact_B(M, w, K).reshape(-1))
        return {"M": torch.cat(Ms), "B": torch.cat(Bs)}
    p = g["params"]
    mu, nu = _pair_list(len(g["alp"]))
    D = [_gpu(d) for d in g["D"]]
    if kind == "boxes":
        return _exact_boxes(g, case, p, D[0], mu, nu)
    w, K = _tables(p)
    if kind == "screened":
        a, cen = _gpu(g["alp"]), _gpu(g["cen"])
        r2 = ((cen[mu] - cen[nu]) ** 2).sum(1)
        pairs = torch.nonzero(torch.exp(-a[mu] * a[nu] / (a[mu] + a[nu]) * r2) > SCREEN_TAU).flatten()
        mu, nu = mu[pairs], nu[pairs]
        M = _moments(g["cen"], g["alp"], g["pw"], p.n, p.L, mu, nu)
        return {"kept": pairs.numel(), "J": _exact_J(M, D[0], mu, nu, w, K)}
    M = _moments(g["cen"], g["alp"], g["pw"], p.n, p.L, mu, nu, g.get("coef"))
    if kind == "B":
        return {"M": M, "B": _exact_B(M, w, K)}
    if kind == "J" and "coef" in g:
        fn = torch.as_tensor(g["fn"], device="cuda").long()
        S = torch.zeros((D[0].shape[0], len(fn)), dtype=F64, device="cuda")
        S[fn, torch.arange(len(fn), device="cuda")] = 1.0
        return S @ _exact_J(M, D[0][fn][:, fn], mu, nu, w, K) @ S.T
    if kind == "J":
        return _exact_J(M, D[0], mu, nu, w, K)
    if kind == "compressed":
        W = torch.cat([M[0], M[1], M[2]], 1).cpu()
        V, sv, _ = torch.linalg.svd(torch.linalg.qr(W.T.contiguous(), mode="r").R.T)
        R = max(1, int((sv > p.rank_tol * sv[0]).sum()))
        V = V[:, :R].cuda()
        U, Kc = torch.stack([V.T @ M[d] for d in range(3)]), torch.stack([V.T @ k @ V for k in K])
        return {"rank": R, "J": [_exact_J(U, d, mu, nu, w, Kc) for d in D]}
    Q = _gpu(g["Q"])
    if kind == "exchange":
        return _exact_exchange(M, Q, w, K)
    rho = torch.stack([_rho(M, _density_pairs(torch.outer(q, q), mu, nu)) for q in Q])
    return rho.reshape(len(Q), -1) @ _phi(rho, w, K).reshape(len(Q), -1).T
