"""Cases of the grid operations, as a program that uses the library calls them.

Each case is one structure (or several) with the calls a self-consistency cycle makes on it:
`scf` (density from D, then the Hamiltonian from v), `density` and `h` alone, `gga` (density with
its gradient, then the Kohn-Sham Hamiltonian with a vector field), `forces` (the local Pulay term at
the end of a cycle) and `many` (the `scf` calls of several structures in one launch sequence).

Structures follow the shapes of the repository's workloads: atoms in a cube with a minimal basis
(5 functions per atom), simple-cubic blocks with 14 functions, layered slabs with 28, and blocks
that alternate two species; atom-centred shell grids with partition weights; a potential that is a
sum of Gaussians; D = C C^T from random orbitals, cut off at a distance.
"""
import math

import numpy as np
import torch

from paper_1912_06636_amd import nao

DEV = "cuda:0"
N_KNOTS, R_MIN = 200, 1.0e-4

# Species of the styles: (shells l, cutoff in Angstrom), and what goes with them.
LIGHT, BLOCK, SLAB = ((0, 0, 1), 4.0), ((0, 0, 0, 1, 1, 2), 5.0), ((0, 0, 1, 1, 1, 2, 2, 3), 6.0)
STYLES = {
    "cube": dict(species=[LIGHT], n_r=30, n_ang=110, max_batch=200, d_max=None, n_gauss=8),
    "block": dict(species=[BLOCK], n_r=50, n_ang=302, max_batch=256, d_max=10.0, n_gauss=64),
    "mixed": dict(species=[BLOCK, LIGHT], n_r=50, n_ang=302, max_batch=256, d_max=10.0, n_gauss=64),
    "slab": dict(species=[SLAB], n_r=60, n_ang=434, max_batch=256, d_max=12.0, n_gauss=256),
}


def _case(name, op, style, atoms, precision, **more):
    s = STYLES[style]
    c = dict(name=name, op=op, style=style, atoms=atoms, precision=precision, n_r=s["n_r"], n_ang=s["n_ang"],
             max_batch=s["max_batch"], batcher="octree", structures=1, graph=False)
    c.update(more)
    return c


def listed():
    return [
        # the smallest molecule: one tile of functions, a few hundred batches; launches count
        _case("cube8_scf_fp64", "scf", "cube", 8, "fp64"),
        # a small molecule's density with its electron count, the call a cycle waits for
        _case("block20_density_fp64", "density", "block", 20, "fp64"),
        # a two-species cluster on cut-plane batches: ragged lists, the Hamiltonian alone
        _case("mixed27_h_fp64", "h", "mixed", 27, "fp64", batcher="cutplane"),
        # a medium cluster, one iteration of an ordinary cycle
        _case("block100_scf_fp64", "scf", "block", 100, "fp64"),
        # the largest: the layered slab of the benchmark, one iteration
        _case("slab375_scf_fp64", "scf", "slab", 375, "fp64"),
        # a served structure in single precision, the serving path's default
        _case("slab100_scf_fp32", "scf", "slab", 100, "fp32"),
        # split-BF16 products, the other reduced mode
        _case("block64_scf_bf16x6", "scf", "block", 64, "bf16x6"),
        # one iteration with a gradient-corrected functional and the kinetic term
        _case("block100_gga_fp64", "gga", "block", 100, "fp64"),
        # the same in single precision on a small slab
        _case("slab45_gga_fp32", "gga", "slab", 45, "fp32"),
        # forces at the end of a cycle
        _case("slab60_forces_fp64", "forces", "slab", 60, "fp64"),
        # a set of small molecules in one captured sequence, replayed every iteration
        _case("many12_scf_fp64", "many", "block", 12, "fp64", structures=12, graph=True),
        # what a server launches: a few requests of different sizes, eager, in single precision
        _case("many6_scf_fp32", "many", "slab", 20, "fp32", structures=6),
    ]


def draw(rng):
    op = rng.choice(["scf", "scf", "scf", "density", "h", "gga", "forces", "many"])
    style = rng.choice(["cube", "block", "block", "mixed", "slab", "slab"])
    most = {"scf": 375, "density": 375, "h": 375, "gga": 160, "forces": 120, "many": 48}[op]
    atoms = int(round(math.exp(rng.uniform(math.log(8.0), math.log(float(most))))))
    kinds = ["fp64", "fp64", "fp64", "fp32"]
    if op in ("scf", "density", "h", "many"):
        kinds += ["bf16x3", "bf16x6"]
    c = _case("", op, style, atoms, rng.choice(kinds))
    del c["name"]
    c["n_r"] = rng.randint(24, c["n_r"])
    c["n_ang"] = rng.randint(86, c["n_ang"])
    c["max_batch"] = rng.choice([96, 150, 200, 256])
    c["batcher"] = rng.choice(["octree", "octree", "cutplane"])
    if op == "many":
        c["structures"] = rng.randint(2, 12)
        c["graph"] = rng.random() < 0.5
    return c


# ----------------------------------------------------------------------------------------------
# inputs

def _positions(style, n, rng):
    if style == "cube":  # rejection sampling with a minimum separation
        side, out = 6.0 * (n / 8.0) ** (1.0 / 3.0), []
        while len(out) < n:
            p = rng.uniform(0.0, side, size=3)
            if all(((p - q) ** 2).sum() >= 1.0 for q in out):
                out.append(p)
        return np.array(out)
    if style == "slab":  # five honeycomb layers, the sites nearest the centre
        per, ax, ay = -(-n // 5), math.sqrt(3.0) * 2.5, 7.5
        k = int(math.sqrt(per)) + 3
        cell = np.array([[0.0, 0.0], [ax / 2, 1.25], [ax / 2, 3.75], [0.0, 5.0]])
        s = np.array([[i * ax, j * ay] + cell[b] for i in range(-k, k + 1) for j in range(-k, k + 1) for b in range(4)])
        plane = s[np.argsort(((s - [0.3, 0.2]) ** 2).sum(axis=1), kind="stable")[:per]]
        xyz = np.concatenate([np.column_stack([plane + [2.5 * (l % 2), 0.0], np.full(per, 3.75 * l)]) for l in range(5)])[:n]
        return xyz + rng.normal(0.0, 0.05, size=xyz.shape)
    side = 1
    while side ** 3 < n:
        side += 1
    k, j, i = np.meshgrid(np.arange(side), np.arange(side), np.arange(side), indexing="ij")
    xyz = np.stack([i.ravel(), j.ravel(), k.ravel()], axis=1)[:n] * 2.2
    return xyz + rng.normal(0.0, 0.1, size=xyz.shape)


def _basis(case, xyz, rng):
    species = STYLES[case["style"]]["species"]
    ptr, ls, rad, rcut, samples = [0], [], [], [], []
    for shells, rc in species:
        r = R_MIN * np.exp(np.arange(N_KNOTS) * (math.log(rc / R_MIN) / (N_KNOTS - 1)))
        r[0], r[-1] = R_MIN, rc
        x = (np.arange(4000) + 0.5) * (rc / 4000)
        for l in shells:
            c, a = rng.normal(size=3), np.exp(rng.uniform(math.log(0.25), math.log(4.0), size=3))

            def R(q):
                return np.maximum(0.0, 1.0 - (q / rc) ** 2) ** 3 * q ** l * (c * np.exp(-a * q[:, None] ** 2)).sum(axis=1)

            y = R(r) / math.sqrt(float((R(x) ** 2 * x ** 2).sum() * (rc / 4000)))
            y[-1] = 0.0
            rad.append(len(samples))
            ls.append(l)
            rcut.append(rc)
            samples.append(y)
        ptr.append(len(ls))
    return dict(atom_xyz=np.ascontiguousarray(xyz), atom_species=(np.arange(len(xyz)) % len(species)).astype(np.int32),
                species_shell_ptr=np.array(ptr, np.int32), shell_l=np.array(ls, np.int32), shell_radial=np.array(rad, np.int32),
                radial_rmin=np.full(len(rad), R_MIN), radial_rcut=np.array(rcut), radial_samples=np.array(samples), n_knots=N_KNOTS)


def _shape(case, xyz):
    """(functions per atom, cutoff per atom) as arrays."""
    species = STYLES[case["style"]]["species"]
    sp = np.arange(len(xyz)) % len(species)
    return np.array([sum(2 * l + 1 for l in s[0]) for s in species])[sp], np.array([s[1] for s in species])[sp]


def _points(case, atoms):
    """Atom-centred shell grid on the GPU: Becke's radial map, Fibonacci spheres."""
    n_r, n_ang = case["n_r"], case["n_ang"]
    th = torch.arange(1, n_r + 1, dtype=torch.float64, device=DEV) * (math.pi / (n_r + 1))
    x = torch.cos(th)
    r = (1.0 + x) / (1.0 - x)
    wr = (math.pi / (n_r + 1)) * torch.sin(th) * 2.0 / (1.0 - x) ** 2 * r ** 2
    k = torch.arange(n_ang, dtype=torch.float64, device=DEV)
    z = 1.0 - (2.0 * k + 1.0) / n_ang
    ph, s = k * (math.pi * (3.0 - math.sqrt(5.0))), torch.sqrt(1.0 - z * z)
    u = torch.stack([s * torch.cos(ph), s * torch.sin(ph), z], dim=1)
    shell = (r[:, None, None] * u[None]).reshape(-1, 3)
    return (atoms[:, None] + shell[None]).reshape(-1, 3).contiguous(), (wr * (4.0 * math.pi / n_ang)).repeat_interleave(n_ang)


def _weights(pts, shell_w, atoms):
    """Stockholder partition with one-atom profiles exp(-2 r) / (r^2 + 0.1)."""
    out = torch.empty(len(pts), dtype=torch.float64, device=DEV)
    owner = torch.arange(len(pts), device=DEV) // len(shell_w)
    step = max(1, 60_000_000 // len(atoms))
    for a in range(0, len(pts), step):
        d = torch.sqrt(sum((pts[a:a + step, c, None] - atoms[None, :, c]) ** 2 for c in range(3)))
        lg = -2.0 * d - torch.log(d * d + 0.1)
        out[a:a + step] = torch.softmax(lg, dim=1).gather(1, owner[a:a + step, None])[:, 0]
    return out * shell_w.repeat(len(atoms))


def _inputs(case, seed, index=0):
    """The structure and its fields: the points and the basis on the host, v, a, D, Q on the GPU."""
    rng = np.random.default_rng([seed, index, 1912])
    st = STYLES[case["style"]]
    n_at = case["atoms"] + (index * case["atoms"]) // 4 if case["op"] == "many" else case["atoms"]
    xyz = _positions(case["style"], n_at, rng)
    basis = _basis(case, xyz, rng)
    at = torch.from_numpy(xyz).to(DEV)
    pts, shell_w = _points(case, at)
    w = _weights(pts, shell_w, at)
    gen = torch.Generator(device=DEV).manual_seed(int(rng.integers(1 << 62)))
    f64 = dict(dtype=torch.float64, device=DEV)
    v = torch.zeros(len(pts), **f64)
    lo, hi = torch.from_numpy(xyz.min(axis=0)).to(DEV), torch.from_numpy(xyz.max(axis=0)).to(DEV)
    for _ in range(st["n_gauss"]):
        c = lo + (hi - lo) * torch.rand(3, generator=gen, **f64)
        amp, sig = torch.randn(1, generator=gen, **f64), 0.5 + 1.5 * torch.rand(1, generator=gen, **f64)
        v += amp * torch.exp(-sum((pts[:, k] - c[k]) ** 2 for k in range(3)) / (2.0 * sig * sig))
    nf, rc = _shape(case, xyz)
    of = torch.from_numpy(np.repeat(np.arange(n_at), nf)).to(DEV)
    C = torch.randn(len(of), max(2, 4 * n_at), generator=gen, **f64)
    near = torch.ones(n_at, n_at, dtype=torch.bool, device=DEV) if st["d_max"] is None else torch.cdist(at, at) <= st["d_max"]
    keep = near[of][:, of]
    def matrix(X):
        return torch.where(keep, 0.5 * (X + X.T), torch.zeros((), **f64)).contiguous()

    inp = dict(basis=basis, pts=pts, w=w, v=v, nf=nf, rc=rc, n_basis=len(of))
    if case["op"] != "h":
        inp["D"] = matrix(C @ C.T)
    if case["op"] == "forces":
        e = -1.0 + 0.95 * torch.rand(C.shape[1], generator=gen, **f64)
        inp["Q"] = matrix((C * e) @ C.T)
    if case["op"] == "gga":
        inp["a"] = 0.3 * torch.randn(len(pts), 3, generator=gen, **f64)
    return inp


def prepare(case, seed):
    ctx = nao.Context(0)
    parts = []
    for k in range(case["structures"]):
        inp = _inputs(case, seed, k)
        sysm = nao.build_batches(ctx, inp["basis"], inp["pts"].cpu().numpy(), inp["w"].cpu().numpy(), case["max_batch"],
                                 batcher=case["batcher"])
        p = {key: inp[key] for key in ("v", "D", "Q", "a") if key in inp}
        p["sys"] = sysm
        f64 = dict(dtype=torch.float64, device=DEV)
        if case["op"] == "forces":
            p["F"] = torch.zeros(sysm.n_atoms, 3, **f64)
        else:
            if case["op"] != "h":
                p["n"] = torch.zeros(sysm.n_points, **f64)
            if case["op"] != "density":
                p["H"] = torch.zeros(sysm.n_basis, sysm.n_basis, **f64)
        if case["op"] == "gga":
            p["gn"] = torch.zeros(sysm.n_points, 3, **f64)
        parts.append(p)
    work = None
    if case["op"] == "many":
        work = [x for p in parts for x in ((p["sys"], "n", p["D"], p["n"]), (p["sys"], "h", p["v"], p["H"]))]
    return dict(case=case, ctx=ctx, parts=parts, work=work)


def run(state):
    case, p = state["case"], state["parts"][0]
    op, prec = case["op"], case["precision"]
    if op == "many":
        state["ctx"].run_many(state["work"], precision=prec, capture_graph=case["graph"])
        return [{"n": q["n"], "H": q["H"]} for q in state["parts"]]
    s = p["sys"]
    if op == "density":
        n, ne = s.update_density(p["D"], precision=prec, out=p["n"], electrons=True)
        return {"n": n, "ne": ne}
    if op == "h":
        return {"H": s.integrate_h(p["v"], precision=prec, out=p["H"])}
    if op == "scf":
        s.update_density(p["D"], precision=prec, out=p["n"])
        s.integrate_h(p["v"], precision=prec, out=p["H"])
        return {"n": p["n"], "H": p["H"]}
    if op == "gga":
        s.update_density_gradient(p["D"], precision=prec, out=p["n"], out_grad=p["gn"])
        s.integrate_h_ks(p["v"], p["a"], precision=prec, out=p["H"])
        return {"n": p["n"], "gn": p["gn"], "H": p["H"]}
    return {"F": s.pulay_forces(p["D"], p["Q"], p["v"], precision=prec, out=p["F"])}


# ----------------------------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    """Flops: per point with m functions that reach it, the symmetric product m (m + 1) of the
    density or of the Hamiltonian (twice that for two-factor products, 2 m^2 for a full product).
    Bytes: points, fields and matrices, each once."""
    nbytes = flops = 0.0
    op = case["op"]
    for k in range(case["structures"]):
        rng = np.random.default_rng([0, k, 1912])
        n_at = case["atoms"] + (k * case["atoms"]) // 4 if op == "many" else case["atoms"]
        xyz = _positions(case["style"], n_at, rng)
        nf, rc = _shape(case, xyz)
        at = torch.from_numpy(xyz).to(DEV)
        nft, rc2 = torch.from_numpy(nf.astype(np.float64)).to(DEV), torch.from_numpy(rc ** 2).to(DEV)
        pts, _ = _points(case, at)
        s1 = s2 = 0.0
        step = max(1, 60_000_000 // n_at)
        for a in range(0, len(pts), step):
            d2 = sum((pts[a:a + step, c, None] - at[None, :, c]) ** 2 for c in range(3))
            m = ((d2 < rc2).double() * nft).sum(dim=1)
            s1 += float(m.sum())
            s2 += float((m * m).sum())
        npt, nb2 = len(pts), float(nf.sum()) ** 2
        sym = s2 + s1
        flops += {"density": sym + 2 * s1, "h": sym + s1, "scf": 2 * sym + 3 * s1, "many": 2 * sym + 3 * s1,
                  "gga": 2 * s2 + 8 * s1 + 2 * sym, "forces": 4 * s2 + 6 * s1}[op]
        words = {"density": 6 * npt + nb2, "h": 5 * npt + nb2, "scf": 10 * npt + 2 * nb2, "many": 10 * npt + 2 * nb2,
                 "gga": 15 * npt + 2 * nb2, "forces": 5 * npt + 2 * nb2}[op]
        nbytes += 8.0 * words
    return {"bytes": nbytes, "flops": flops}


# ----------------------------------------------------------------------------------------------
# the same results from plain FP64 tensor operations

def _spline(basis):
    """(y, M) per radial function: natural cubic splines over unit-spaced knots."""
    y = np.asarray(basis["radial_samples"])
    n = y.shape[1]
    A = np.zeros((n, n))
    i = np.arange(1, n - 1)
    A[i, i - 1], A[i, i], A[i, i + 1] = 1.0, 4.0, 1.0
    A[0, 0] = A[-1, -1] = 1.0
    rhs = np.zeros_like(y)
    rhs[:, 1:-1] = 6.0 * (y[:, :-2] - 2.0 * y[:, 1:-1] + y[:, 2:])
    return torch.from_numpy(y).to(DEV), torch.from_numpy(np.linalg.solve(A, rhs.T).T.copy()).to(DEV)


def _harmonics(l, x, y, z):
    """Real harmonics of degree l as (value, d/dx, d/dy, d/dz) of their polynomials on the sphere."""
    o, q = torch.zeros_like(x), torch.ones_like(x)
    s = math.sqrt
    if l == 0:
        return [(q * (0.5 / s(math.pi)), o, o, o)]
    if l == 1:
        c = s(0.75 / math.pi)
        return [(c * y, o, c * q, o), (c * z, o, o, c * q), (c * x, c * q, o, o)]
    if l == 2:
        a, b, c = 0.5 * s(15 / math.pi), 0.25 * s(5 / math.pi), 0.25 * s(15 / math.pi)
        return [(a * x * y, a * y, a * x, o), (a * y * z, o, a * z, a * y), (b * (3 * z * z - 1), o, o, 6 * b * z),
                (a * x * z, a * z, o, a * x), (c * (x * x - y * y), 2 * c * x, -2 * c * y, o)]
    a, b, c = 0.25 * s(35 / (2 * math.pi)), 0.5 * s(105 / math.pi), 0.25 * s(21 / (2 * math.pi))
    d, e = 0.25 * s(7 / math.pi), 0.25 * s(105 / math.pi)
    return [(a * y * (3 * x * x - y * y), 6 * a * x * y, 3 * a * (x * x - y * y), o),
            (b * x * y * z, b * y * z, b * x * z, b * x * y),
            (c * y * (5 * z * z - 1), o, c * (5 * z * z - 1), 10 * c * y * z),
            (d * (5 * z ** 3 - 3 * z), o, o, d * (15 * z * z - 3)),
            (c * x * (5 * z * z - 1), c * (5 * z * z - 1), o, 10 * c * x * z),
            (e * z * (x * x - y * y), 2 * e * x * z, -2 * e * y * z, e * (x * x - y * y)),
            (a * x * (x * x - 3 * y * y), 3 * a * (x * x - y * y), -6 * a * x * y, o)]


def _values(basis, spl, pts, atoms, extra):
    """phi [points, functions of atoms] and, with extra, its gradient and Laplacian."""
    y, M = spl
    A = torch.from_numpy(basis["atom_xyz"][atoms]).to(DEV)
    d = [pts[:, c, None] - A[None, :, c] for c in range(3)]
    d2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
    r = torch.sqrt(d2)
    ir = torch.where(r > 0, 1.0 / r, torch.zeros_like(r))
    u = [d[0] * ir, d[1] * ir, torch.where(r > 0, d[2] * ir, torch.ones_like(r))]
    cols = [[] for _ in range(5 if extra else 1)]
    species = basis["atom_species"][atoms]
    out = [None] * len(atoms)
    for sp in np.unique(species):
        sel = torch.from_numpy(np.nonzero(species == sp)[0]).to(DEV)
        rs, us = r[:, sel], [q[:, sel] for q in u]
        cols = [[] for _ in range(5 if extra else 1)]
        for j in range(basis["species_shell_ptr"][sp], basis["species_shell_ptr"][sp + 1]):
            l, k = int(basis["shell_l"][j]), int(basis["shell_radial"][j])
            rmin, rc = float(basis["radial_rmin"][k]), float(basis["radial_rcut"][k])
            delta = math.log(rc / rmin) / (N_KNOTS - 1)
            t = torch.clamp(torch.log(torch.clamp(rs, min=rmin) / rmin) / delta, 0.0, float(N_KNOTS - 1))
            i = torch.clamp(t.floor().long(), max=N_KNOTS - 2)
            w = t - i
            v, ya, yb, ma, mb = 1.0 - w, y[k][i], y[k][i + 1], M[k][i] / 6.0, M[k][i + 1] / 6.0
            live = d2[:, sel] < rc * rc
            R = torch.where(live, v * (ya + (v * v - 1.0) * ma) + w * (yb + (w * w - 1.0) * mb), torch.zeros_like(v))
            if extra:
                on = live & (rs > rmin)
                q = torch.where(on, 1.0 / rs, torch.zeros_like(rs))
                S1 = ((yb - ya) - (3 * v * v - 1) * ma + (3 * w * w - 1) * mb) / delta
                S2 = 6.0 * (v * ma + w * mb) / (delta * delta)
                lap, dR = (S2 + S1 - l * (l + 1) * R) * q * q, S1 * q
            for val, gx, gy, gz in _harmonics(l, *us):
                cols[0].append(R * val)
                if extra:
                    ug = us[0] * gx + us[1] * gy + us[2] * gz
                    for c, g in enumerate((gx, gy, gz)):
                        cols[1 + c].append(torch.where(on, dR * us[c] * val + R * q * (g - us[c] * ug), torch.zeros_like(R)))
                    cols[4].append(lap * val)
        block = [torch.stack(c, dim=2) for c in cols]
        for n, a in enumerate(sel.tolist()):
            out[a] = [b[:, n] for b in block]
    return [torch.cat([o[q] for o in out], dim=1) for q in range(5 if extra else 1)]


def _exact_one(case, seed, index):
    inp = _inputs(case, seed, index)
    basis, pts, op = inp["basis"], inp["pts"], case["op"]
    spl = _spline(basis)
    xyz, rc, nf = basis["atom_xyz"], inp["rc"], inp["nf"]
    first = np.concatenate([[0], np.cumsum(nf)])
    f64 = dict(dtype=torch.float64, device=DEV)
    nb, npt = inp["n_basis"], len(pts)
    res = {}
    if op in ("scf", "density", "gga", "many"):
        res["n"] = torch.zeros(npt, **f64)
    if op in ("scf", "h", "gga", "many"):
        res["H"] = torch.zeros(nb, nb, **f64)
    if op == "gga":
        res["gn"] = torch.zeros(npt, 3, **f64)
    F = torch.zeros(nb, 3, **f64) if op == "forces" else None
    # cells of 3 Angstrom: the points of a cell against the atoms that reach any of them
    lo = torch.from_numpy(xyz.min(axis=0) - rc.max()).to(DEV)
    span = np.ceil((xyz.max(axis=0) - xyz.min(axis=0) + 2 * rc.max()) / 3.0).astype(np.int64) + 1
    cell = torch.floor((pts - lo) / 3.0).long()
    inside = ((cell >= 0) & (cell < torch.from_numpy(span).to(DEV))).all(dim=1)
    key = (cell[:, 0] * int(span[1]) + cell[:, 1]) * int(span[2]) + cell[:, 2]
    order = torch.argsort(torch.where(inside, key, torch.full_like(key, -1)), stable=True)
    order = order[int((~inside).sum()):]
    ids, counts = torch.unique_consecutive(key[order], return_counts=True)
    at, rct = torch.from_numpy(xyz).to(DEV), torch.from_numpy(rc).to(DEV)
    begin = 0
    for count in counts.tolist():
        for b in range(begin, begin + count, 16384):
            ix = order[b:min(b + 16384, begin + count)]
            P = pts[ix]
            atoms = np.nonzero((torch.cdist(P, at, compute_mode="donot_use_mm_for_euclid_dist").amin(dim=0) < rct + 1e-9).cpu().numpy())[0]
            if not len(atoms):
                continue
            fn = torch.from_numpy(np.concatenate([np.arange(first[a], first[a + 1]) for a in atoms])).to(DEV)
            val = _values(basis, spl, P, atoms, op in ("gga", "forces"))
            phi, w = val[0], inp["w"][ix, None]
            v = inp["v"][ix, None]
            if "D" in inp:
                Db = inp["D"][fn][:, fn]
            if op in ("scf", "density", "gga", "many"):
                T = phi @ Db
                res["n"][ix] = (T * phi).sum(dim=1)
            if op == "gga":
                res["gn"][ix] = torch.stack([2.0 * (T * val[1 + c]).sum(dim=1) for c in range(3)], dim=1)
                a = inp["a"][ix]
                L = w * (0.5 * v * phi - 0.25 * val[4] + sum(a[:, c, None] * val[1 + c] for c in range(3)))
                K = phi.T @ L
                res["H"].index_put_((fn[:, None], fn[None, :]), K + K.T, accumulate=True)
            elif "H" in res:
                res["H"].index_put_((fn[:, None], fn[None, :]), (phi * (w * v)).T @ phi, accumulate=True)
            if op == "forces":
                G = (w * (v * phi - 0.5 * val[4])) @ Db - (w * phi) @ inp["Q"][fn][:, fn]
                F.index_put_((fn,), torch.stack([(val[1 + c] * G).sum(dim=0) for c in range(3)], dim=1), accumulate=True)
        begin += count
    if op == "density":
        res["ne"] = float((inp["w"] * res["n"]).sum())
    if op == "forces":
        owner = torch.from_numpy(np.repeat(np.arange(len(nf)), nf)).to(DEV)
        res["F"] = 2.0 * torch.zeros(len(nf), 3, **f64).index_add_(0, owner, F)
    return res


def exact(case, seed):
    if case["op"] == "many":
        return [_exact_one(case, seed, k) for k in range(case["structures"])]
    return _exact_one(case, seed, 0)
