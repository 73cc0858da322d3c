"""Basis values whose rows are staged on chip (launches of 512 units or more, 12 FP64 functions per atom
and more): one, two and three parts of 16 atoms, ragged last parts, units of two to five rows, two
species of different width, radial grids that differ between the shells of a species, rows too wide for
the stage, and with basis values in unpadded rows; every plane (values, gradient, L, h phi) through the
operations that read it, against the oracle."""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import integrals as oi
from tests.gpu_cases import rel_max
from workloads import generate as g

pytestmark = pytest.mark.gpu

BLOCK, HEAVY = (0, 0, 0, 1, 1, 2), (0, 0, 1, 1, 2, 2, 3)
# (atoms, shells per species, cutoffs, points, largest batch); 16 shells of l = 3 make 112 functions, past the stage
CASES = [
    (1, [BLOCK], [9.0], 1100, 2),
    (16, [BLOCK, HEAVY], [5.0, 7.0], 2600, 5),
    (17, [HEAVY], [6.0], 1700, 3),
    (40, [HEAVY, BLOCK], [4.0, 6.0], 1300, 2),
    (2, [(3,) * 16], [8.0], 1100, 2),
]


@pytest.mark.parametrize("n_atoms,shells,rcut,n_points,max_batch", CASES)
def test_staged_rows(n_atoms, shells, rcut, n_points, max_batch):
    from paper_1912_06636_amd import nao
    rng = g.rng_for(7, 37, 0, n_atoms)
    xyz = g.geometry_sc_first_n(n_atoms, 2.2, 0.1, rng)
    basis = g.make_basis(xyz, (np.arange(n_atoms) % len(shells)).astype(np.int32), shells, rcut, 7, 37)
    if n_atoms == 17:  # the last shell on a grid of its own
        basis["radial_rcut"] = basis["radial_rcut"].copy()
        basis["radial_rcut"][-1] = 4.5
    X = xyz.mean(0) + rng.normal(0.0, 2.5, size=(n_points, 3))
    w, v, a = rng.uniform(0.1, 1.0, n_points), rng.normal(size=n_points), 0.3 * rng.normal(size=(n_points, 3))
    nb = g.n_basis(basis)
    D, Q = (lambda x, y: (x + x.T, y + y.T))(*rng.normal(size=(2, nb, nb)))
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, max_batch)
    s.set_group_max(0)  # one unit per batch
    assert s.n_batches >= 512
    B = ob.Basis(basis)
    perm, bp, lp, li = s.get_batches()
    phi, ptr = s.eval_basis()
    for b in range(0, s.n_batches, 37):
        rb = oi.batch_phi(B, X, perm, bp, lp, li, b)
        assert rb.size == 0 or np.max(np.abs(phi[ptr[b]:ptr[b + 1]].reshape(rb.shape) - rb)) <= 1e-13 * np.max(np.abs(phi))
    n_ref, g_ref = oi.density_gradient(B, X, D)
    refs = [n_ref, n_ref, g_ref, oi.hamiltonian(B, X, w, v), oi.hamiltonian_ks(B, X, w, v, a), oi.pulay_forces(B, X, w, v, D, Q)]
    # as for the same operations on small launches: 1e-12 in FP64; FP32 rounds D and phi, 1e-5
    for prec, tol in (("fp64", 1e-12), ("fp32", 1e-5)):
        n2, gn = s.update_density_gradient(D, precision=prec)
        got = [s.update_density(D, precision=prec), n2, gn, s.integrate_h(v, precision=prec),
               s.integrate_h_ks(v, a, precision=prec), s.pulay_forces(D, Q, v, precision=prec)]
        e = [rel_max(x, y) for x, y in zip(got, refs)]
        print(prec, n_atoms, n_points, ["%.1e" % x for x in e], flush=True)
        assert max(e) <= tol
    ctx.close()
