"""Staged basis rows over every split of a wave's lanes: one part of 1 to 12 atoms, of 13 to 16, even
parts of 9 to 12, and parts of 16 with a short last one; units of two to many rows, last rows ragged.
Basis values, and every plane through the operations that read it, against the oracle."""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import integrals as oi
from tests.gpu_cases import rel_max
from workloads import generate as g

pytestmark = pytest.mark.gpu
HEAVY, BLOCK = (0, 0, 1, 1, 1, 2, 2, 3), (0, 0, 0, 1, 1, 2)


def _system(n_atoms, shells, n_points, max_batch):
    from paper_1912_06636_amd import nao
    rng = g.rng_for(7, 41, 0, n_atoms)
    xyz = g.geometry_sc_first_n(n_atoms, 1.5, 0.1, rng)
    basis = g.make_basis(xyz, (np.arange(n_atoms) % len(shells)).astype(np.int32), shells, [12.0] * len(shells), 7, 41)
    X = xyz.mean(0) + rng.normal(0.0, 1.5, size=(n_points, 3))  # every atom reaches every point
    w = rng.uniform(0.1, 1.0, n_points)
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, max_batch)
    s.set_group_max(0)  # one unit per batch
    return ctx, s, ob.Basis(basis), X, w, rng


# atoms, species, points, largest batch: at least 4,096 atoms over all units
@pytest.mark.parametrize("n_atoms,shells,n_points,max_batch", [
    (1, [HEAVY], 220000, 100), (2, [BLOCK, HEAVY], 40000, 30), (5, [HEAVY], 80000, 200), (5, [BLOCK], 3000, 5), (12, [BLOCK, HEAVY], 30000, 150),
    (13, [HEAVY], 6000, 29), (17, [BLOCK], 6000, 40), (24, [BLOCK, HEAVY], 3000, 21), (25, [HEAVY], 1500, 7), (33, [BLOCK], 3000, 33), (36, [BLOCK], 900, 9)])
def test_values(n_atoms, shells, n_points, max_batch):
    ctx, s, B, X, w, rng = _system(n_atoms, shells, n_points, max_batch)
    assert s.n_batches * n_atoms >= 4096
    perm, bp, lp, li = s.get_batches()
    phi, ptr = s.eval_basis()
    for b in range(0, s.n_batches, 61):
        rb = oi.batch_phi(B, X, perm, bp, lp, li, b)
        assert np.max(np.abs(phi[ptr[b]:ptr[b + 1]].reshape(rb.shape) - rb)) <= 1e-13 * np.max(np.abs(phi))
    ctx.close()


# as the same operations elsewhere: 1e-12 in FP64, 1e-5 in FP32 (D and phi are rounded)
@pytest.mark.parametrize("n_atoms,shells,n_points,max_batch", [
    (1, [HEAVY], 12000, 4), (5, [HEAVY, BLOCK], 9000, 12), (12, [BLOCK], 8000, 37), (17, [HEAVY], 2600, 13), (24, [BLOCK], 2600, 18), (36, [BLOCK], 900, 9)])
def test_planes(n_atoms, shells, n_points, max_batch):
    ctx, s, B, X, w, rng = _system(n_atoms, shells, n_points, max_batch)
    assert s.n_batches * n_atoms >= 4096
    v, a = rng.normal(size=n_points), 0.3 * rng.normal(size=(n_points, 3))
    D, Q = (lambda x, y: (x + x.T, y + y.T))(*rng.normal(size=(2, s.n_basis, s.n_basis)))
    n_ref, g_ref = oi.density_gradient(B, X, D)
    refs = [n_ref, g_ref, oi.hamiltonian_ks(B, X, w, v, a), oi.pulay_forces(B, X, w, v, D, Q)]
    for prec, tol in (("fp64", 1e-12), ("fp32", 1e-5)):
        got = [*s.update_density_gradient(D, precision=prec), s.integrate_h_ks(v, a, precision=prec), s.pulay_forces(D, Q, v, precision=prec)]
        e = [rel_max(x, y) for x, y in zip(got, refs)]
        print(prec, n_atoms, s.n_batches, ["%.1e" % x for x in e], flush=True)
        assert max(e) <= tol
    ctx.close()
