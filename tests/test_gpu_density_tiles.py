"""Density tiles (n_tiles): units whose point counts meet the edges of its row parts (one row block,
8 and 9 row blocks, a ragged last block), lists that end inside a step or a tile, columns that do not
come in neighbouring pairs, and lists of more than one window of 512 functions; density, gradient
and forces against the oracle."""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import integrals as oi
from tests.gpu_cases import rel_max
from workloads import generate as g

pytestmark = pytest.mark.gpu

# (atoms, shells per species, points, largest batch): 5, 14 and 9 functions per atom, so that lists end
# at 5, 14, 70, 38 (odd and even pairs) and 616 columns (two windows)
CASES = [
    (1, [(0, 0, 1)], 3, 256),
    (1, [(0, 0, 0, 1, 1, 2)], 17, 256),
    (5, [(0, 0, 0, 1, 1, 2)], 128, 128),
    (5, [(0, 0, 0, 1, 1, 2)], 129, 256),
    (4, [(0, 0, 0, 1, 1, 2), (0, 0, 1)], 255, 256),
    (44, [(0, 0, 0, 1, 1, 2)], 700, 256),
    (45, [(0, 1, 2), (0, 0, 1)], 512, 200),
]


@pytest.mark.parametrize("n_atoms,shells,n_points,max_batch", CASES)
def test_density_tiles(n_atoms, shells, n_points, max_batch):
    from paper_1912_06636_amd import nao
    rng = g.rng_for(7, 31, 0, n_atoms)
    xyz = g.geometry_sc_first_n(n_atoms, 1.9, 0.1, rng)
    basis = g.make_basis(xyz, (np.arange(n_atoms) % len(shells)).astype(np.int32), shells, [9.0] * len(shells), 7, 31)
    X = xyz.mean(0) + rng.normal(0.0, 1.5, size=(n_points, 3))
    w, v = rng.uniform(0.1, 1.0, n_points), rng.normal(size=n_points)
    nb = g.n_basis(basis)
    D, Q = (lambda a, b: (a + a.T, b + b.T))(*rng.normal(size=(2, nb, nb)))
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, max_batch)
    B = ob.Basis(basis)
    n_ref, g_ref = oi.density(B, X, D), oi.density_gradient(B, X, D)
    g_ref = g_ref[1] if isinstance(g_ref, tuple) else g_ref
    F_ref = oi.pulay_forces(B, X, w, v, D, Q)
    # sums of up to 616^2 products: 1e-12 of the largest value in FP64; FP32 rounds D and phi, 1e-5
    for prec, tol in (("fp64", 1e-12), ("fp32", 1e-5)):
        n = s.update_density(D, precision=prec)
        n2, gn = s.update_density_gradient(D, precision=prec)
        F = s.pulay_forces(D, Q, v, precision=prec)
        e = [rel_max(n, n_ref), rel_max(n2, n_ref), rel_max(gn, g_ref), rel_max(F, F_ref)]
        print(prec, n_atoms, n_points, ["%.1e" % x for x in e], flush=True)
        assert max(e) <= tol
    ctx.close()
