"""Force sums kept in copies: the forces of four atoms among none or many far ones (the copies' stride),
from a few items (some copies stay empty) and from many, against the four alone."""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import integrals as oi
from tests.gpu_cases import rel_max
from tests.test_density_wide_d import far_structure

pytestmark = pytest.mark.gpu


# as the other force cases: 1e-12 in FP64, 1e-5 in FP32 (D, Q, phi and h phi are rounded)
@pytest.mark.parametrize("n_atoms", [4, 205])
def test_forces_from_the_copies(n_atoms):
    from paper_1912_06636_amd import nao
    full, four, X, w, fn = far_structure(n_atoms)
    rng = np.random.default_rng(4)
    D4, Q4 = (lambda x, y: (x + x.T, y + y.T))(*rng.normal(size=(2, 40, 40)))
    v = rng.normal(size=len(X))
    D, Q = np.zeros((2, 10 * n_atoms, 10 * n_atoms))
    D[np.ix_(fn, fn)], Q[np.ix_(fn, fn)] = D4, Q4
    ref = np.zeros((n_atoms, 3))
    ref[[0, 1, n_atoms - 2, n_atoms - 1]] = oi.pulay_forces(ob.Basis(four), X, w, v, D4, Q4)
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, full, X, w, 20)
    for groups in (256, 16):
        s.set_group_max(groups)
        for prec, tol in (("fp64", 1e-12), ("fp32", 1e-5)):
            F = s.pulay_forces(D, Q, v, precision=prec)
            print("[gpu-case] N_b %d, groups %d, %s: %.1e" % (10 * n_atoms, groups, prec, rel_max(F, ref)), flush=True)
            assert rel_max(F, ref) <= tol
    ctx.close()
