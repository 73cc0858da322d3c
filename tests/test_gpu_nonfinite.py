"""What a value that is not finite reaches.  A non-finite v (or vector field) at a point makes every
Hamiltonian entry of two functions that both reach the point non-finite; with a vector field or the
kinetic term, entries of two functions that both do not reach it are what they are without the
point.  A non-finite D_ij makes n non-finite wherever both functions reach."""
import numpy as np
import pytest

from tests.gpu_cases import rel_max
from tests.test_h_clusters import _structure

pytestmark = pytest.mark.gpu
TWO = [(0, 0, 0, 1, 1, 2), (0, 0, 1)]
# a few batches in one unit (pairs of the basis kernel), and units in number (rows, clusters)
SHAPES = {"small": (12, TWO, [3.0, 2.5], 6, 14), "large": (64, TWO, [5.0, 4.0], 44, 194)}


def _reach(basis, X, p):
    """Of every function: whether point p lies within its atom's largest cutoff."""
    out = []
    for xyz, sp in zip(basis["atom_xyz"], basis["atom_species"]):
        sh = range(basis["species_shell_ptr"][sp], basis["species_shell_ptr"][sp + 1])
        rc = max(basis["radial_rcut"][basis["shell_radial"][j]] for j in sh)
        out += [((X[p] - xyz) ** 2).sum() < rc * rc] * sum(2 * basis["shell_l"][j] + 1 for j in sh)
    return np.array(out)


def _some_point(basis, X):
    """A point that some functions reach and some do not."""
    for p in range(len(X) // 2, len(X)):
        r = _reach(basis, X, p)
        if 0 < r.sum() < len(r):
            return p, r
    raise AssertionError("no such point")


# entries apart from the point are sums of the same values in another order of FP64 atomics
# (FP32: the same FP32 sums, but for the chunk whose point is left out): 1e-12, 1e-6 of the largest
@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x6"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_potential(shape, prec, bad):
    from paper_1912_06636_amd import nao
    basis, X, w, v = _structure(*SHAPES[shape])
    p, reach = _some_point(basis, X)
    w = w.copy()
    w[p] = 0.25
    both, neither = np.ix_(reach, reach), np.ix_(~reach, ~reach)
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, 200)
    vb, v0 = v.copy(), v.copy()
    vb[p], v0[p] = bad, 0.0
    print("[gpu-case] non-finite v", shape, prec, bad, flush=True)
    assert not np.isfinite(s.integrate_h(vb, precision=prec)[both]).any()
    if prec != "bf16x6":
        a = 0.3 * np.random.default_rng(3).normal(size=(len(X), 3))
        ab = a.copy()
        ab[p] = bad
        for H, H0 in ((s.integrate_h_gga(vb, a, precision=prec), s.integrate_h_gga(v0, a, precision=prec)),
                      (s.integrate_h_gga(v0, ab, precision=prec), s.integrate_h_gga(v0, a, precision=prec)),
                      (s.integrate_h_ks(vb, a, precision=prec), s.integrate_h_ks(v0, a, precision=prec)),
                      (s.integrate_h_ks(vb, precision=prec), s.integrate_h_ks(v0, precision=prec))):
            assert not np.isfinite(H[both]).any()
            assert np.isfinite(H[neither]).all()
            assert rel_max(H[neither], H0[neither]) <= (1e-12 if prec == "fp64" else 1e-6)
    ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x6"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_density_matrix(shape, prec):
    from paper_1912_06636_amd import nao
    basis, X, w, v = _structure(*SHAPES[shape])
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, 200)
    C = np.random.default_rng(5).normal(size=(s.n_basis, 8))
    D = C @ C.T
    i, j = 3, s.n_basis // 2
    D[i, j] = D[j, i] = np.nan
    xyz = basis["atom_xyz"]
    first = np.cumsum([0] + [sum(2 * basis["shell_l"][q] + 1 for q in range(basis["species_shell_ptr"][sp], basis["species_shell_ptr"][sp + 1]))
                             for sp in basis["atom_species"]])
    at = [int(np.searchsorted(first, f, side="right")) - 1 for f in (i, j)]
    rc = [SHAPES[shape][2][basis["atom_species"][k]] for k in at]
    hit = np.all([((X - xyz[k]) ** 2).sum(axis=1) < r * r for k, r in zip(at, rc)], axis=0)
    print("[gpu-case] non-finite D", shape, prec, int(hit.sum()), flush=True)
    assert hit.any() or shape == "small"
    assert np.isnan(s.update_density(D, precision=prec)[hit]).all()
    if prec != "bf16x6":
        n, g = s.update_density_gradient(D, precision=prec)
        assert np.isnan(n[hit]).all() and np.isnan(g[hit]).all()
    ctx.close()
