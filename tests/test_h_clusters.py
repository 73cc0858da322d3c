"""Hamiltonian clusters (runs of execution units contracted as one): the host rule on the CPU, and
on the GPU the same Hamiltonian over clusters, over the units (the form resident basis values
keep) and from the oracle on sampled rows."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import basis as ob
from tests.gpu_cases import rel_max
from workloads import generate as g

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_cluster_rule(tmp_path):
    exe = str(tmp_path / "cluster_check")
    src = [os.path.join(ROOT, "tests", "native", "cluster_check.cpp"),
           os.path.join(ROOT, "paper_1912_06636_amd", "csrc", "plan.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1912_06636_amd", "csrc")] + src + ["-o", exe, "-lpthread"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "all ok" in r.stdout, r.stdout + r.stderr


def _structure(n_atoms, shells, rcut, n_r, n_ang):
    """Two species on a simple-cubic block: columns of odd and even width, ragged lists."""
    xyz = g.geometry_sc_first_n(n_atoms, 2.2, 0.1, g.rng_for(7, 21, 0))
    basis = g.make_basis(xyz, (np.arange(n_atoms) % 2).astype(np.int32), shells, rcut, 7, 21)
    X, w, _ = g.make_grid(xyz, max(rcut), n_r, n_ang)
    v = g.gaussian_potential(X, 8, xyz.min(0), xyz.max(0), g.rng_for(7, 21, 2))
    return basis, X, w, v


def _oracle_rows(B, X, wv, rows):
    """H[rows] = sum_p w v phi_row phi_j in FP64."""
    H = np.zeros((len(rows), B.n_basis))
    for a in range(0, len(X), 20000):
        phi = B.phi(X[a:a + 20000], np.arange(len(B.atom_xyz)))
        H += (phi[:, rows] * wv[a:a + 20000, None]).T @ phi
    return H


# FP64: sums of up to 3e5 products in another order, 1e-12 of the largest entry.  FP32: clusters
# keep each unit's FP32 sums, so the two forms agree like FP64.
@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_atoms,n_r,n_ang,max_batch,batcher", [(34, 44, 194, 200, "octree"), (64, 44, 194, 256, "cutplane")])
def test_clusters_equal_units(prec, n_atoms, n_r, n_ang, max_batch, batcher):
    from paper_1912_06636_amd import nao
    basis, X, w, v = _structure(n_atoms, [(0, 0, 0, 1, 1, 2), (0, 0, 1)], [5.0, 4.0], n_r, n_ang)
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, max_batch, batcher=batcher)
    H = s.integrate_h(v, precision=prec)
    s.set_resident_basis(True)
    H0 = s.integrate_h(v, precision=prec)
    s.set_resident_basis(False)
    s.set_group_max(64)  # other units, other clusters
    H1 = s.integrate_h(v, precision=prec)
    e, e1 = rel_max(H, H0), rel_max(H1, H0)
    print("clusters against units %.2e, other units %.2e" % (e, e1), flush=True)
    assert np.array_equal(H, H.T) and e <= 1e-12 and e1 <= (1e-12 if prec == "fp64" else 1e-6)
    if prec == "fp64":
        B = ob.Basis(basis)
        rows = np.array([0, 13, 14, 18, B.n_basis // 2, B.n_basis - 1])
        ref = _oracle_rows(B, X, w * v, rows)
        er = float(np.max(np.abs(H[rows] - ref))) / float(np.max(np.abs(H)))
        print("against the oracle's rows %.2e" % er, flush=True)
        assert er <= 1e-12
    ctx.close()


@pytest.mark.gpu
def test_clusters_dropped_when_they_do_not_fit():
    """A budget without room for the cluster tables still builds the system and integrates."""
    from paper_1912_06636_amd import nao
    basis, X, w, v = _structure(34, [(0, 0, 0, 1, 1, 2), (0, 0, 1)], [5.0, 4.0], 44, 194)
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, 200)
    H = s.integrate_h(v)
    used = ctx.memory()[0]
    ctx.close()
    for cut in (1 << 16, 1 << 20):  # less than every table, and less than the larger scratch
        small = nao.Context(0, hbm_budget=used - cut)
        t = nao.build_batches(small, basis, X, w, 200)
        import torch
        vd = torch.from_numpy(v).to("cuda:0")
        Hd = torch.empty(t.n_basis, t.n_basis, dtype=torch.float64, device="cuda:0")
        t.integrate_h(vd, out=Hd)
        small.synchronize()
        assert rel_max(Hd.cpu().numpy(), H) <= 1e-12
        small.close()


# The split-BF16 sums of 32 points are the units' own, and what is above them is FP64: 1e-12.
@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["bf16x3", "bf16x6"])
@pytest.mark.parametrize("n_atoms,n_r,n_ang,max_batch,batcher", [(34, 44, 194, 200, "octree"), (64, 44, 194, 256, "cutplane")])
def test_clusters_equal_units_bf16(prec, n_atoms, n_r, n_ang, max_batch, batcher):
    from paper_1912_06636_amd import nao
    basis, X, w, v = _structure(n_atoms, [(0, 0, 0, 1, 1, 2), (0, 0, 1)], [5.0, 4.0], n_r, n_ang)
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, max_batch, batcher=batcher)
    H = s.integrate_h(v, precision=prec)
    s.set_resident_basis(True)
    e = rel_max(H, s.integrate_h(v, precision=prec))
    s.set_resident_basis(False)
    s.set_group_max(0)  # one unit per batch, no clusters, units that end inside a chunk
    e1 = rel_max(H, s.integrate_h(v, precision=prec))
    e64 = rel_max(H, s.integrate_h(v))
    print("clusters against units %.2e, batches %.2e, FP64 %.2e" % (e, e1, e64), flush=True)
    assert np.array_equal(H, H.T) and e <= 1e-12
    tol = {"bf16x3": 3e-5, "bf16x6": 1e-6}[prec]
    assert e1 <= tol and e64 <= tol
    ctx.close()
