"""D beyond 2^31 bytes: the 32-bit offsets on the CPU, and on the GPU n and grad n of four atoms at the
two ends of a list of far ones against the four alone."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import basis as ob
from oracle import integrals as oi
from tests.gpu_cases import rel_max
from workloads import generate as g

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_06636_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def far_structure(n_atoms):
    """Atoms of 10 functions far from the points and from each other, but for the first two and the last
    two: (basis, basis of those four, points, weights, the four's functions in the whole basis)."""
    near = np.array([0, 1, n_atoms - 2, n_atoms - 1])
    xyz = np.zeros((n_atoms, 3))
    xyz[:, 0] = 200.0 + 10.0 * np.arange(n_atoms)
    xyz[near] = [[0.0, 0.0, 0.0], [1.7, 0.4, 0.0], [0.3, 2.1, 0.2], [1.1, 0.9, 1.6]]
    full = g.make_basis(xyz, np.zeros(n_atoms, np.int32), [(0, 1, 1, 1)], [4.0], 11, 5)
    four = dict(full, atom_xyz=xyz[near].copy(), atom_species=np.zeros(4, np.int32))
    X = np.random.default_rng(1).normal(0.8, 1.4, size=(700, 3))
    return full, four, X, np.full(len(X), 0.1), (10 * near[:, None] + np.arange(10)).ravel()


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")), reason="needs g++ and the HIP headers")
def test_offsets(tmp_path):
    exe = str(tmp_path / "offset_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I", CSRC,
                    "-isystem", os.path.join(ROCM, "include"), os.path.join(ROOT, "tests", "native", "offset_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "all ok" in r.stdout, r.stdout + r.stderr


# 10 functions per atom: 16,380 and 16,390 lie on either side of 2^31 bytes, 23,170 and 23,180 on either
# side of the switch to addresses by row.  FP64 as the other parity cases (1e-12), FP32 its stated 1e-6.
@pytest.mark.gpu
@pytest.mark.parametrize("n_atoms", [1638, 1639, 2317, 2318])
def test_density_of_a_wide_matrix(n_atoms):
    import torch
    from paper_1912_06636_amd import nao
    full, four, X, w, fn = far_structure(n_atoms)
    C = np.random.default_rng(2).normal(size=(40, 9))
    D4 = C @ C.T
    nb = 10 * n_atoms
    D = torch.zeros(nb, nb, dtype=torch.float64, device="cuda")
    ix = torch.from_numpy(fn).cuda()
    D[ix[:, None], ix[None, :]] = torch.from_numpy(D4).cuda()
    B = ob.Basis(four)
    ref, (_, gref) = oi.density(B, X, D4), oi.density_gradient(B, X, D4)
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, full, X, w, 200)
    out = [torch.full((len(X),), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]
    gn = torch.full((len(X), 3), float("nan"), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    s.update_density(D, out=out[0])
    s.update_density(D, precision="fp32", out=out[1])
    s.update_density_gradient(D, out=out[2], out_grad=gn)
    ctx.synchronize()
    e = [rel_max(o.cpu().numpy(), ref) for o in out] + [rel_max(gn.cpu().numpy(), gref)]
    print("[gpu-case] N_b %d: n %.1e, FP32 %.1e, with gradient %.1e, gradient %.1e" % (nb, *e), flush=True)
    assert s.n_basis == nb and e[0] <= 1e-12 and e[1] <= 1e-6 and e[2] <= 1e-12 and e[3] <= 1e-12
    ctx.close()
