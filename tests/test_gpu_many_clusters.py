"""nao_run_many over a system large enough for Hamiltonian clusters beside small ones: eager and
captured, before and after other execution groups, against the single calls; and a Hamiltonian
whose clusters an allocation of the same context took back."""
import numpy as np
import pytest

from tests.gpu_cases import rel_max
from tests.test_h_clusters import _structure

pytestmark = pytest.mark.gpu
BIG = (64, [(0, 0, 0, 1, 1, 2), (0, 0, 1)], [5.0, 4.0], 44, 194)  # about 21,000 tile pairs; clusters start at 12,288
SMALL = (6, [(0, 0, 0, 1, 1, 2), (0, 0, 1)], [5.0, 4.0], 12, 38)


def _density(n_basis, seed):
    C = np.random.default_rng(seed).normal(size=(n_basis, 12))
    return C @ C.T


# The same kernels with the same FP32 and split-BF16 sums as the single calls; only FP64 sums differ in
# order, 5e5 of them at most: 1e-12 of the largest entry.
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x6"])
@pytest.mark.parametrize("capture", [False, True])
def test_many_with_clusters_equals_single_calls(prec, capture):
    import torch
    from paper_1912_06636_amd import nao
    ctx = nao.Context(0)
    parts = []
    for k, shape in enumerate((SMALL, BIG, SMALL)):
        basis, X, w, v = _structure(*shape)
        s = nao.build_batches(ctx, basis, X, w, 200)
        parts.append((s, v, _density(s.n_basis, k)))
    dev = [(torch.from_numpy(v).cuda(), torch.from_numpy(D).cuda(), torch.empty(s.n_basis, s.n_basis, dtype=torch.float64, device="cuda"),
            torch.empty(s.n_points, dtype=torch.float64, device="cuda")) for s, v, D in parts]
    work = [x for (s, _, _), (v, D, H, n) in zip(parts, dev) for x in ((s, "h", v, H), (s, "n", D, n))]
    for groups in (256, 96, 256):
        for s, _, _ in parts:
            if groups != 256 or capture:
                s.set_group_max(groups)
        for rep in range(3):
            for _, _, H, n in dev:
                H.fill_(7.0)
                n.fill_(-3.0)
            torch.cuda.synchronize()
            ctx.run_many(work, precision=prec, capture_graph=capture)
            ctx.synchronize()
            print("[gpu-case] many with clusters", prec, capture, groups, rep, flush=True)
            for (s, v, D), (_, _, H, n) in zip(parts, dev):
                assert rel_max(H.cpu().numpy(), s.integrate_h(v, precision=prec)) <= 1e-12
                assert rel_max(n.cpu().numpy(), s.update_density(D, precision=prec)) <= 1e-12
    ctx.close()


def test_clusters_given_back_to_a_second_system():
    import torch
    from paper_1912_06636_amd import nao
    basis, X, w, v = _structure(*BIG)
    ctx = nao.Context(0)
    s = nao.build_batches(ctx, basis, X, w, 200)
    own, used = s.info()[3], ctx.memory()[0]
    H = s.integrate_h(v)
    ctx.close()
    # room for the system, its clusters and not quite another one
    tight = nao.Context(0, hbm_budget=used + own * 4 // 5)
    a = nao.build_batches(tight, basis, X, w, 200)
    vd = torch.from_numpy(v).cuda()
    Hd = torch.full((a.n_basis, a.n_basis), float("nan"), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    tight.run_many([(a, "h", vd, Hd)], capture_graph=True)
    tight.synchronize()
    assert rel_max(Hd.cpu().numpy(), H) <= 1e-12
    with_clusters = a.info()[3]
    b = nao.build_batches(tight, basis, X, w, 200)
    print("[gpu-case] clusters given back: %d -> %d bytes" % (with_clusters, a.info()[3]), flush=True)
    assert a.info()[3] < with_clusters
    for s, captured in ((a, False), (b, False), (a, True), (b, True), (a, True)):
        Hd.fill_(float("nan"))
        torch.cuda.synchronize()
        if captured:
            tight.run_many([(s, "h", vd, Hd)], capture_graph=True)
        else:
            s.integrate_h(vd, out=Hd)
        tight.synchronize()
        assert rel_max(Hd.cpu().numpy(), H) <= 1e-12
    tight.close()
