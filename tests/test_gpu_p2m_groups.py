"""Moments at the edges of the lane groups of the P2M kernels (box occupancies
around one, two, four, ... lanes and around the slices of the coarse levels), FP64,
every basis, against the CPU oracle.  Tolerance 1e-12 relative L2 of the
potentials, the FP64 mode's; the deepest level alone carries a mean occupancy of
about one, the coarsest one all particles over 16 or 64 boxes."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / max(np.linalg.norm(b), 1e-300))


CASES = [("log2d", 9, 40, 2), ("log2d", 13, 99, 2), ("log2d", 6, 385, 3), ("log2d", 16, 777, 4),
         ("log2d", 21, 3300, 4), ("log2d", 8, 33000, 3), ("log2d", 4, 70001, 2),
         ("log2d", 12, 530001, 6), ("points2d", 4, 500, 3), ("points2d", 4, 33001, 3),
         ("cheb2d", 7, 2000, 3), ("coulomb3d", 3, 100, 2), ("coulomb3d", 8, 1300, 2),
         ("coulomb3d", 5, 140001, 2), ("points3d", 4, 1700, 2), ("cheb3d", 5, 6000, 2),
         ("cheb3d", 3, 700, 3)]


@pytest.mark.parametrize("basis,p,n,L", CASES)
def test_moments_of_every_group_size(basis, p, n, L):
    dim = 2 if basis.endswith("2d") else 3
    kernel = {"log2d": F.FMM_LOG2D, "points2d": F.FMM_LOG2D_POINTS, "cheb2d": F.FMM_LOG2D_CHEBYSHEV,
              "coulomb3d": F.FMM_COULOMB3D, "points3d": F.FMM_COULOMB3D_POINTS,
              "cheb3d": F.FMM_COULOMB3D_CHEBYSHEV}[basis]
    pos, q = workloads.gaussian_mixture(n, dim, seed=n, sigma=0.6)
    f = F.FMM(kernel, levels=L, order=p, max_particles=n, flags=F.FMM_SYNC_CHECK)
    pot, fld = f.evaluate(torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda())
    pot, fld = pot.cpu().numpy(), fld.cpu().numpy()
    f.close()
    tg = workloads.sample_targets(n, 400)
    if basis == "log2d":
        want, wfld = oracle.fmm2d(pos, q, L, p, targets=tg)
    elif basis == "coulomb3d":
        want, wfld = oracle.fmm3d(pos, q, L, p, targets=tg)
    else:
        nodes = oracle.PAPER_NODES if basis.startswith("points") else oracle.chebyshev_nodes(p)
        fn = oracle.fmm2d_lagrange if dim == 2 else oracle.fmm3d_lagrange_nodes
        want, wfld = fn(pos, q, L, nodes=nodes, targets=tg)
    assert rel(pot[tg], want) < 1e-12
    assert rel(fld[tg], wfld) < 1e-12
