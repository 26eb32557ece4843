"""The 3D contraction at the levels where its launches change (levels 2 to 4 split
over offset chunks, level 5 and beyond whole tiles; one or two operator buffers;
four and eight waves), every basis and precision, against the CPU oracle.
Tolerances: 1e-12 (FP64) and 1e-6 (FP32) relative L2 of the potentials, as for the
modes."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("prec,tol", [(F.FMM_FP64, 1e-12), (F.FMM_FP32, 1e-6)])
@pytest.mark.parametrize("basis,p,n,L", [("harm", 8, 900, 2), ("harm", 8, 5000, 4),
                                         ("harm", 3, 20000, 5), ("harm", 8, 9000, 5),
                                         ("harm", 4, 30000, 6), ("points", 4, 9000, 4),
                                         ("points", 4, 9000, 5), ("cheb", 3, 5000, 4),
                                         ("cheb", 5, 5000, 4), ("cheb", 5, 6000, 5)])
def test_levels_and_bases(basis, p, n, L, prec, tol):
    kernel = {"harm": F.FMM_COULOMB3D, "points": F.FMM_COULOMB3D_POINTS,
              "cheb": F.FMM_COULOMB3D_CHEBYSHEV}[basis]
    pos, q = workloads.uniform(n, 3, seed=n + L)
    f = F.FMM(kernel, levels=L, order=p, precision=prec, max_particles=n, flags=F.FMM_SYNC_CHECK)
    dpos, dq = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    pot, _ = f.evaluate(dpos, dq)
    variants = [1, 2] if prec == F.FMM_FP64 else [1, 2, 4]
    for mb in variants:  # the same sums in the same order
        f.set_m2l_variant(mb)
        again, _ = f.evaluate(dpos, dq)
        assert torch.equal(again, pot)
    pot = pot.cpu().numpy()
    f.close()
    tg = workloads.sample_targets(n, 60)
    if basis == "harm":
        want, _ = oracle.fmm3d(pos, q, L, p, targets=tg)
    else:
        nodes = oracle.PAPER_NODES if basis == "points" else oracle.chebyshev_nodes(p)
        want, _ = oracle.fmm3d_lagrange_nodes(pos, q, L, nodes=nodes, targets=tg)
    assert rel(pot[tg], want) < tol
