"""The FP64 2D contraction of few tiles (a workgroup per parity class, a quarter
of the offsets per wave): every order bucket at the smallest and largest trees
it takes, against the oracle (1e-12 relative L2, the bound of the other FP64
evaluations: only the order of 27 sums differs), the same bits for every tile
height, and the plan-free evaluation, whose operators are built on the device."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def rel(a, b):
    return float(np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b))


@pytest.mark.parametrize("p", [1, 8, 9, 12, 15, 16, 18, 20, 23, 24, 30])
@pytest.mark.parametrize("L,n", [(2, 501), (3, 2000), (6, 3001)])
def test_few_tiles(p, L, n):
    pos, q = workloads.uniform(n, 2, seed=10 * L + p)
    want, wfld = oracle.fmm2d(pos, q, L, p)
    dpos, dq = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    f = F.FMM(F.FMM_LOG2D, levels=L, order=p, max_particles=n, flags=F.FMM_SYNC_CHECK)
    out = []
    for mb in (1, 2, 3):
        try:
            f.set_m2l_variant(mb, 1)
        except F.FmmError:
            continue  # not compiled for this order
        out.append(f.evaluate(dpos, dq))
    f.close()
    for pot, fld in out:
        assert rel(pot, want) < 1e-12 and rel(fld, wfld) < 1e-12
        assert torch.equal(pot, out[0][0]) and torch.equal(fld, out[0][1])


@pytest.mark.parametrize("p", [1, 8, 11, 16, 17, 20])
@pytest.mark.parametrize("L,n,prec,tol", [(0, 70, F.FMM_FP64, 1e-12), (2, 501, F.FMM_FP64, 1e-12),
                                          (6, 3001, F.FMM_FP64, 1e-12),
                                          (5, 20011, F.FMM_FP32, 1e-6)])
def test_operators_built_on_the_device(p, L, n, prec, tol):
    pos, q = workloads.uniform(n, 2, seed=20 * L + p)
    want, wfld = oracle.fmm2d(pos, q, L, p)
    dpos, dq = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    pot = torch.empty_like(dq)
    fld = torch.empty_like(dpos)
    o = F.fmm_default_options(F.FMM_LOG2D)
    o.levels, o.order_p, o.precision, o.flags = L, p, prec, F.FMM_SYNC_CHECK
    F.fmm_eval_noalloc(o, n, dpos, dq, pot, fld)
    torch.cuda.synchronize()
    assert rel(pot, want) < tol  # FP32: the bar of the FP32 potentials
    assert prec == F.FMM_FP32 or rel(fld, wfld) < tol
