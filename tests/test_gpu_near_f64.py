"""The FP64 near field of the 2D log kernel (tile form, direct form with one,
four and sixteen lanes a target) against the CPU oracle.

Tolerance: 1e-12 relative L2, the FP64 mode's: both sides sum the same FP64
terms in another order, and a term's own error is a few units in 1e-16.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / max(np.linalg.norm(b), 1e-300))


def evaluate(pos, q, L, p, **kw):
    f = F.FMM(F.FMM_LOG2D, levels=L, order=p, max_particles=max(len(q), 1),
              flags=F.FMM_SYNC_CHECK, **kw)
    pot, fld = f.evaluate(torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda())
    torch.cuda.synchronize()
    out = pot.cpu().numpy(), fld.cpu().numpy()
    f.close()
    return out


# Up to 16384 targets: sixteen lanes each; up to 65536: four; beyond, one lane,
# and from 1024 tiles (level 7) the tile form, whose stage a clustered halo
# exceeds (those targets go to the direct form).  Empty leaves, leaves of 1..5
# particles and the remainders of the batches of four are in all of them.
@pytest.mark.parametrize("kind,n,L", [("uniform", 1, 2), ("uniform", 5, 2), ("uniform", 63, 1),
                                      ("uniform", 1021, 3), ("mixture", 4099, 4),
                                      ("uniform", 16384, 5), ("uniform", 16385, 5),
                                      ("mixture", 20011, 5), ("uniform", 65537, 6),
                                      ("mixture", 66001, 4), ("uniform", 40009, 7),
                                      ("uniform", 300007, 7), ("mixture", 150001, 7),
                                      ("mixture", 30011, 8)])
def test_near_field_forms(kind, n, L):
    pos, q = (workloads.uniform if kind == "uniform" else workloads.gaussian_mixture)(n, 2, seed=n)
    pot, fld = evaluate(pos, q, L, 6)
    targets = workloads.sample_targets(n, 1500)
    want, wfld = oracle.fmm2d(pos, q, L, 6, targets=targets)
    assert rel(pot[targets], want) < 1e-12
    assert rel(fld[targets], wfld) < 1e-12


# r = 0 counts nothing; r^2 near the end of the FP64 range (pairs astride the
# coordinates' zero, and a box of side 1e130) takes the library's functions.
@pytest.mark.parametrize("n", [300, 20000])
def test_near_field_extreme_distances(n):
    pos, q = workloads.uniform(n, 2, seed=3)
    pos -= 2.5
    pos[1::40] = pos[::40][:len(pos[1::40])]  # coincident pairs
    for i, d in enumerate((1e-60, 1e-130, 1e-140, 1e-146)):
        pos[2 + 4 * i] = (-d, d)
        pos[3 + 4 * i] = (d, 0.0)
    keep = np.arange(18, 118, 4)
    pot, fld = evaluate(pos, q, 0, 4, origin=(-2.5, -2.5))
    for t in (np.arange(2, 18), keep):
        want, wfld = oracle.direct(pos, q, targets=t)
        np.testing.assert_allclose(pot[t], want, rtol=1e-11, atol=1e-11 * np.abs(want).max())
        np.testing.assert_allclose(fld[t], wfld, rtol=1e-11,
                                   atol=1e-11 * np.abs(wfld[np.isfinite(wfld)]).min())


def test_near_field_of_a_huge_box():
    pos, q = workloads.uniform(500, 2, seed=4)
    pot, fld = evaluate(pos * 2e129, q, 1, 4, side=1e130)
    want, wfld = oracle.direct(pos * 2e129, q)
    assert rel(pot, want) < 1e-12
    assert rel(fld * 1e129, wfld * 1e129) < 1e-12
