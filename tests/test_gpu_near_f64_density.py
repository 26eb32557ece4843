"""The FP64 near field of the 2D log kernel on both sides of the particle densities
between which it works in tiles (6 and 40 a leaf), and in sparse trees, against
the CPU oracle: 1e-12 relative L2, as for its other forms."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def rel(a, b):
    return float(np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,L", [(6 * 4 ** 7 - 1, 7), (6 * 4 ** 7, 7), (40 * 4 ** 7, 7),
                                 (40 * 4 ** 7 + 1, 7), (801, 7), (17001, 8), (65536, 8),
                                 (65537, 9)])
def test_densities(n, L):
    pos, q = workloads.uniform(n, 2, seed=n)
    f = F.FMM(F.FMM_LOG2D, levels=L, order=6, max_particles=n, flags=F.FMM_SYNC_CHECK)
    pot, fld = f.evaluate(torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda())
    targets = workloads.sample_targets(n, 500)
    want, wfld = oracle.fmm2d(pos, q, L, 6, targets=targets)
    assert rel(pot[targets], want) < 1e-12 and rel(fld[targets], wfld) < 1e-12
    f.close()
