"""Small FP64 2D evaluations, whose near field and moments share a launch, at the
edges of its forms (16 and 4 lanes a target, the largest particle count, sliced
boxes, every order bucket, per-level orders): against the oracle (1e-12 relative
L2, the bound of the FP64 evaluations) and bit for bit against the same
evaluation with its phases timed, which runs them apart on two streams."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def rel(a, b):
    return float(np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,L,p,kind", [
    (1, 2, 8, "uniform"), (2, 3, 1, "uniform"), (501, 2, 12, "uniform"), (4096, 4, 12, "uniform"),
    (16384, 5, 16, "uniform"), (16385, 5, 20, "mixture"), (16384, 2, 5, "mixture"),
    (20011, 7, 24, "mixture"), (5000, 4, 30, "uniform"), (65536, 6, 16, "uniform"),
    (65537, 6, 8, "uniform")])
def test_one_launch(n, L, p, kind):
    pos, q = (workloads.uniform if kind == "uniform" else workloads.gaussian_mixture)(n, 2,
                                                                                      seed=n + p)
    want, wfld = oracle.fmm2d(pos, q, L, p)
    dpos, dq = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    out = []
    for flags in (0, F.FMM_TIMING):
        f = F.FMM(F.FMM_LOG2D, levels=L, order=p, max_particles=n, flags=F.FMM_SYNC_CHECK | flags)
        for _ in range(2):
            pot, fld = f.evaluate(dpos, dq)
        torch.cuda.synchronize()
        out.append((pot, fld))
        f.close()
    if n > 1:
        assert rel(out[0][0], want) < 1e-12 and rel(out[0][1], wfld) < 1e-12
    else:
        assert abs(float(out[0][0][0]) - want[0]) < 1e-12
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
