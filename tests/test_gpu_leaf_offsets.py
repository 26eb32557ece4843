"""Leaf offsets of trees with more leaves than one workgroup of the offset
kernel takes and far more, or fewer, leaves than particles: bit-exact against
the sorted keys.  The adaptive depth flags at the edges of their levels, against
the oracle's adaptive evaluation (FP64, to the 1e-12 of the other adaptive
tests)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def positions(kind, n, dim):
    pos, _ = workloads.uniform(n, dim, seed=n)
    if kind == "first":
        return pos * 1e-4
    if kind == "last":
        return 5.0 - pos * 1e-4
    if kind == "ends":
        pos *= 1e-4
        pos[n // 2:] = 5.0 - pos[n // 2:]
    return pos


@pytest.mark.parametrize("dim,L", [(2, 9), (2, 10), (3, 6)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 4097, 100003])
@pytest.mark.parametrize("kind", ["uniform", "first", "last", "ends"])
def test_leaf_offsets(dim, L, n, kind):
    pos = positions(kind, n, dim)
    f = F.FMM(F.FMM_LOG2D if dim == 2 else F.FMM_COULOMB3D, levels=L, order=4, max_particles=n,
              precision=F.FMM_FP32, flags=F.FMM_SYNC_CHECK)
    f.evaluate(torch.from_numpy(pos).cuda(), torch.ones(n, dtype=torch.float64, device="cuda"))
    nleaf = 2 ** (dim * L)
    keys = np.frombuffer(F.fmm_debug_level_data(f.plan, 0, F.FMM_DBG_SORTED_KEYS, 4 * n), np.uint32)
    start = np.frombuffer(F.fmm_debug_level_data(f.plan, 0, F.FMM_DBG_LEAF_START, 4 * (nleaf + 1)),
                          np.int32)
    f.close()
    assert np.all(np.diff(keys.astype(np.int64)) >= 0) and keys[-1] < nleaf
    np.testing.assert_array_equal(start, np.searchsorted(keys, np.arange(nleaf + 1), "left"))


@pytest.mark.parametrize("n,L,near", [(5000, 2, 50), (5000, 3, 1), (5000, 3, 10 ** 6), (700, 9, 1),
                                      (700, 5, 699), (700, 5, 700)])
def test_adaptive_flag_levels(n, L, near):
    pos, q = workloads.gaussian_mixture(n, 2, seed=n + L, ncomp=4, sigma=0.08)
    want, wfld, _ = oracle.fmm2d_adaptive(pos, q, L, 12, near)
    f = F.FMM(F.FMM_LOG2D, levels=L, order=12, max_particles=n, flags=F.FMM_SYNC_CHECK,
              adaptive_near=near)
    pot, fld = f.evaluate(torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda())
    pot, fld = pot.cpu().numpy(), fld.cpu().numpy()
    f.close()
    assert np.linalg.norm(pot - want) < 1e-12 * np.linalg.norm(want)
    assert np.linalg.norm(fld - wfld) < 1e-12 * np.linalg.norm(wfld)
