"""The forms of the particle sort (one workgroup; two digits with four or
sixteen waves a bucket; full radix passes) at the edges of their ranges:
permutation, keys and leaf offsets bit-exact, the permutation being the stable
argsort of the leaf Morton keys."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def morton(c):
    key = np.zeros(len(c), np.int64)
    for b in range(13):
        for d in range(c.shape[1]):
            key |= ((c[:, d] >> b) & 1) << (b * c.shape[1] + d)
    return key


@pytest.mark.parametrize("dim,n,L,kind", [
    (2, 1, 0, "uniform"), (2, 2049, 0, "uniform"), (2, 63, 2, "uniform"), (2, 2048, 4, "uniform"),
    (2, 2049, 5, "mixture"), (2, 4096, 6, "uniform"), (2, 4097, 6, "mixture"),
    (2, 8191, 1, "uniform"), (2, 8192, 6, "mixture"), (2, 8193, 6, "uniform"),
    (2, 8000, 7, "uniform"), (2, 8193, 4, "uniform"), (2, 20011, 5, "mixture"),
    (2, 294912, 8, "mixture"), (2, 294913, 6, "uniform"), (2, 1179648, 7, "mixture"),
    (2, 1179649, 7, "uniform"), (3, 70, 1, "uniform"), (3, 5000, 4, "mixture"),
    (3, 8192, 3, "uniform"), (3, 8193, 3, "uniform"), (3, 300007, 5, "uniform")])
@pytest.mark.parametrize("prec", [F.FMM_FP64, F.FMM_FP32])
def test_sort_forms(dim, n, L, kind, prec):
    pos, q = (workloads.uniform if kind == "uniform" else workloads.gaussian_mixture)(n, dim,
                                                                                      seed=n)
    f = F.FMM(F.FMM_LOG2D if dim == 2 else F.FMM_COULOMB3D, levels=L, order=4, precision=prec,
              max_particles=n, flags=F.FMM_SYNC_CHECK)
    f.evaluate(torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda())
    nleaf = 2 ** (dim * L)
    perm = np.frombuffer(F.fmm_debug_level_data(f.plan, 0, F.FMM_DBG_PERM, 4 * n), np.int32)
    keys = np.frombuffer(F.fmm_debug_level_data(f.plan, 0, F.FMM_DBG_SORTED_KEYS, 4 * n), np.uint32)
    start = np.frombuffer(F.fmm_debug_level_data(f.plan, 0, F.FMM_DBG_LEAF_START, 4 * (nleaf + 1)),
                          np.int32)
    f.close()
    k = morton(np.minimum(np.floor(pos * (2 ** L / 5.0)).astype(np.int64), 2 ** L - 1))
    want = np.argsort(k, kind="stable")
    np.testing.assert_array_equal(perm, want)
    np.testing.assert_array_equal(keys.astype(np.int64), k[want])
    np.testing.assert_array_equal(start, np.searchsorted(k[want], np.arange(nleaf + 1), "left"))


def test_one_workgroup_reports_positions_outside():
    pos, q = workloads.uniform(3000, 2, seed=1)
    for bad in (np.nan, 5.1, -0.1):
        p = pos.copy()
        p[1234, 1] = bad
        f = F.FMM(F.FMM_LOG2D, levels=4, order=4, max_particles=3000, flags=F.FMM_SYNC_CHECK)
        with pytest.raises(F.FmmError) as e:
            f.evaluate(torch.from_numpy(p).cuda(), torch.from_numpy(q).cuda())
        assert e.value.status == F.FMM_ERR_DOMAIN
        f.close()
