"""The two-digit particle sort where buckets outgrow their LDS stage: one, two or
several dense boxes holding all or most particles, at the edges of the stages (1280
and 5120 elements) and of the parts (2048 and 8192): permutation, keys and leaf
offsets bit-exact, the permutation being the stable argsort of the leaf keys, and the
charges of the level-2 boxes (sums in FP64 of at most n terms below 1, each rounding
at most n 2^-53: the sorted records and coordinates that the sort writes beside)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def morton(c):
    key = np.zeros(len(c), np.int64)
    for b in range(9):
        for d in range(c.shape[1]):
            key |= ((c[:, d] >> b) & 1) << (b * c.shape[1] + d)
    return key


def particles(n, dim, dense, seed):
    """`dense` boxes of a 16^dim (2D) or 4^dim (3D) grid share 90 % of the particles."""
    rng = np.random.default_rng(seed)
    cells = 16 if dim == 2 else 4
    pos = 5.0 * rng.random((n, dim))
    inside = rng.random(n) < (0.9 if dense > 1 else 1.0)
    box = rng.integers(0, cells, (dense, dim))[rng.integers(0, dense, n)]
    pos[inside] = ((box + rng.random((n, dim))) * (5.0 / cells))[inside]
    return np.minimum(pos, np.nextafter(5.0, 0.0)), rng.uniform(-1.0, 1.0, n)


@pytest.mark.parametrize("dim,n,L,dense", [
    (2, 1280, 7, 1), (2, 1281, 7, 1), (2, 2049, 8, 1), (2, 4097, 5, 1), (2, 6145, 8, 2),
    (2, 30011, 5, 1), (2, 100003, 7, 3), (2, 294912, 8, 2), (2, 294913, 7, 1), (2, 300007, 8, 5),
    (2, 400000, 6, 40), (3, 9001, 3, 1), (3, 200003, 4, 7), (3, 300001, 5, 2)])
@pytest.mark.parametrize("prec", [F.FMM_FP64, F.FMM_FP32])
def test_dense_buckets(dim, n, L, dense, prec):
    pos, q = particles(n, dim, dense, seed=n + L)
    f = F.FMM(F.FMM_LOG2D if dim == 2 else F.FMM_COULOMB3D, levels=L, order=2, precision=prec,
              max_particles=n, flags=F.FMM_SYNC_CHECK)
    f.evaluate(torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda())
    nleaf = 2 ** (dim * L)
    perm = np.frombuffer(F.fmm_debug_level_data(f.plan, 0, F.FMM_DBG_PERM, 4 * n), np.int32)
    keys = np.frombuffer(F.fmm_debug_level_data(f.plan, 0, F.FMM_DBG_SORTED_KEYS, 4 * n), np.uint32)
    start = np.frombuffer(F.fmm_debug_level_data(f.plan, 0, F.FMM_DBG_LEAF_START, 4 * (nleaf + 1)),
                          np.int32)
    # the moments of level 2 come from the sorted records or coordinates
    cs = F.fmm_coef_stride(f.plan)
    mom = np.frombuffer(F.fmm_debug_level_data(f.plan, 2, F.FMM_DBG_MOMENTS, 8 * 4 ** 2 * cs
                                               if dim == 2 else 8 * 8 ** 2 * cs), np.float64)
    pb = F.fmm_coef_order(f.plan)
    f.close()
    k = morton(np.minimum(np.floor(pos * (2 ** L / 5.0)).astype(np.int64), 2 ** L - 1))
    want = np.argsort(k, kind="stable")
    np.testing.assert_array_equal(perm, want)
    np.testing.assert_array_equal(keys.astype(np.int64), k[want])
    np.testing.assert_array_equal(start, np.searchsorted(k[want], np.arange(nleaf + 1), "left"))
    col = 2 * pb if dim == 2 else (pb + 1) ** 2 - 1
    box = np.zeros(2 ** (2 * dim))
    np.add.at(box, k >> (dim * (L - 2)), np.float32(q) if prec else q)
    np.testing.assert_allclose(mom.reshape(-1, cs)[:, col], box, rtol=0.0, atol=n * n * 2.0 ** -53)
