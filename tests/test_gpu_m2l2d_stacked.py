"""The FP64 2D contraction on both sides of its form for few tiles: systems of one
depth stacked to just below, exactly at and above 128 tiles (a system of depth 2, 3,
4, 5 has 1, 2, 6, 22 tiles on its levels), against the oracle system by system
(1e-12 relative L2, the FP64 bar); above the line every tile height that is compiled
gives the same bits; and the autotuner, which has nothing to choose below it."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# 127, 128, 129 (depth 2); 128, 130 (3); 126, 132 (4); 110, 132 (5); two depths at once
@pytest.mark.parametrize("depths", [{2: 127}, {2: 128}, {2: 129}, {3: 64}, {3: 65}, {4: 21},
                                    {4: 22}, {5: 5}, {5: 6}, {3: 64, 4: 22}])
@pytest.mark.parametrize("p", [7, 16])
def test_stacked_tiles(depths, p):
    levels = np.concatenate([np.full(c, d, np.int32) for d, c in depths.items()])
    levels = np.random.default_rng(len(levels)).permutation(levels)
    systems = [workloads.uniform(40 * int(d) + i % 7, 2, seed=31 * i + int(d))
               for i, d in enumerate(levels)]
    off = np.concatenate([[0], np.cumsum([len(q) for _, q in systems])]).astype(np.int64)
    pos = torch.from_numpy(np.concatenate([x for x, _ in systems])).cuda()
    q = torch.from_numpy(np.concatenate([x for _, x in systems])).cuda()
    f = F.FMM(F.FMM_LOG2D, levels=int(levels.max()), order=p, max_particles=len(q),
              flags=F.FMM_SYNC_CHECK, max_systems=len(levels), max_levels=int(levels.max()))
    out = []
    for mb in (1, 2, 3):
        try:
            f.set_m2l_variant(mb, 1)
        except F.FmmError:
            continue  # not compiled for this order
        pot, fld = f.evaluate_batched(off, pos, q, sys_levels=levels)
        torch.cuda.synchronize()
        out.append((pot.cpu().numpy(), fld.cpu().numpy()))
    f.close()
    assert len(out) >= 2
    for o in out[1:]:
        np.testing.assert_array_equal(o[0], out[0][0])
        np.testing.assert_array_equal(o[1], out[0][1])
    for i in range(0, len(systems), 7):
        a, b = off[i], off[i + 1]
        want, wfld = oracle.fmm2d(*systems[i], int(levels[i]), p)
        assert rel(out[0][0][a:b], want) < 1e-12 and rel(out[0][1][a:b], wfld) < 1e-12, i


def test_autotuner_has_one_height_for_few_tiles():
    for L in (3, 4, 5, 6):
        for p in (8, 12, 16, 20, 24):
            f = F.FMM(F.FMM_LOG2D, levels=L, order=p, max_particles=1000, flags=F.FMM_AUTOTUNE)
            st = f.stats()
            f.close()
            assert st.m2l_tile_mb == 1 and st.m2l_tuned_ms > 0, (L, p, st.m2l_tile_mb)
