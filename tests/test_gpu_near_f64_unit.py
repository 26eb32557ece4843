"""The FP64 near field of the 2D log kernel for pairs about one unit apart, where
log r^2 vanishes, and for infinite charges, in every form of the kernel (sixteen,
four and one lane a target, tiles, the plan-free evaluation).

Every charge is zero but one, so a target's potential is one pair's term.  The
distances are exact in FP64 and so is r^2; relative tolerance 8 * 2^-53: the
logarithm's factors and its last sum (at most five roundings), times the charge,
1, and (ln 2) / 2, itself rounded, with a rounding each."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")

# n, levels, side: 16, 4 and 1 lanes a target; tiles (level 7); plan-free (level 1)
FORMS = [(300, 1, 8.0, False), (20000, 1, 8.0, False), (66000, 1, 8.0, False),
         (300000, 7, 256.0, False), (300, 1, 8.0, True)]


def potentials(n, L, side, noalloc, centre, offsets, charge):
    """Potentials at centre + offset, for a charge at the centre."""
    rng = np.random.default_rng(n)
    pos = rng.uniform(0.0, side, (n, 2))
    q = np.zeros(n)
    pos[0] = centre
    q[0] = charge
    pos[1:1 + len(offsets)] = np.asarray(centre) + offsets
    dpos, dq = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    if noalloc:
        o = F.fmm_default_options(F.FMM_LOG2D)
        o.levels, o.order_p, o.side, o.flags = L, 4, side, F.FMM_SYNC_CHECK
        pot, fld = torch.empty_like(dq), torch.empty_like(dpos)
        F.fmm_eval_noalloc(o, n, dpos, dq, pot, fld)
    else:
        f = F.FMM(F.FMM_LOG2D, levels=L, order=4, max_particles=n, side=side,
                  flags=F.FMM_SYNC_CHECK)
        pot, fld = f.evaluate(dpos, dq)
        f.close()
    torch.cuda.synchronize()
    return pot.cpu().numpy()[1:1 + len(offsets)]


@pytest.mark.parametrize("n,L,side,noalloc", FORMS)
def test_unit_distance(n, L, side, noalloc):
    off, want = [(1.0, 0.0)], [0.0]
    for k in (2, 4, 7, 10, 13, 20, 26):
        off.append((1.0, 2.0 ** -k))  # r^2 = 1 + 2^-2k
        want.append(0.5 * math.log1p(2.0 ** (-2 * k)))
        for s in (1.0, -1.0):
            off.append((0.0, 1.0 + s * 2.0 ** -k))
            want.append(math.log1p(s * 2.0 ** -k))
    c = 0.5 * side + 0.25
    pot = potentials(n, L, side, noalloc, (c, c), np.array(off), 1.0)
    assert pot[0] == 0.0
    np.testing.assert_allclose(pot, want, rtol=8 * 2.0 ** -53, atol=0.0)


@pytest.mark.parametrize("charge", [np.inf, -np.inf])
@pytest.mark.parametrize("n,L,side,noalloc", FORMS)
def test_infinite_charge(n, L, side, noalloc, charge):
    r = np.array([0.25, 0.6, 0.8, 0.9, 1.1, 1.3, 1.75])
    c = 0.5 * side + 0.25
    pot = potentials(n, L, side, noalloc, (c, c), np.stack([r, 0.0 * r], axis=1), charge)
    np.testing.assert_array_equal(pot, np.where(r < 1.0, -charge, charge))


# Leaves too small for unit distances (side 11/32) take the shorter logarithm.
@pytest.mark.parametrize("charge", [np.inf, -np.inf])
@pytest.mark.parametrize("n,L,side,noalloc", [(300, 1, 0.6875, False), (20000, 1, 0.6875, False),
                                              (66000, 1, 0.6875, False),
                                              (300000, 7, 44.0, False), (300, 1, 0.6875, True)])
def test_infinite_charge_small_leaves(n, L, side, noalloc, charge):
    off = np.array([(0.02, 0.3), (0.3, 0.3), (0.5, 0.5), (0.6, 0.4), (0.6, 0.6), (0.62, 0.62)])
    c = (0.5 * side if L > 1 else 0.0) + 0.02  # just inside a leaf's lower corner
    pot = potentials(n, L, side, noalloc, (c, c), off, charge)
    np.testing.assert_array_equal(pot, np.full(len(off), -charge))
