"""The order network's gradient over batches of several tiles a workgroup: the
FP32 sums end with 16 samples, whatever the batch.

The first and the last 4096 samples are the same inputs with errors of 2^26 and
-2^26, the ones between have errors of order one: the large terms cancel, and
what is left is lost by any FP32 sum that runs on from one group of 16 samples
to another (2^27 * 16 has an ulp of 256).  All weights and inputs are small whole
numbers and the outputs multiples of 8, so the forward pass and the errors are
exact in FP32, and the large terms are exact negatives of each other.  Tolerance
1e-4, as for the network's other gradients."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")

SPLITS = {"W1": 0, "b1": 192, "W2": 256, "b2": 4352, "W3": 4416, "b3": 5760, "end": 5781}


@pytest.mark.parametrize("m", [3 * 4096, 3 * 4096 + 48, 25 * 4096])
def test_small_terms_survive_cancelling_ones(m):
    rng = np.random.default_rng(m)
    w = np.concatenate([rng.integers(-1, 2, 192), rng.integers(0, 2, 64),
                        rng.integers(-1, 2, 4096) * (rng.random(4096) < 0.2),
                        rng.integers(0, 2, 64), 8 * rng.integers(-1, 2, 1344),
                        np.zeros(21)]).astype(np.float64)
    x = rng.integers(-2, 3, (m, 3)).astype(np.float64)
    x[-4096:] = x[:4096]
    e = rng.integers(1, 4, (m, 21)).astype(np.float64)
    e[:4096] = 2.0 ** 26
    e[-4096:] = -(2.0 ** 26)
    t = oracle.mlp_forward(w, x) - e
    assert np.array_equal(np.float64(np.float32(t)), t)
    _, want = oracle.mlp_loss_grad(w, x, t)
    dw, dx, dt = (torch.from_numpy(np.float32(v)).cuda() for v in (w, x, t))
    g = torch.empty_like(dw)
    loss = torch.empty(1, device="cuda")
    F.fmm_mlp_loss_grad(dw, dx, dt, g, loss)
    got = g.cpu().numpy().astype(np.float64)
    names = list(SPLITS)
    for a, b in zip(names[:-1], names[1:]):
        s = slice(SPLITS[a], SPLITS[b])
        assert np.linalg.norm(got[s] - want[s]) < 1e-4 * np.linalg.norm(want[s]), a
