"""The samples that pad the last group of 16 of a batch take no part in the
gradient, also where a padding sample's hidden layer would overflow."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


@pytest.mark.parametrize("m", [1, 15, 17])
def test_padding_does_not_overflow_into_the_gradient(m):
    rng = np.random.default_rng(m)
    w = np.float32(rng.normal(0.0, 0.3, F.FMM_MLP_NPARAM))
    x = np.float32(rng.normal(size=(m, 3)))
    t = np.float32(rng.normal(size=(m, 21)))
    x[:, 0] = 1.0  # hidden unit 0: 1e20 - 1e20 x_0 = 0 for these samples, 1e20 for a zero input
    w[0:3] = (-1e20, 0.0, 0.0)
    w[192] = 1e20
    w[256:256 + 4096:64] = 1e20  # its weights in the second layer
    g = torch.empty(F.FMM_MLP_NPARAM, device="cuda")
    loss = torch.empty(1, device="cuda")
    F.fmm_mlp_loss_grad(*(torch.from_numpy(v).cuda() for v in (w, x, t)), g, loss)
    _, want = oracle.mlp_loss_grad(np.float64(w), np.float64(x), np.float64(t))
    assert np.linalg.norm(g.cpu().numpy() - want) < 1e-4 * np.linalg.norm(want)
