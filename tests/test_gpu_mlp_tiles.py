"""The order network's batches at the edges of their tiles of 16 samples and of
the 256 workgroups of a gradient, and two gradients at once from two threads,
against the FP64 oracle.  Tolerances as for the network's other tests: FP32 sums
of at most 64 terms a product give 1e-5 on outputs, 1e-4 on the gradient."""
import threading

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
F = pytest.importorskip("paper_2009_00767_amd")


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b))


def data(m):
    rng = np.random.default_rng(m)
    return [np.float32(v) for v in (rng.normal(0.0, 0.3, F.FMM_MLP_NPARAM), rng.normal(size=(m, 3)),
                                    rng.normal(size=(m, 21)))]


def gradient(w, x, t, out):
    g = torch.empty_like(w)
    loss = torch.empty(1, device="cuda")
    F.fmm_mlp_loss_grad(w, x, t, g, loss, stream=torch.cuda.Stream())
    out.append((g.cpu().numpy(), float(loss.item())))


@pytest.mark.parametrize("m", [15, 16, 33, 4096, 4097, 9001])
def test_tiles(m):
    w, x, t = data(m)
    dw, dx, dt = (torch.from_numpy(v).cuda() for v in (w, x, t))
    y = torch.empty((m, 21), device="cuda")
    F.fmm_mlp_forward(dw, dx, y)
    assert rel(y.cpu().numpy(), oracle.mlp_forward(np.float64(w), np.float64(x))) < 1e-5
    torch.cuda.synchronize()
    out = []
    gradient(dw, dx, dt, out)
    wl, wg = oracle.mlp_loss_grad(np.float64(w), np.float64(x), np.float64(t))
    assert rel(out[0][0], wg) < 1e-4 and abs(out[0][1] - wl) < 1e-5 * wl


def test_gradients_of_two_threads():
    sets = [[torch.from_numpy(v).cuda() for v in data(m)] for m in (700, 5000)]
    torch.cuda.synchronize()
    want = [[], []]
    for s, o in zip(sets, want):
        gradient(*s, o)
    got = [[], []]
    threads = [threading.Thread(target=lambda s=s, o=o: [gradient(*s, o) for _ in range(20)])
               for s, o in zip(sets, got)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for o, w in zip(got, want):
        assert len(o) == 20
        for g, loss in o:
            np.testing.assert_array_equal(g, w[0][0])
            assert loss == w[0][1]
