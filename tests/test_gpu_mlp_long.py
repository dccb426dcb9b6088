"""The network on long batches through narrow layers, whose forward pass takes one wave a
tile, at the edges of its tiles of 16 and 32 and of the k-range and widths that it is
taken for; tolerances as for the other sizes (test_gpu_learned.py)."""
import time

import numpy as np
import pytest

from oracle import learned as L
from test_gpu_learned import dev, seeded_net

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("widths,batch", [
    ([4, 4, 4], 65521), ([1, 16, 1], 65537),     # tiles of 16, the first batch that has enough
    ([128, 33, 32, 17], 32769), ([129, 32, 31], 65536), ([15, 130, 16, 5], 70001),
    ([129, 33, 128, 40], 22000)])                # eight waves and one in turn
def test_long_batches(widths, batch):
    import paper_1707_03771_amd as dfx
    rng = np.random.default_rng(5)
    th = seeded_net(widths, 6)
    X = rng.normal(size=(batch, widths[0])).astype(np.float32)
    T = rng.normal(size=(batch, widths[-1])).astype(np.float32)
    Y = dfx.mlp_forward(widths, dev(th), dev(X)).cpu().numpy()
    Yo, _ = L.forward(th.astype(np.float64), widths, X.astype(np.float64))
    assert np.linalg.norm(Y - Yo) <= 1e-5 * np.linalg.norm(Yo)
    loss, g = dfx.mlp_loss_grad(widths, dev(th), dev(X), dev(T))
    lo, go = L.loss_and_grad(th.astype(np.float64), widths, X.astype(np.float64), T.astype(np.float64))
    assert abs(loss - lo) <= 1e-5 * lo
    assert np.linalg.norm(g.cpu().numpy() - go) <= 1e-4 * np.linalg.norm(go)


def test_a_long_batch_is_no_dearer_a_row():
    """Five times the rows of a batch that is still mostly launches take less than 2.6 times
    as long (3.5 with eight waves a tile, 1.9 with one)."""
    import paper_1707_03771_amd as dfx
    w, best = [4, 4, 4], {}
    th = dev(seeded_net(w, 6))
    for batch in (20000, 100000):
        X = torch.randn(batch, 4, device="cuda")
        for _ in range(25):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            dfx.mlp_forward(w, th, X)
            best[batch] = min(best.get(batch, 1.0), time.perf_counter() - t0)
    print(f"{best[20000] * 1e6:.1f} and {best[100000] * 1e6:.1f} us")
    assert best[100000] <= 2.6 * best[20000]
