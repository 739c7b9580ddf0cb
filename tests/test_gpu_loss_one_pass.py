"""The backward that writes both gradients in one pass (no mate_a, few blocks or
long rows) and the forward's walk over coordinates, at the edges of their blocks,
with unmatched rows and columns, against the oracle's closed form."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n,d", [(2, 63, 1), (3, 64, 1025), (1, 65, 7), (2, 1025, 2), (2, 1000, 1024),
                                       (1, 8192, 3), (1, 8193, 3)])
def test_edges_and_unmatched(batch, n, d):
    import paper_2203_03732_amd as prot
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n * 31 + d)
    X = rng.standard_normal((batch, n, d), dtype=np.float32)
    Y = rng.standard_normal((batch, n, d), dtype=np.float32)
    mates = np.stack([rng.permutation(n) for _ in range(batch)]).astype(np.int32)
    mates[:, rng.integers(0, n, 5)] = -1
    g = np.linspace(0.5, 2.0, batch).astype(np.float32)
    ctx = prot.context()
    args = [torch.from_numpy(a).cuda() for a in (X, Y, mates)]
    loss = ctx.ot_loss(*args).cpu().numpy()
    dX, dY = (t.cpu().numpy() for t in ctx.ot_loss_grad(*args, torch.from_numpy(g).cuda()))
    for i in range(batch):
        # a binary64 sum rounded to binary32 once
        np.testing.assert_allclose(loss[i], oracle.ot_loss(X[i], Y[i], mates[i]), rtol=2.0**-23)
        # binary32 2 g / n, difference and product: 4 units in the last place at most
        wX, wY = oracle.ot_loss_grad(X[i], Y[i], mates[i], float(g[i]))
        np.testing.assert_allclose(dX[i], wX, rtol=2.0**-21, atol=0)
        np.testing.assert_allclose(dY[i], wY, rtol=2.0**-21, atol=0)
        held = np.zeros(n, bool)
        held[mates[i][mates[i] >= 0]] = True
        assert not dX[i][mates[i] < 0].any() and not dY[i][~held].any()
