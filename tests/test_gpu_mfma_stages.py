"""The matrix-core build around its staging depth (32 coordinates) and its list of
uncertain entries (1,792 a tile): rounded costs bit-exact with the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,eps", [
    (130, 31, 0.01), (130, 32, 0.0005), (257, 33, 0.002), (200, 64, 0.0004), (129, 65, 0.01),
    (256, 128, 0.0002)])  # the small eps leave most of a tile uncertain
def test_stages_and_lists(n, d, eps):
    import paper_2203_03732_amd as prot
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n * d)
    X, Y = (rng.standard_normal((n, d), dtype=np.float32) for _ in range(2))
    ctx = prot.Context(0)
    ctx.set_cost_path("matrix_cores")
    k, m = ctx.build_costs(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), eps)
    ref, m_ref = oracle.round_points_f32(X, Y, eps)
    assert float(m[0]) == m_ref
    assert np.array_equal(k.cpu().numpy()[:, :n], ref)
    ctx.close()
