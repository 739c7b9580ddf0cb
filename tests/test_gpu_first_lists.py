"""Lists made before the solve (batches of at most 256 instances, single
instances by one workgroup; more than three dimensions or a cost matrix): rows
with more columns at one cost than a list holds, list and layout edges, bytes.
Bit-exact with the oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_batch import STAT_KEYS, ctx, pack  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("law", ["normal", "equal", "clusters"])
@pytest.mark.parametrize("ns", [[1, 2, 8, 31, 33, 65, 511, 512], [513, 1024, 9], [1025, 2048, 7]])
def test_batches(ctx, ns, law):  # noqa: F811
    rng = np.random.default_rng(len(ns))
    Xs, Ys = [], []
    for n in ns:
        x, y = (rng.standard_normal((n, 5)).astype(np.float32) for _ in range(2))
        if law == "equal":
            x[:], y[:] = 0.0, 1.0
        if law == "clusters":
            x, y = (np.where(rng.random((n, 1)) < 0.3, 4.0, 0.0) + 0 * v for v in (x, y))
        Xs.append(x.astype(np.float32))
        Ys.append(y.astype(np.float32))
    plan = ctx.batch(ns, 5, 0.03, config={"engine": "lds"})
    plan.run(pack(Xs), pack(Ys))
    stats, off = plan.stats(), np.concatenate([[0], np.cumsum(ns)])
    for i, n in enumerate(ns):
        k, m = oracle.round_points_f32(Xs[i], Ys[i], 0.03)
        ref = oracle.solve_rounded(k, oracle.threshold(0.03, n))
        for name in ("mate_a", "mate_b", "y_a", "y_b"):
            got = getattr(plan, name)[off[i]:off[i + 1]].cpu().numpy()
            assert np.array_equal(got, ref[name]), (n, name)
        for s in STAT_KEYS:
            assert stats[i][s] == ref["stats"][s], (n, s)
        assert stats[i]["cost_scale"] == m


@pytest.mark.parametrize("k_type", ["int16", "uint8"])
@pytest.mark.parametrize("n_b,n_a,cells", [(1, 2, 1), (60, 120, 2), (60, 121, 2), (150, 300, 40),
                                           (200, 200, 1), (399, 401, 9)])
def test_cost_matrices(ctx, n_b, n_a, cells, k_type):  # noqa: F811
    """cells: how many different costs there are."""
    rng = np.random.default_rng(n_a)
    C = (rng.integers(0, cells, (n_b, n_a)) / 50.0).astype(np.float32)
    res = ctx.solve_cost(torch.from_numpy(C).cuda(), 0.02, k_type=k_type)
    ref = oracle.solve_rounded(oracle.round_cost(C, 0.02), oracle.threshold(0.02, n_b))
    for name in ("mate_a", "mate_b", "y_a", "y_b"):
        assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), name
    for s in ("phases", "rounds", "max_rounds", "scanned", "sum_free", "sum_k"):
        assert res.stats[s] == ref["stats"][s], s
