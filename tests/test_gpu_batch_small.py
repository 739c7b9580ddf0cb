"""Batches of instances of at most 512 points, whose workgroups have 16, 8 or 4
waves by the number of instances: bit-exact with the oracle."""
import numpy as np
import pytest

from test_gpu_batch import check_instances, ctx, pack  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n_max,eps", [(12, 512, 0.01), (257, 512, 0.05), (257, 255, 0.02),
                                             (1024, 256, 0.1), (1023, 40, 0.03)])
def test_waves_by_batch(ctx, batch, n_max, eps):  # noqa: F811
    rng = np.random.default_rng(batch + n_max)
    ns = [int(n) for n in rng.integers(1, min(n_max, 64), batch)]
    ns[:6] = [n_max, n_max - 1, 1, 33, 7, 8]
    Xs = [rng.standard_normal((n, 3)).astype(np.float32) for n in ns]
    Ys = [(0.4 + rng.standard_normal((n, 3))).astype(np.float32) for n in ns]
    plan = ctx.batch(ns, 3, eps, config={"engine": "lds"})
    plan.run(pack(Xs), pack(Ys))
    out = (plan.mate_a, plan.mate_b, plan.y_a, plan.y_b)
    check_instances(ns, Xs, Ys, eps, out, plan.stats())
