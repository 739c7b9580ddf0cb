"""Batches whose rows find their column among the first they look at (large eps,
few dimensions): 16 rows of a wave looked at together, 32 columns each. Every
instance bit-exact with the CPU oracle at the sizes where the groups of rows and
the windows end, in every kernel width, and on both sides of the choice between
one workgroup and teams."""
import numpy as np
import pytest

from test_gpu_batch import check_instances, ctx, pack  # noqa: F401

pytestmark = pytest.mark.gpu


def sets(ns, d, law, seed):
    rng = np.random.default_rng(seed)
    draw = {"uniform": lambda n: rng.random((n, d)),
            "normal": lambda n: rng.standard_normal((n, d)),
            # half the rows far from most columns: hits and misses in every group
            "mixed": lambda n: rng.random((n, d)) + 3.0 * (np.arange(n)[:, None] % 2 == 0)}[law]
    Xs = [draw(n).astype(np.float32) for n in ns]
    Ys = [(draw(n) + 0.2).astype(np.float32) for n in ns]
    return Xs, Ys


@pytest.mark.parametrize("origin", ["diag", "zero"])
@pytest.mark.parametrize("d,eps,law", [(2, 0.2, "normal"), (2, 0.05, "uniform"), (3, 0.1, "mixed"),
                                       (5, 0.25, "normal")])
def test_groups_and_windows(ctx, d, eps, law, origin):  # noqa: F811
    for ns in ([1, 3, 7, 8, 33, 63, 64, 65], [66, 127, 128, 129, 191, 255, 257, 511, 512],
               [513, 521, 777, 1023, 1024], [1025, 1301, 2047, 2048, 40]):
        Xs, Ys = sets(ns, d, law, ns[0])
        plan = ctx.batch(ns, d, eps, origin=origin, config={"engine": "lds"})
        plan.run(pack(Xs), pack(Ys))
        check_instances(ns, Xs, Ys, eps, (plan.mate_a, plan.mate_b, plan.y_a, plan.y_b),
                        plan.stats(), origin)
        plan.close()


@pytest.mark.parametrize("batch,n_max", [(300, 100), (300, 300), (300, 600), (1100, 200)])
def test_widths(ctx, batch, n_max):  # noqa: F811
    rng = np.random.default_rng(batch + n_max)
    ns = [int(x) for x in rng.integers(2, n_max + 1, batch - 1)] + [n_max]
    Xs, Ys = sets(ns, 2, "normal", n_max)
    plan = ctx.batch(ns, 2, 0.15)
    plan.run(pack(Xs), pack(Ys))
    check_instances(ns, Xs, Ys, 0.15, (plan.mate_a, plan.mate_b, plan.y_a, plan.y_b), plan.stats(),
                    which=list(range(0, batch, 7)) + [batch - 1])
    plan.close()


@pytest.mark.parametrize("batch,n,d,eps", [
    (3, 1100, 2, 0.02), (3, 1100, 2, 0.04), (2, 1600, 3, 0.05), (2, 1600, 3, 0.14),
    (34, 1100, 5, 0.1), (50, 1100, 2, 0.1), (66, 1040, 6, 0.1)])
def test_teams_or_one(ctx, batch, n, d, eps):  # noqa: F811
    """Either side of the automatic choice above 1,024 points."""
    ns = [n] * batch
    Xs, Ys = sets(ns, d, "uniform", n)
    plan = ctx.batch(ns, d, eps)
    plan.run(pack(Xs), pack(Ys))
    check_instances(ns, Xs, Ys, eps, (plan.mate_a, plan.mate_b, plan.y_a, plan.y_b), plan.stats(),
                    which=[0, batch - 1])
    plan.close()
