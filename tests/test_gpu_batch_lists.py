"""The one-workgroup batch engine with per-row candidate lists: every instance
bit-exact with the CPU oracle (matching, duals, statistics) at the sizes where
its tiles, lists and packed 16-bit sums can go wrong."""
import numpy as np
import pytest

import oracle

from test_gpu_batch import check_instances, ctx, pack  # noqa: F401

pytestmark = pytest.mark.gpu

LDS = {"engine": "lds"}


def run(ctx, ns, Xs, Ys, eps, **kw):  # noqa: F811
    plan = ctx.batch(ns, Xs[0].shape[1], eps, config=LDS, **kw)
    plan.run(pack(Xs), pack(Ys))
    return (plan.mate_a, plan.mate_b, plan.y_a, plan.y_b), plan.stats()


@pytest.mark.parametrize("origin", ["diag", "zero"])
@pytest.mark.parametrize("d,eps", [(1, 0.05), (2, 0.01), (24, 0.02)])
def test_tile_and_list_edges(ctx, d, eps, origin):  # noqa: F811
    """Row lengths around the 8-column chunks, the 32-entry lists, the
    512-column tiles and the LDS layouts (n_max <= 1024 and above). d = 1
    gives rows with far more admissible columns than a list holds, d = 24
    rows whose lists run out many times."""
    rng = np.random.default_rng(d)
    for ns in ([1, 2, 7, 8, 9, 31, 32, 33, 63, 64, 65, 511, 512, 513, 1023, 1024],
               [1025, 1536, 1537, 2047, 2048, 5]):
        Xs = [rng.standard_normal((n, d)).astype(np.float32) for n in ns]
        Ys = [(0.3 + rng.standard_normal((n, d))).astype(np.float32) for n in ns]
        out, stats = run(ctx, ns, Xs, Ys, eps, origin=origin)
        check_instances(ns, Xs, Ys, eps, out, stats, origin)


@pytest.mark.parametrize("law", ["equal", "clusters", "line"])
def test_degenerate_points(ctx, law):  # noqa: F811
    """Equal points (one cost, every column admissible at once), two tight
    clusters (two costs) and points on a line (long convoys)."""
    rng = np.random.default_rng(7)
    ns = [40, 300, 1100]
    Xs, Ys = [], []
    for n in ns:
        if law == "equal":
            x, y = np.zeros((n, 3)), np.ones((n, 3))
        elif law == "clusters":
            x = np.where(np.arange(n)[:, None] % 3 == 0, 5.0, 0.0) * np.ones((n, 3))
            y = np.where(np.arange(n)[:, None] % 2 == 0, 5.0, 0.0) * np.ones((n, 3))
        else:
            x, y = rng.random((n, 1)), 1.0 + rng.random((n, 1))
        Xs.append(x.astype(np.float32))
        Ys.append(y.astype(np.float32))
    out, stats = run(ctx, ns, Xs, Ys, 0.03)
    check_instances(ns, Xs, Ys, 0.03, out, stats)


@pytest.mark.parametrize("eps", [1 / 3000, 1 / 32000])
def test_large_duals(ctx, eps):  # noqa: F811
    """Small eps: rounded costs and duals up to the ends of their 15 bits."""
    rng = np.random.default_rng(3)
    ns = [3, 12, 24]
    Xs = [rng.random((n, 2), dtype=np.float32) for n in ns]
    Ys = [(0.5 + rng.random((n, 2))).astype(np.float32) for n in ns]
    out, stats = run(ctx, ns, Xs, Ys, eps)
    check_instances(ns, Xs, Ys, eps, out, stats)


@pytest.mark.parametrize("engine", ["auto", "lds", "teams"])
@pytest.mark.parametrize("n_max", [1024, 1025])
@pytest.mark.parametrize("d,eps", [(2, 0.02), (8, 0.02)])
def test_phase_bound(ctx, monkeypatch, n_max, engine, d, eps):  # noqa: F811
    """The caller's phase bound stops every instance, whichever engine runs."""
    import functools
    import paper_2203_03732_amd as prot
    rng = np.random.default_rng(n_max)
    ns = [n_max, 300]
    Xs = [rng.random((n, d), dtype=np.float32) for n in ns]
    Ys = [(0.5 + rng.random((n, d))).astype(np.float32) for n in ns]
    monkeypatch.setattr(prot.Context, "_opts",
                        staticmethod(functools.partial(prot.Context._opts, phase_bound=3)))
    plan = ctx.batch(ns, d, eps, config={"engine": engine})
    plan.run(pack(Xs), pack(Ys), check=False)
    with pytest.raises(prot.ProtError) as e:
        plan.status()
    assert e.value.name == "phase_bound"
    at = 0
    for n, X, Y, st in zip(ns, Xs, Ys, plan.stats()):
        k, _ = oracle.round_points_f32(X, Y, eps)
        ref = oracle.solve_rounded(k, oracle.threshold(eps, n), max_phases=3, complete=False)
        assert ref["stats"]["phases"] == 3 and st["phases"] == 3 and st["status"] == -4
        for name in ("mate_a", "mate_b", "y_a", "y_b"):
            got = getattr(plan, name)[at:at + n].cpu().numpy()
            assert np.array_equal(got, ref[name]), name
        at += n
    plan.close()
