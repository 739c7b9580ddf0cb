"""A single instance of few columns, solved by one workgroup from the start or
from a state with few free rows: bit-exact with the oracle, phase by phase, at
the sizes where the routes meet, for every stop and option the caller has."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2203_03732_amd as prot
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = prot.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def check(ctx, C, eps, origin="diag", **kw):
    strict = kw.get("eps_mode") == "strict"
    ei = eps / 3 if strict else eps
    res = ctx.solve_cost(torch.from_numpy(C).cuda(), eps, origin=origin, **kw)
    kw.pop("eps_mode", None), kw.pop("k_type", None)
    k = oracle.round_cost(C, ei)
    ref = oracle.solve_rounded(k, oracle.threshold(ei, C.shape[0]), origin=origin, trace=True, **kw)
    for name in ("mate_a", "mate_b", "y_a", "y_b"):
        assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), name
    for s in ("phases", "rounds", "max_rounds", "scanned", "sum_free", "sum_k"):
        assert res.stats[s] == ref["stats"][s], s
    assert np.array_equal(ctx.trace(), ref["trace"])
    return res, ref


def costs(n_b, n_a, seed, low=False):
    """low: columns that every row likes in the same order (long phases)."""
    rng = np.random.default_rng(seed)
    C = rng.random((n_b, n_a), dtype=np.float32)
    return np.minimum(C * 0.2 + rng.random(n_a, dtype=np.float32) * 0.7, 1.0) if low else C


@pytest.mark.parametrize("origin", ["diag", "zero"])
@pytest.mark.parametrize("n_b,n_a,eps", [
    (1, 1, 0.5), (1, 2000, 0.1), (63, 65, 0.02), (400, 400, 0.02),   # from the start
    (401, 401, 0.02), (129, 1241, 0.01),                         # either side of it
    (1024, 1024, 0.03), (1017, 1025, 0.02), (2048, 2048, 0.01),      # taken over, both layouts
    (2041, 2049, 0.01),                                              # too many columns
])
def test_routes(ctx, n_b, n_a, eps, origin):
    C = costs(n_b, n_a, n_b + n_a, low=n_b % 2 == 0)
    check(ctx, C, eps, origin)
    check(ctx, C, eps, origin, k_type="uint8")


@pytest.mark.parametrize("n", [300, 900, 1500])
def test_stops_and_options(ctx, n):
    C = costs(n, n, n, low=True)
    _, ref = check(ctx, C, 0.02)
    free = ref["trace"][:, 0]
    late = int(np.argmax(free <= 128)) if (free <= 128).any() else len(free) - 1
    for phases in sorted({1, late, late + 1, late + 2, len(free)} - {0}):
        res, _ = check(ctx, C, 0.02, max_phases=phases)
        assert res.status == ("ok" if phases >= len(free) else "partial")
    check(ctx, C, 0.02, complete=False)
    check(ctx, C, 0.06, eps_mode="strict")
    check(ctx, C, 0.02, k_type="uint8")


def test_watchdog_and_bad_costs(ctx):
    import paper_2203_03732_amd as prot
    rng = np.random.default_rng(5)
    for n in (200, 1000):
        X, Y = (torch.from_numpy(rng.random((n, 3), dtype=np.float32)).cuda() for _ in range(2))
        full = ctx.solve_points(X, Y, 0.01)
        res = ctx.solve_points(X, Y, 0.01, phase_bound=full.stats["phases"] - 1)
        assert res.stats["phases"] == full.stats["phases"] - 1 and res.status == "phase_bound"
        C = costs(n, n, n)
        C[3, 4] = np.nan
        with pytest.raises(prot.ProtError):
            ctx.solve_cost(torch.from_numpy(C).cuda(), 0.05)
        # the context goes on
        check(ctx, costs(n, n, n), 0.05)


def test_enqueued_and_repeated(ctx):
    """Solves of several sizes one after another without synchronisation."""
    rng = np.random.default_rng(9)
    jobs = [(n, *(torch.from_numpy(rng.random((n, 2), dtype=np.float32)).cuda() for _ in range(2)))
            for n in (300, 1024, 64, 2048, 300)]
    out = [ctx.solve_points(X, Y, 0.01, stats=False) for _, X, Y in jobs]
    torch.cuda.synchronize()
    for (n, X, Y), res in zip(jobs, out):
        ref = oracle.solve_points(X.cpu().numpy(), Y.cpu().numpy(), 0.01)
        for name in ("mate_a", "mate_b", "y_a", "y_b"):
            assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), (n, name)


@pytest.mark.parametrize("k_type", ["int16", "uint8"])
@pytest.mark.parametrize("n,bad_rows,eps", [(40, 40, 0.1), (450, 100, 0.05)])
def test_bad_costs_without_watchdog(ctx, monkeypatch, n, bad_rows, eps, k_type):
    """Rows that hold only costs far above 1 never find a column; with the
    watchdog off their duals' range ends the loop."""
    import functools
    import paper_2203_03732_amd as prot
    C = costs(n, n, n)
    C[:bad_rows] = 1e9
    monkeypatch.setattr(ctx, "_opts", functools.partial(ctx._opts, phase_bound=-1), raising=False)
    with pytest.raises(prot.ProtError) as e:
        ctx.solve_cost(torch.from_numpy(C).cuda(), eps, k_type=k_type)
    assert e.value.code in (-2, -5)  # range, state
    if bad_rows == n:
        assert e.value.code == -5
    monkeypatch.undo()
    check(ctx, costs(n, n, n), eps, k_type=k_type)


@pytest.mark.parametrize("kind,n_b,n_a,eps", [
    ("cost", 2048, 2048, 0.006), ("cost", 2048, 2048, 0.0063), ("cost", 1900, 2000, 0.0065),
    ("cost", 1874, 2000, 0.006),                                     # too many spare columns
    ("points", 2041, 2041, 0.0103), ("points", 2041, 2041, 0.011), ("points", 2040, 2048, 0.005),
    ("euclidean", 1793, 2048, 0.0175), ("euclidean", 1791, 2048, 0.0175)])
def test_rule_above_1024(ctx, kind, n_b, n_a, eps):
    """Either side of the lines between the grid's loop alone and the hand-over
    to one workgroup, above 1,024 columns."""
    if kind == "cost":
        C = costs(n_b, n_a, n_b, low=True)
        check(ctx, C, eps, max_phases=60)
        return
    rng = np.random.default_rng(n_b)
    X, Y = (rng.random((n, 2), dtype=np.float32) for n in (n_b, n_a))
    ctx.set_cost_metric("sqeuclidean" if kind == "points" else kind)
    try:
        res = ctx.solve_points(*(torch.from_numpy(a).cuda() for a in (X, Y)), eps)
    finally:
        ctx.set_cost_metric("sqeuclidean")
    round_f32 = oracle.round_points_f32 if kind == "points" else oracle.round_points_euclid_f32
    k, _ = round_f32(X, Y, eps)
    ref = oracle.solve_rounded(k, oracle.threshold(eps, n_b), trace=True)
    for name in ("mate_a", "mate_b", "y_a", "y_b"):
        assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), name
    for s in ("phases", "rounds", "max_rounds", "scanned", "sum_free", "sum_k"):
        assert res.stats[s] == ref["stats"][s], s
    assert np.array_equal(ctx.trace(), ref["trace"])
