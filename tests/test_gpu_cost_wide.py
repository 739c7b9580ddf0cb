"""The point-set builds of many pairs (128 x 128 tiles): rounded costs and the
largest squared distance bit-exact with the oracle at ragged edges, for rows that
allow 16-byte loads and rows that do not, and for batches of uneven instances."""
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


def unaligned(a):
    """a on the device, 4 bytes past a 16-byte boundary."""
    buf = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")
    out = buf[1:].view(a.shape)
    out.copy_(torch.from_numpy(a))
    return out


@pytest.mark.parametrize("metric", ["sqeuclidean", "euclidean"])
@pytest.mark.parametrize("n_b,n_a,d,eps", [
    (2497, 2497, 4, 0.01), (2433, 2561, 5, 0.003), (2560, 2560, 16, 0.05), (2500, 2625, 20, 0.02)])
def test_builds(ctx, n_b, n_a, d, eps, metric):
    rng = np.random.default_rng(n_b + d)
    X, Y = (rng.standard_normal((n, d), dtype=np.float32) for n in (n_b, n_a))
    round_f32 = oracle.round_points_f32 if metric == "sqeuclidean" else oracle.round_points_euclid_f32
    k_ref, m_ref = round_f32(X, Y, eps)
    ctx.set_cost_metric(metric)
    try:
        for put in (lambda a: torch.from_numpy(a).cuda(), unaligned):
            k, m = ctx.build_costs(put(X), put(Y), eps)
            k = k.cpu().numpy()
            assert float(m[0]) == m_ref
            assert np.array_equal(k[:, :n_a], k_ref)
            assert (k[:, n_a:] == 0x7FFF).all()
    finally:
        ctx.set_cost_metric("sqeuclidean")


@pytest.mark.parametrize("k_type", ["auto", "uint8"])
def test_batch_and_bytes(ctx, k_type):
    rng = np.random.default_rng(3)
    if k_type == "uint8":
        X, Y = (rng.standard_normal((2500, 8), dtype=np.float32) for _ in range(2))
        res = ctx.solve_points(*(torch.from_numpy(a).cuda() for a in (X, Y)), 0.05, k_type=k_type)
        k, _ = oracle.round_points_f32(X, Y, 0.05)
        ref = oracle.solve_rounded(k, oracle.threshold(0.05, 2500))
        for name in ("mate_b", "y_a", "y_b"):
            assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), name
        return
    ns = [1, 63, 64, 65, 127, 129, 300, 511, 640] * 5
    off = np.concatenate([[0], np.cumsum(ns)])
    X, Y = (rng.standard_normal((off[-1], 12), dtype=np.float32) for _ in range(2))
    ma, mb, ya, yb, st = ctx.solve_batched_points(ns, *(torch.from_numpy(a).cuda() for a in (X, Y)),
                                                  0.05)
    for i in range(9):
        s = slice(off[i], off[i + 1])
        k, _ = oracle.round_points_f32(X[s], Y[s], 0.05)
        ref = oracle.solve_rounded(k, oracle.threshold(0.05, ns[i]))
        assert np.array_equal(mb[s].cpu().numpy(), ref["mate_b"]) and \
            np.array_equal(ya[s].cpu().numpy(), ref["y_a"]), ns[i]


def test_non_finite(ctx):
    import paper_2203_03732_amd as prot
    for bad in (np.nan, -np.inf, 3e38):
        X = np.ones((2500, 8), np.float32)
        X[2400, 7] = bad
        with pytest.raises(prot.ProtError):
            ctx.solve_points(torch.from_numpy(X).cuda(), torch.zeros_like(torch.from_numpy(X)).cuda(),
                             0.1)


@pytest.mark.parametrize("scale", [1e-19, 1e-20, 3e-22])
@pytest.mark.parametrize("d", [4, 8, 16])
def test_smallest_scales(ctx, d, scale):
    """Squared distances down to the smallest binary32 numbers: 1 / (m eps)
    leaves the range of binary32."""
    rng = np.random.default_rng(d)
    X, Y = (rng.random((2500, d), dtype=np.float32) * np.float32(scale) for _ in range(2))
    k_ref, m_ref = oracle.round_points_f32(X, Y, 0.01)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    k, m = ctx.build_costs(Xd, Yd, 0.01)
    assert float(m[0]) == m_ref
    assert np.array_equal(k.cpu().numpy()[:, :2500], k_ref)
    # a byte matrix is read through the solve
    res = ctx.solve_points(Xd, Yd, 0.01, k_type="uint8", max_phases=2)
    ref = oracle.solve_rounded(k_ref, oracle.threshold(0.01, 2500), max_phases=2)
    assert res.stats["scanned"] == ref["stats"]["scanned"]
    for name in ("mate_b", "y_a", "y_b"):
        assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), name


@pytest.mark.parametrize("metric", ["sqeuclidean", "euclidean"])
@pytest.mark.parametrize("n_b,n_a,d", [
    (1, 98305, 4), (70, 49025, 16), (70, 49153, 16),  # thin: 1,534 and 1,538 small tiles
    (2880, 2881, 7), (2896, 2945, 32), (2945, 2945, 33),  # the Euclidean lines
    (2561, 2560, 40), (2561, 2560, 41), (4097, 4033, 48), (65, 17, 5)])
def test_rules(ctx, n_b, n_a, d, metric):
    """Either side of the lines between small and wide tiles, and rectangles
    whose grid follows both sides."""
    rng = np.random.default_rng(n_b + d)
    X, Y = (rng.standard_normal((n, d), dtype=np.float32) for n in (n_b, n_a))
    round_f32 = oracle.round_points_f32 if metric == "sqeuclidean" else oracle.round_points_euclid_f32
    k_ref, m_ref = round_f32(X, Y, 0.02)
    ctx.set_cost_metric(metric)
    try:
        k, m = ctx.build_costs(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), 0.02)
        k = k.cpu().numpy()
        assert float(m[0]) == m_ref
        assert np.array_equal(k[:, :n_a], k_ref)
        assert (k[:, n_a:] == 0x7FFF).all()
    finally:
        ctx.set_cost_metric("sqeuclidean")
