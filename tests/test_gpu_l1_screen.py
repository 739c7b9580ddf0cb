"""The screened build of the L1 image cost: k equals the definition on every
entry, for sparse and dense vectors, ragged sizes, pairs on a rounding boundary
(no common pixel, 1 / eps whole) and lists that overflow."""
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
    c.set_cost_metric("l1_normalized")
    yield c
    torch.cuda.synchronize()
    c.close()


def vectors(law, n, d, rng):
    if law == "dense":
        return (0.1 + rng.random((n, d))).astype(np.float32)
    if law == "sparse":  # a few common pixels, many pairs without any
        x = np.where(rng.random((n, d)) < 0.03, rng.random((n, d)), 0.0)
        x[np.arange(n), rng.integers(0, d, n)] += 0.5
        return x.astype(np.float32)
    if law == "disjoint":  # two halves: every other pair at cost 1 (lists overflow)
        x = np.zeros((n, d))
        for i in range(n):
            half = slice(0, d // 2) if i % 2 else slice(d // 2, d)
            x[i, half] = rng.random(d)[half]
        return x.astype(np.float32)
    x = np.zeros((n, d))  # "levels": equal pixels, costs on whole fractions
    for i in range(n):
        x[i, rng.permutation(d)[:20]] = 1.0
    return x.astype(np.float32)


@pytest.mark.parametrize("law,n_b,n_a,d,eps", [
    ("sparse", 600, 700, 784, 0.1),
    ("sparse", 513, 513, 785, 0.07),
    ("sparse", 3000, 3001, 257, 0.1),
    ("dense", 640, 641, 1024, 0.05),
    ("disjoint", 600, 600, 600, 0.1),
    ("levels", 1025, 1030, 300, 0.05),
    ("dense", 500, 520, 801, 0.1 / 3),
])
def test_k_equals_the_definition(ctx, law, n_b, n_a, d, eps):
    assert n_b * n_a * d >= 5e7  # large enough to be screened
    rng = np.random.default_rng(n_b + d)
    X, Y = vectors(law, n_b, d, rng), vectors(law, n_a, d, rng)
    k, _ = ctx.build_costs(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), eps)
    ref = oracle.round_l1_normalized_f32(X, Y, eps)
    got = k.cpu().numpy()
    assert np.array_equal(got[:, :n_a], ref)
    assert (got[:, n_a:] == 0x7FFF).all()


def test_bytes_and_solve(ctx):
    """The byte matrix through a whole solve: matching and duals as with int16."""
    rng = np.random.default_rng(5)
    X, Y = (torch.from_numpy(vectors("sparse", 700, 500, rng)).cuda() for _ in range(2))
    a = ctx.solve_points(X, Y, 0.1, k_type="uint8")
    b = ctx.solve_points(X, Y, 0.1)
    for name in ("mate_a", "mate_b", "y_a", "y_b"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    assert a.stats["sum_k"] == b.stats["sum_k"]


def test_without_workspace(monkeypatch):
    """Where the screening workspace cannot be had, every pair is taken by the
    definition."""
    import paper_2203_03732_amd as prot
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(11)
    X, Y = vectors("sparse", 300, 784, rng), vectors("sparse", 310, 784, rng)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    ref = oracle.round_l1_normalized_f32(X, Y, 0.1)
    c = prot.Context(0)
    try:
        c.set_cost_metric("l1_normalized")
        c.solve_points(Xd, Yd, 0.005)  # too fine for the screen: all other workspaces
        monkeypatch.setenv("PROT_ALLOC_LIMIT", "65536")
        for limited in (True, False):
            k, _ = c.build_costs(Xd, Yd, 0.1)
            assert np.array_equal(k.cpu().numpy()[:, :310], ref), limited
            res = c.solve_points(Xd, Yd, 0.1)
            want = oracle.solve_rounded(ref, oracle.threshold(0.1, 300))
            assert np.array_equal(res.mate_b.cpu().numpy(), want["mate_b"]), limited
            monkeypatch.delenv("PROT_ALLOC_LIMIT", raising=False)
    finally:
        torch.cuda.synchronize()
        c.close()
