"""Rows that chase the same few columns: thousands of proposals to a column in
a round, which the workgroups combine in LDS before they reach the column's
key. Bit-exact with the oracle, phase by phase."""
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


@pytest.mark.parametrize("origin", ["diag", "zero"])
@pytest.mark.parametrize("n_b,n_a,step", [
    (5000, 5000, 1),     # 40 neighbouring cheap columns: every table slot its own
    (5000, 5000, 64),    # cheap columns that share one slot of the table
    (6000, 7001, 67),    # unbalanced, ragged
    (700, 700, 5),       # fewer rows a workgroup than the combining needs
])
def test_convoys(ctx, n_b, n_a, step, origin):
    rng = np.random.default_rng(step)
    k = rng.integers(2, 5, (n_b, n_a)).astype(np.int16)
    cheap = np.arange(40) * step % n_a
    k[:, cheap] = rng.integers(0, 2, (n_b, len(cheap)))
    ldk = -(-n_a // 128) * 128
    kd = torch.full((n_b, ldk), 0x7FFF, dtype=torch.int16, device="cuda")
    kd[:, :n_a] = torch.from_numpy(k).cuda()
    res = ctx.solve_rounded(kd, 10, n_b, n_a=n_a, origin=origin, complete=False, max_phases=3)
    ref = oracle.solve_rounded(k, 10, origin=origin, complete=False, max_phases=3)
    for name in ("mate_a", "mate_b", "y_a", "y_b"):
        assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), name
    for s in ("phases", "rounds", "max_rounds", "scanned", "sum_free"):
        assert res.stats[s] == ref["stats"][s], s


@pytest.mark.parametrize("n_a", [262144, 262145, 262144 + 200])
def test_columns_beyond_the_table(monkeypatch, n_a):
    """Cheap columns 262,144 apart, chased by rows of the same workgroup: the
    first columns by half of them, the last ones by the others."""
    import paper_2203_03732_amd as prot
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("PROT_LOOP_MAX_GRID", "4")  # 75 rows a workgroup
    n_b, m = 300, 200
    far = 262144 if n_a >= 262144 + m else n_a - m
    k = np.full((n_b, n_a), 2, np.int16)
    rng = np.random.default_rng(7)
    high = rng.random(n_b) < 0.5
    k[~high, :m] = 0
    k[high, far:far + m] = 0
    ldk = -(-n_a // 128) * 128
    kd = torch.full((n_b, ldk), 0x7FFF, dtype=torch.int16, device="cuda")
    kd[:, :n_a] = torch.from_numpy(k).cuda()
    c = prot.Context(0)
    try:
        res = c.solve_rounded(kd, 3, n_b, n_a=n_a, origin="zero", complete=False, max_phases=3)
        ref = oracle.solve_rounded(k, 3, origin="zero", complete=False, max_phases=3)
        for name in ("mate_a", "mate_b", "y_a", "y_b"):
            assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), name
        for s in ("phases", "rounds", "max_rounds", "scanned", "sum_free"):
            assert res.stats[s] == ref["stats"][s], s
    finally:
        torch.cuda.synchronize()
        c.close()
