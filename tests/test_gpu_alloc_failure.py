"""An allocation that fails while a context's workspace grows: the call returns
'nomem', and later calls of sizes that had fitted give what they gave."""
import numpy as np
import pytest

import oracle
from paper_2203_03732_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx():
    import paper_2203_03732_amd as prot
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = prot.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def rounded(n, seed):
    k = np.random.default_rng(seed).integers(0, 20, (n, n)).astype(np.int16)
    kd = torch.full((n, -(-n // 128) * 128), 0x7FFF, dtype=torch.int16, device="cuda")
    kd[:, :n] = torch.from_numpy(k).cuda()
    return k, kd


# bytes of the last array that can be had: the loop's keys, its column duals,
# its lists' scratch; the 6 MB of tagged lists cannot
@pytest.mark.parametrize("limit", [1000, 13000, 60000, 1000000])
def test_loop(ctx, monkeypatch, limit):
    import paper_2203_03732_amd as prot
    k, kd = rounded(500, 1)
    _, big = rounded(6000, 2)
    ref = oracle.solve_rounded(k, 5)
    for i in range(2):
        res = ctx.solve_rounded(kd, 5, 500)
        for name in ("mate_a", "mate_b", "y_a", "y_b"):
            assert np.array_equal(getattr(res, name).cpu().numpy(), ref[name]), (i, name)
        if i == 0:
            monkeypatch.setenv("PROT_ALLOC_LIMIT", str(limit))
            with pytest.raises(prot.ProtError) as e:
                ctx.solve_rounded(big, 60, 6000)
            assert e.value.name == "nomem"
            monkeypatch.delenv("PROT_ALLOC_LIMIT")


@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("limit", [1000, 3000, 6000, 200000])
def test_transport(ctx, monkeypatch, limit, clustered):
    import paper_2203_03732_amd as prot

    def solve(n):
        C, nu, mu = synth.transport_clouds(n, n, seed=3, shift=0.5)
        args = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (C, nu, mu))
        return ctx.ot_solve(*args, 0.2, clustered=clustered)

    first = solve(40)
    monkeypatch.setenv("PROT_ALLOC_LIMIT", str(limit))
    with pytest.raises(prot.ProtError) as e:
        solve(500)
    assert e.value.name == "nomem"
    monkeypatch.delenv("PROT_ALLOC_LIMIT")
    again = solve(40)
    assert torch.equal(first.plan, again.plan) and torch.equal(first.y_b_lo, again.y_b_lo)
    assert first.stats["rounds"] == again.stats["rounds"]
