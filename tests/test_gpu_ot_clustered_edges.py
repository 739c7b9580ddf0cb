"""Clustered transport at the edges of its row listing: rows of one step (2 or 4
chunks a lane) and of several, supply points of one, two and four a thread,
lists in LDS and beyond. Bit-exact with the oracle after three phases."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_b,n_a,cap", [
    (1024, 1016, None), (33, 1017, "5"), (1025, 2040, None), (64, 2041, None), (2049, 65, None),
    (1, 4096, None), (4096, 3, "0")])
def test_listing_edges(n_b, n_a, cap, monkeypatch):
    import paper_2203_03732_amd as prot
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if cap is not None:
        monkeypatch.setenv("PROT_CLUSTER_LIST_CAP", cap)
    rng = np.random.default_rng(n_b + n_a)
    C = rng.random((n_b, n_a), dtype=np.float32)
    nu, mu = (w / w.sum() for w in (rng.random(n) + 0.05 for n in (n_b, n_a)))
    orc = oracle.ot_solve_clustered(C, nu, mu, 0.3, max_phases=3, trace=True)
    ctx = prot.Context(0)
    args = (torch.from_numpy(a).cuda() for a in (C, nu, mu))
    gpu = ctx.ot_solve(*args, 0.3, max_phases=3, clustered=True)
    for k in ("phases", "sum_free", "rounds", "max_rounds", "scanned", "matched_in_phases"):
        assert gpu.stats[k] == orc["stats"][k], k
    assert np.array_equal(ctx.trace(), orc["trace"])
    # the larger dual of a point's copies: lo + 1 unless all its copies are at lo
    for lo, n_lo, copies, top in ((gpu.y_b_lo, gpu.y_b_nlo, orc["s"], orc["Y"]),
                                  (gpu.y_a_lo, gpu.y_a_nlo, orc["d"], orc["Z"])):
        lo, n_lo = lo.cpu().numpy(), n_lo.cpu().numpy()
        held = copies > 0
        assert np.array_equal((lo + (n_lo < copies))[held], top[held])
    ctx.close()
