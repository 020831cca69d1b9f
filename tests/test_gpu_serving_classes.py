"""Requests of every class a pool advances side by side (Ls = 16, the other Ls
with M_ee^-1 inside the hop, and those with it in a launch of its own) served
together equal, bit for bit, the same requests served alone, for rounds
shorter and longer than the distance between two offers of a reliable update;
a pool is used again after its first batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inner,every", [(2, 3), (2, 8), (1, 1), (0, 6)])
def test_mixed_classes(inner, every):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01852_amd import qdwf as q
    from paper_2112_01852_amd import serve
    S = serve.Spec
    specs = [S((4, 4, 4, 4), 16, 0.1, 21, 22), S((4, 4, 2, 6), 12, 0.08, 23, 24),
             S((4, 4, 4, 4), 11, 0.1, 25, 26), S((4, 2, 4, 4), 20, 0.1, 27, 28)]
    prm = q.solve_params(inner_prec=inner, layout=q.QDWF_RIRI, tol=1e-10, check_every=every)
    prepared = serve.prepare(specs)
    arena = 64 << 20
    res = serve.run_pool(prepared, np.zeros(4), prm, arena, max_slots=4)
    assert res["status"] == [q.QDWF_OK] * 4
    for i, p in enumerate(prepared):
        together = p.x.clone()
        p.x.zero_()
        alone = serve.run_pool([p], np.zeros(1), prm, arena, max_slots=1)
        assert torch.equal(p.x, together)
        assert alone["stats"][0]["iterations"] == res["stats"][i]["iterations"]
        rc, st, _, solo = serve.solo_solve(p, prm)
        assert rc == q.QDWF_OK
        assert float((solo - together).abs().max()) <= 1e-8 * float(solo.abs().max())
