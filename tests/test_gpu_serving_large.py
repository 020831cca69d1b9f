"""A request with more wavefronts than one block adds (16^3 x 34, Ls = 16:
17408) beside small ones of its class and of others, the last one admitted
after another has gone: each equals the same request served alone, bit for
bit, and qdwf_solve's solution as far as the residual tolerance goes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_large_member():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01852_amd import qdwf as q
    from paper_2112_01852_amd import serve
    S = serve.Spec
    specs = [S((4, 4, 4, 4), 16, 0.1, 21, 22), S((16, 16, 16, 34), 16, 0.1, 23, 24),
             S((4, 4, 2, 6), 12, 0.08, 25, 26), S((4, 2, 4, 4), 16, 0.1, 27, 28)]
    prm = q.solve_params(inner_prec=q.QDWF_F16, layout=q.QDWF_RIRI, tol=1e-6, check_every=8)
    prepared = serve.prepare(specs)
    arena = (32 << 20) + sum(q.qdwf_request_bytes(s.action(), prm) for s in specs)
    res = serve.run_pool(prepared, np.zeros(4), prm, arena, max_slots=3)
    assert res["status"] == [q.QDWF_OK] * 4
    for i, p in enumerate(prepared):
        together = p.x.clone()
        p.x.zero_()
        alone = serve.run_pool([p], np.zeros(1), prm, arena, max_slots=1)
        assert torch.equal(p.x, together)
        assert alone["stats"][0]["iterations"] == res["stats"][i]["iterations"]
        rc, st, _, solo = serve.solo_solve(p, prm)
        assert rc == q.QDWF_OK
        assert float((solo - together).abs().max()) <= 1e-5 * float(solo.abs().max())
