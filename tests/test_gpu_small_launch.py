"""The forms small launches take (a site's directions on four wavefronts;
blocks of one wavefront) against the form large ones take (QDWF_HOP_THREADS
fixes the block and with it the ordinary form), on both sides of the line
between them, with ragged last wavefronts, for every operator that hops.
The results
are equal bit for bit, which is what lets a right-hand side not depend on
the batch it comes in.
"""
import os

import pytest

from paper_2112_01852_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Ls,nrhs", [((4, 4, 4, 4), 8, 1), ((6, 2, 2, 6), 16, 1), ((4, 2, 4, 6), 12, 3),
                                       ((2, 2, 2, 2), 4, 1), ((6, 6, 4, 6), 10, 1), ((8, 8, 8, 8), 8, 1),
                                       ((8, 8, 8, 8), 8, 2), ((4, 2, 2, 2), 20, 1), ((4, 2, 2, 2), 2, 1)])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_forms_agree(L, Ls, nrhs, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01852_amd import qdwf as q
    D = q.Dirac(L, Ls, M5=1.8, mf=0.2, b=1.5, c=0.5)
    D.set_gauge(I.gauge_field(L, "haar", 9))
    n = q.qdwf_field_reals(D.ctx, q.QDWF_ODD)
    f = torch.randn(2 * n * nrhs, generator=torch.Generator(device="cuda").manual_seed(prec),
                    device="cuda").to(q.TORCH_DTYPE[prec])
    h = f[: n * nrhs]
    ws = D.workspace(q.QDWF_OP_MPC, prec, nrhs)

    def results():
        out = []
        for dagger in (0, 1):
            a, b, c = D.field(prec, nrhs=nrhs), D.field(prec, q.QDWF_EVEN, nrhs), D.field(prec, q.QDWF_ODD, nrhs)
            q.qdwf_apply_D(D.ctx, a, f, dagger, prec, q.QDWF_RIRI, nrhs)
            q.qdwf_apply_Deo(D.ctx, b, h, q.QDWF_EVEN, dagger, prec, q.QDWF_RIRI, nrhs)
            q.qdwf_apply_Mpc(D.ctx, c, h, dagger, prec, q.QDWF_RIRI, nrhs, ws)
            out += [a, b, c]
        torch.cuda.synchronize()
        return out

    small = results()
    os.environ["QDWF_HOP_THREADS"] = "256" if Ls > 4 else "64"
    try:
        large = results()
    finally:
        del os.environ["QDWF_HOP_THREADS"]
    assert all(torch.equal(x, y) for x, y in zip(small, large))
    D.close()
