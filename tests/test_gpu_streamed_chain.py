"""M_pc^dag M_pc on both sides of the size from which a batch's intermediates
are stored non-temporally (100 MiB): every right-hand side gets the bits it
has alone."""
import pytest

from paper_2112_01852_amd import inputs as I

pytestmark = pytest.mark.gpu

L, LS = (8, 6, 4, 8), 16     # 288 Ki reals per half field


@pytest.mark.parametrize("prec,nrhs", [(0, 44), (0, 45), (1, 88), (1, 89), (2, 177), (2, 178), (3, 178)])
def test_batch_equals_single(prec, nrhs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01852_amd import qdwf as q
    D = q.Dirac(L, LS, M5=1.8, mf=0.01, b=1.5, c=0.5)
    D.set_gauge(I.gauge_field(L, "haar", 37))
    n = q.qdwf_field_reals(D.ctx, q.QDWF_ODD)
    f = torch.randn(n * nrhs, generator=torch.Generator(device="cuda").manual_seed(prec),
                    device="cuda").to(q.TORCH_DTYPE[prec])
    o, o1 = D.field(prec, q.QDWF_ODD, nrhs), D.field(prec, q.QDWF_ODD)
    w, w1 = (D.workspace(q.QDWF_OP_MDAGM, prec, k) for k in (nrhs, 1))
    q.qdwf_apply_MdagM(D.ctx, o, f, prec, q.QDWF_RIRI, nrhs, w)
    for r in (0, nrhs // 2, nrhs - 1):
        q.qdwf_apply_MdagM(D.ctx, o1, f[r * n:(r + 1) * n], prec, q.QDWF_RIRI, 1, w1)
        assert torch.equal(o[r * n:(r + 1) * n], o1)
    D.close()
