"""Launches on both sides of the size from which outputs are stored
non-temporally: a batch large enough gives every right-hand side the bits it
has alone (one launch of a few MB), in one launch and through the stages of
M_pc^dag M_pc, whose intermediates turn non-temporal later."""
import pytest

from paper_2112_01852_amd import inputs as I

pytestmark = pytest.mark.gpu

L, LS = (8, 6, 4, 8), 16     # 1.2 MB per FP32 half field


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01852_amd import qdwf as q
    d = q.Dirac(L, LS, M5=1.8, mf=0.01, b=1.5, c=0.5)
    d.set_gauge(I.gauge_field(L, "haar", 31))
    yield d
    d.close()


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("nrhs", [14, 66])
def test_batch_equals_single(D, prec, layout, nrhs):
    import torch
    from paper_2112_01852_amd import qdwf as q
    g = torch.Generator(device="cuda").manual_seed(prec + 10 * layout)
    n = q.qdwf_field_reals(D.ctx, q.QDWF_ODD)
    f = torch.randn(n * nrhs, generator=g, device="cuda").to(q.TORCH_DTYPE[prec])
    o, o1 = D.field(prec, q.QDWF_ODD, nrhs), D.field(prec, q.QDWF_ODD)
    w, w1 = (D.workspace(q.QDWF_OP_MDAGM, prec, k) for k in (nrhs, 1))
    pick = (0, nrhs // 2, nrhs - 1)
    q.qdwf_apply_MdagM(D.ctx, o, f, prec, layout, nrhs, w)
    for r in pick:
        q.qdwf_apply_MdagM(D.ctx, o1, f[r * n:(r + 1) * n], prec, layout, 1, w1)
        assert torch.equal(o[r * n:(r + 1) * n], o1)
    for dagger in (0, 1):
        q.qdwf_apply_Deo(D.ctx, o, f, q.QDWF_ODD, dagger, prec, layout, nrhs)
        for r in pick:
            q.qdwf_apply_Deo(D.ctx, o1, f[r * n:(r + 1) * n], q.QDWF_ODD, dagger, prec, layout)
            assert torch.equal(o[r * n:(r + 1) * n], o1)
    q.qdwf_apply_Dh(D.ctx, o, f, q.QDWF_ODD, 0, prec, layout, nrhs)
    for r in pick:
        q.qdwf_apply_Dh(D.ctx, o1, f[r * n:(r + 1) * n], q.QDWF_ODD, 0, prec, layout)
        assert torch.equal(o[r * n:(r + 1) * n], o1)
