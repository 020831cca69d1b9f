"""The Wilson kernel's block order that takes one half field after another:
batches and both parities, numbers of blocks that the XCDs do not divide, and
both sides of the line to the other order, against the FP64 oracle right-hand
side by right-hand side. Tolerances as in test_gpu_wilson.py."""
import numpy as np
import pytest

from oracle import cpu
from paper_2112_01852_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = {0: 1e-13, 1: 1e-6, 2: 5e-3, 3: 5e-3}
SHAMIR = dict(M5=1.8, mf=0.01, b=1.0, c=0.0)


@pytest.mark.parametrize("L,Ls,nrhs", [((8, 6, 4, 8), 1, 1), ((8, 6, 4, 8), 1, 5), ((16, 6, 10, 6), 1, 3),
                                       ((6, 4, 4, 6), 8, 2), ((10, 6, 6, 6), 5, 3),
                                       ((16, 16, 16, 48), 1, 1), ((16, 16, 16, 50), 1, 1),
                                       ((16, 16, 16, 24), 1, 2), ((16, 16, 16, 26), 1, 2)])
@pytest.mark.parametrize("layout", [0, 1])
def test_hop(L, Ls, nrhs, layout):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01852_amd import qdwf as q
    a = cpu.Action(L=L, Ls=Ls, **SHAMIR)
    U = I.gauge_field(L, "haar", 60 + Ls)
    psi = I.gaussian_spinor(L, Ls, 61 + Ls, nrhs=nrhs)
    ref = [cpu.hop(a, U, v) for v in psi]
    D = q.Dirac(L, Ls, **SHAMIR)
    D.set_gauge(U)
    for prec in range(4):
        f = D.pack(psi, prec, layout, q.QDWF_FULL, nrhs)
        out = D.field(prec, q.QDWF_FULL, nrhs)
        q.qdwf_apply_Dh(D.ctx, out, f, q.QDWF_FULL, 0, prec, layout, nrhs)
        full = D.unpack(out, prec, layout, q.QDWF_FULL, nrhs).cpu().numpy()
        f = D.pack(psi, prec, layout, q.QDWF_EVEN, nrhs)
        out = D.field(prec, q.QDWF_ODD, nrhs)
        q.qdwf_apply_Dh(D.ctx, out, f, q.QDWF_ODD, 0, prec, layout, nrhs)
        odd = D.unpack(out, prec, layout, q.QDWF_ODD, nrhs).cpu().numpy()
        for r in range(nrhs):
            got = full[r] if nrhs > 1 else full
            assert np.linalg.norm(got - ref[r]) < TOL[prec] * np.linalg.norm(ref[r]), (prec, r)
            want = cpu.restrict(ref[r], L, 1)
            got = odd[r] if nrhs > 1 else odd
            assert np.linalg.norm(got - want) < TOL[prec] * np.linalg.norm(want), (prec, r)
    D.close()
