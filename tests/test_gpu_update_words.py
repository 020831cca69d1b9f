"""Solves with 16-bit inner vectors, whose reliable update writes the inner
residual and direction four reals a lane: fields smaller than a block, of
whole blocks and with a ragged last block, one and three sources.

The FP64 residual of what comes back, by the oracle's operator, is at most the
tolerance plus the rounding of the oracle and of x itself, and a source's
solution does not depend on the batch. Updates that restarted the direction
wrongly would cost iterations, so these stay within 1.5 times the FP64 count
plus ten, the bound the other solves hold.
"""
import numpy as np
import pytest

from oracle import cpu
from paper_2112_01852_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Ls", [((2, 2, 2, 2), 2), ((4, 4, 4, 4), 8), ((4, 2, 6, 2), 10)])
@pytest.mark.parametrize("inner", [2, 3])
def test_update_of_16_bit_vectors(L, Ls, inner):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01852_amd import qdwf as q
    P = dict(M5=1.8, mf=0.05, b=1.5, c=0.5)
    a = cpu.Action(L=L, Ls=Ls, **P)
    U = I.gauge_field(L, "smooth", 31, eps=0.3)
    D = q.Dirac(L, Ls, **P)
    D.set_gauge(U)
    bs = np.stack([cpu.restrict(I.gaussian_spinor(L, Ls, 40 + j), L, 1) for j in range(3)])

    def solve(b, nrhs, prec):
        f = D.pack(b, q.QDWF_F64, q.QDWF_RIRI, q.QDWF_ODD, nrhs)
        x = D.field(q.QDWF_F64, q.QDWF_ODD, nrhs)
        prm = q.solve_params(inner_prec=prec, layout=q.QDWF_RIRI, tol=1e-10)
        rc, st = q.qdwf_solve(D.ctx, x, f, nrhs, prm, D.workspace(q.QDWF_OP_SOLVE, prec, nrhs))
        assert rc == q.QDWF_OK, q.qdwf_last_error()
        return D.unpack(x, q.QDWF_F64, q.QDWF_RIRI, q.QDWF_ODD, nrhs).cpu().numpy(), st

    xs, _ = solve(bs, 3, inner)
    for j in range(3):
        x, st = solve(bs[j], 1, inner)
        r = bs[j] - cpu.mpc(a, U, cpu.mpc(a, U, x), dagger=True)
        assert np.linalg.norm(r) / np.linalg.norm(bs[j]) <= 1.5e-10
        assert np.array_equal(xs[j].reshape(x.shape), x)
        assert st.reliable_updates >= 1
        _, st0 = solve(bs[j], 1, q.QDWF_F64)
        assert st.iterations <= 1.5 * st0.iterations + 10, (st.iterations, st0.iterations)
    D.close()
