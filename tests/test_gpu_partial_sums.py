"""The reduction over a hop's workgroups at numbers of partial sums on both sides
of one pass of its 1024 threads x 8 strands (8192), and at several passes.

With 144 lanes a site (Ls = 16, nine right-hand sides) one site per workgroup is
the only shape, so the hops of A leave one partial sum per site of a parity:
alpha of the first CG iteration is a sum over that many, beta of the second too.
The iterates are compared with the same recurrence on torch sums of the fields
and mdagm.  Tolerance: sums of up to 8 million products in FP64 differ by a few
1e-15 times the number of passes and by the cancellation in <p, A p> (a factor
of 100 at most); a lost or repeated partial sum is 1/20000 of one.
"""
import pytest

from paper_1811_08488_amd import mspcg as M
from paper_1811_08488_amd import synth
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

NRHS, LS = 9, 16


@pytest.mark.parametrize("L,sites", [((2, 6, 22, 62), 8184), ((8, 8, 16, 16), 8192), ((2, 10, 10, 82), 8200),
                                     ((10, 10, 20, 20), 20000)], ids=lambda p: str(p) if isinstance(p, int) else "")
def test_cg_iterates_with_one_partial_per_site(L, sites):
    torch = require_gpu()
    A = M.Action(L, LS, M5=1.8, mf=0.05, b=1.5, c=0.5)
    assert A.V // 2 == sites
    h = M.Handle(A, synth.gauge_field(L, 0.45, 101))
    b = h.field(M.F64, NRHS, 0)
    b.data.normal_(generator=torch.Generator("cuda").manual_seed(102))
    dot = lambda u, v: (u.view(NRHS, -1) * v.view(NRHS, -1)).sum(1)
    times = lambda a, u: (a[:, None] * u.view(NRHS, -1)).view(-1)
    x, r, p, q = torch.zeros_like(b.data), b.data.clone(), b.data.clone(), h.field(M.F64, NRHS, 0)
    rho = dot(r, r)
    for it in (1, 2):
        h.mdagm(q, M.Field(p, None, M.F64, NRHS, 0))
        torch.cuda.synchronize()
        alpha = rho / dot(p, q.data)
        x = x + times(alpha, p)
        r = r - times(alpha, q.data)
        rho, old = dot(r, r), rho
        p = r + times(rho / old, p)
        got = h.field(M.F64, NRHS, 0)
        torch.cuda.synchronize()
        st = h.cg_solve(got, b, tol=1e-10, max_iter=it)
        assert st["outer_iters"] == it
        err = (got.data - x).view(NRHS, -1).norm(dim=1) / x.view(NRHS, -1).norm(dim=1)
        assert float(err.max()) <= 1e-11, (it, float(err.max()))
