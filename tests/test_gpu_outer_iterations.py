"""The outer iterations of the FP64 solvers against the FP64 CPU oracle.

The second hop of A sums <p, A p>, the fourth updates the residual in place and
the solution is updated together with the search direction, so x is checked
after a few iterations, where an update that is late, lost or applied twice
shows (the iteration limit ends the solve between two updates).  Tolerance:
both sides run the same recurrence in FP64, whose rounding (1e-16 times the
few operator applications, of norm below 100) stays far below 1e-11 of a site.
"""
import numpy as np
import pytest

import oracle as O
from paper_1811_08488_amd import mspcg as M
from tests.gpu_util import Setup, require_gpu, site_err

pytestmark = pytest.mark.gpu

# one lattice per lane layout of the hops: (Ls, nrhs)
LAYOUTS = {"dpp_ls16": (16, 1), "wave_ls12": (12, 2), "lds_ls24": (24, 1), "bpermute_ls8_rhs3": (8, 3)}


@pytest.fixture(scope="module", params=list(LAYOUTS), ids=list(LAYOUTS))
def S(request):
    require_gpu()
    Ls, nrhs = LAYOUTS[request.param]
    s = Setup((4, 4, 2, 8), Ls, "mobius", mf=0.05, seed=31)
    s.nrhs = nrhs
    return s


@pytest.mark.parametrize("precond", [None, ((1, 1, 1, 2), 3)], ids=["cg", "mspcg"])
@pytest.mark.parametrize("iters,reliable", [(1, 0), (2, 0), (5, 2), (7, 0)])
def test_iterates_match_oracle(S, precond, iters, reliable):
    b = S.rand(S.nrhs, 400 + iters)
    fx = S.h.field(M.F64, S.nrhs, 0)
    if precond is None:
        st = S.h.cg_solve(fx, S.h.upload(b, 0), tol=1e-10, max_iter=iters, reliable=reliable)
        kw = {}
    else:
        nblk, k = precond
        st = S.h.mspcg_solve(fx, S.h.upload(b, 0), nblk, k, M.F64, tol=1e-10, max_iter=iters, reliable=reliable)
        kw = dict(nblk=nblk, k=k)
    x = S.h.download(fx)
    assert st["status"] == M.NOT_CONVERGED and st["outer_iters"] == iters
    for i in {0, S.nrhs - 1}:
        want, _ = O.solve(S.oa, S.U, b[i], tol=1e-10, maxiter=iters, reliable=reliable, **kw)
        assert site_err(x[i], want) <= 1e-11, (i, site_err(x[i], want))


@pytest.mark.parametrize("tol", [1e-1, 1e-4, 1e-10])
def test_running_ahead_changes_nothing(S, tol):
    """Far from convergence the host enqueues an iteration before it has seen
    the last one's residual; with the time split on it always waits.  Both
    stop at the same iteration with the same bits."""
    b = S.h.upload(S.rand(S.nrhs, 410), 0)
    runs = []
    for timing in (0, 1, 0):
        fx = S.h.field(M.F64, S.nrhs, 0)
        st = S.h.cg_solve(fx, b, tol=tol, timing=timing)
        assert st["status"] == M.OK
        runs.append((st["outer_iters"], S.h.download(fx)))
    for it, x in runs[1:]:
        assert it == runs[0][0] and np.array_equal(x, runs[0][1])


def test_sum_of_many_partials():
    """|b|^2-scaled quantities over more workgroups than one pass of the reduction takes
    (8192 partial sums): the reported residual of x = 0 is 1."""
    require_gpu()
    s = Setup((16, 16, 16, 16), 4, "mobius", mf=0.05, seed=32)
    b = s.rand(1, 420)
    fx = s.h.field(M.F64, 1, 0)
    st = s.h.cg_solve(fx, s.h.upload(b, 0), tol=1e-10, max_iter=3)
    x = s.h.download(fx)[0]
    want, _ = O.solve(s.oa, s.U, b[0], tol=1e-10, maxiter=3)
    assert st["outer_iters"] == 3 and site_err(x, want) <= 1e-11
