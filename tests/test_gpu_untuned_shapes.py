"""The workgroup shapes that hops get without the tuner, at the fifth dimensions
whose full workgroups hold the most sites: the links and exchange rows of a
workgroup have to fit the LDS in every variant.  Against the FP64 CPU oracle,
within the per-application bound of the storage type for each stored hop.
"""
import numpy as np
import pytest

import oracle as O
from paper_1811_08488_amd import mspcg as M
from tests import lattice_helpers as H
from tests.gpu_util import PNAME, PRECS, SITE_TOL, Setup, require_gpu, rounded, site_err

pytestmark = pytest.mark.gpu

L = (4, 4, 4, 8)
SHAPES = [(2, 1), (2, 2), (2, 16), (3, 1), (4, 1), (5, 2)]  # (Ls, nrhs)


@pytest.fixture(scope="module", params=SHAPES, ids=lambda p: "ls%d_rhs%d" % p)
def S(request):
    require_gpu()
    with pytest.MonkeyPatch.context() as mp:
        mp.setenv("MSPCG_AUTOTUNE", "0")
        s = Setup(L, request.param[0], "mobius", mf=0.05, seed=91)
    s.nrhs = request.param[1]
    return s


@pytest.mark.parametrize("prec", PRECS, ids=lambda p: PNAME[p])
def test_operators_without_the_tuner(S, prec):
    n, x = S.nrhs, S.rand(S.nrhs, 92)
    fx = S.h.upload(x, 0, prec)
    xr = rounded(S.h, x, 0, prec)
    odd, out, noalloc = S.h.field(prec, n, 1), S.h.field(prec, n, 0), S.h.field(prec, n, 0)
    S.h.dslash_eo(odd, fx, 0)
    S.h.mdagm(out, fx)
    S.h.mdagm_noalloc(noalloc, fx)
    got_odd, got = S.h.download(odd), S.h.download(out)
    assert np.array_equal(got, S.h.download(noalloc))
    for r in {0, n - 1}:
        assert site_err(got_odd[r], O.dslash_eo(S.oa, S.U, xr[r], 1, 0)) <= SITE_TOL[prec]
        assert site_err(got[r], O.mdagm(S.oa, S.U, xr[r])) <= 4 * SITE_TOL[prec]


def test_source_preparation_and_reconstruction_without_the_tuner(S):
    n = S.nrhs
    rng = np.random.default_rng(93)
    phi = [H.rand_c(rng, (2 * S.Vh, S.Ls, 4, 3)) for _ in range(n)]
    psi_e = S.rand(n, 94)
    phi_e = np.stack([H.full_to_cb(L, p, 0) for p in phi])
    phi_o = np.stack([H.full_to_cb(L, p, 1) for p in phi])
    b, psi_o = S.h.field(M.F64, n, 0), S.h.field(M.F64, n, 1)
    S.h.reconstruct(psi_o, S.h.upload(psi_e, 0), S.h.upload(phi_o, 1))
    S.h.prepare_rhs(b, S.h.upload(phi_e, 0), S.h.upload(phi_o, 1))
    got_b, got_o = S.h.download(b), S.h.download(psi_o)
    for r in {0, n - 1}:
        want_o = H.full_to_cb(L, O.reconstruct(S.oa, S.U, psi_e[r], phi[r]), 1)
        assert site_err(got_o[r], want_o) <= 2 * SITE_TOL[M.F64]
        assert site_err(got_b[r], O.prepare_rhs(S.oa, S.U, phi[r])[0]) <= 4 * SITE_TOL[M.F64]


@pytest.mark.parametrize("prec", PRECS, ids=lambda p: PNAME[p])
def test_block_operator_and_solves_without_the_tuner(S, prec):
    n, nblk, x = S.nrhs, (1, 1, 1, 2), S.rand(S.nrhs, 95)
    out = S.h.field(M.F64, n, 0)
    S.h.block_apply(out, S.h.upload(x, 0), nblk, prec)
    got, xr = S.h.download(out), rounded(S.h, x, 0, prec)
    want = sum(O.block_op(S.oa, S.U, xr[0], nblk, b) for b in range(2))
    assert site_err(got[0], want) <= 4 * SITE_TOL[prec]
    for kw in (None, dict(nblk=nblk, n_inner=2, inner_prec=prec)):
        sol = S.h.field(M.F64, n, 0)
        solve = S.h.cg_solve if kw is None else S.h.mspcg_solve
        st = solve(sol, S.h.upload(x, 0), tol=1e-8, **(kw or {}))
        assert st["status"] == M.OK and max(st["true_rel_resid"]) <= 1e-8
