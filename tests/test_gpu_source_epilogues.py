"""Source preparation and reconstruction on every lane layout of the hop: the
sum with the source (and M_5^{-1}) in the hop's epilogue, against the FP64 CPU
oracle within the per-application bound of FP64 (1e-13) per stored stage, and
with an output that shares memory with an input.
"""
import numpy as np
import pytest

import oracle as O
from paper_1811_08488_amd import mspcg as M
from tests import lattice_helpers as H
from tests.gpu_util import Setup, rel, require_gpu, site_err

pytestmark = pytest.mark.gpu

# (L, Ls, nrhs): DPP, whole waves with idle lanes, LDS columns, an Ls that no chain is compiled for
CASES = {"dpp_ls16": ((4, 4, 4, 6), 16, 1), "wave_ls12": ((4, 4, 2, 6), 12, 1), "lds_ls24_rhs2": ((4, 4, 4, 4), 24, 2),
         "ls5_rhs3": ((6, 4, 2, 4), 5, 3)}


@pytest.mark.parametrize("case", list(CASES), ids=list(CASES))
def test_prepare_and_reconstruct_every_layout(case):
    require_gpu()
    L, Ls, nrhs = CASES[case]
    S = Setup(L, Ls, "mobius", mf=0.05, seed=41)
    rng = np.random.default_rng(42)
    V = int(np.prod(L))
    phi = [H.rand_c(rng, (V, Ls, 4, 3)) for _ in range(nrhs)]
    psi_e = np.stack([H.rand_c(rng, (V // 2, Ls, 4, 3)) for _ in range(nrhs)])
    phi_e = np.stack([H.full_to_cb(L, p, 0) for p in phi])
    phi_o = np.stack([H.full_to_cb(L, p, 1) for p in phi])
    b, psi_o = S.h.field(M.F64, nrhs, 0), S.h.field(M.F64, nrhs, 1)
    S.h.prepare_rhs(b, S.h.upload(phi_e, 0), S.h.upload(phi_o, 1))
    S.h.reconstruct(psi_o, S.h.upload(psi_e, 0), S.h.upload(phi_o, 1))
    got_b, got_o = S.h.download(b), S.h.download(psi_o)
    for r in range(nrhs):
        want_b, _ = O.prepare_rhs(S.oa, S.U, phi[r])
        want_o = H.full_to_cb(L, O.reconstruct(S.oa, S.U, psi_e[r], phi[r]), 1)
        assert rel(got_b[r], want_b) <= 1e-13 and site_err(got_b[r], want_b) <= 4e-13
        assert rel(got_o[r], want_o) <= 1e-13 and site_err(got_o[r], want_o) <= 2e-13
    # psi_o in the memory of phi_o, and of psi_e, on a handle that has tuned and on one that has not
    for h in (S.h, Setup(L, Ls, "mobius", mf=0.05, seed=41).h):
        f = h.upload(phi_o, 1)
        h.reconstruct(f, h.upload(psi_e, 0), f)
        assert np.array_equal(h.download(f), got_o)
        e = h.upload(psi_e, 0)
        o = M.Field(e.data, None, M.F64, nrhs, 1)
        h.reconstruct(o, e, h.upload(phi_o, 1))
        assert np.array_equal(h.download(o), got_o)
