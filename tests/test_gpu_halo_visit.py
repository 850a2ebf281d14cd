"""The halo layers of the first two block hops, which are visited by the side of
the block they lie on and whose waves do the directions that lie inside only:
blocks one site thick (a wave's sites have neighbours on both sides), sides
larger and smaller than a wave, uneven splits and several right-hand sides,
against the FP64 CPU oracle.  Bounds: the per-application bound of the storage
type for each of the four stored hops.
"""
import numpy as np
import pytest

import oracle as O
from paper_1811_08488_amd import mspcg as M
from tests.gpu_util import PNAME, PRECS, SITE_TOL, Setup, require_gpu, rounded, site_err

pytestmark = pytest.mark.gpu

# (L, nblk, Ls, nrhs)
CASES = {"one_thick_ls8": ((6, 4, 4, 10), (6, 1, 1, 2), 8, 1), "two_thick_ls16": ((6, 6, 4, 4), (3, 3, 1, 1), 16, 1),
         "wide_sides_ls12": ((8, 4, 8, 12), (2, 1, 1, 1), 12, 1), "uneven_ls5_rhs3": ((10, 4, 2, 8), (3, 1, 1, 2), 5, 3),
         "ls20_rhs2": ((4, 4, 4, 10), (1, 1, 1, 2), 20, 2)}


@pytest.mark.parametrize("prec", PRECS, ids=lambda p: PNAME[p])
@pytest.mark.parametrize("case", list(CASES), ids=list(CASES))
def test_block_apply_halo_layers(case, prec):
    require_gpu()
    L, nblk, Ls, nrhs = CASES[case]
    S = Setup(L, Ls, "mobius", mf=0.05, seed=61)
    x = S.rand(nrhs, 62)
    fout = S.h.field(M.F64, nrhs, 0)
    S.h.block_apply(fout, S.h.upload(x, 0), nblk, prec)
    got, xr = S.h.download(fout), rounded(S.h, x, 0, prec)
    for r in range(nrhs):
        want = sum(O.block_op(S.oa, S.U, xr[r], nblk, b) for b in range(int(np.prod(nblk))))
        assert site_err(got[r], want) <= 4 * SITE_TOL[prec], (case, PNAME[prec], r, site_err(got[r], want))
