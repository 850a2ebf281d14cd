"""FP16 hops whose link products run on the matrix cores (Ls a multiple of four)
or in the vector units (other Ls), on every exchange and with idle lanes,
partial waves and several right-hand sides: the hop and A against the FP64 CPU
oracle within the per-application bound of FP16 storage.
"""
import pytest

import oracle as O
from paper_1811_08488_amd import mspcg as M
from tests.gpu_util import SITE_TOL, Setup, require_gpu, rounded, site_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ls,nrhs", [(4, 1), (4, 3), (5, 1), (6, 2), (8, 1), (10, 3), (12, 1), (12, 5), (16, 3),
                                     (20, 1), (24, 3), (28, 1), (32, 2)])
@pytest.mark.parametrize("dagger", [0, 1])
def test_f16_hop_every_width(Ls, nrhs, dagger):
    require_gpu()
    S = Setup((4, 2, 6, 4), Ls, "mobius", mf=0.05, seed=81)
    x = S.rand(nrhs, 82)
    fout = S.h.field(M.F16, nrhs, dagger)
    S.h.dslash_eo(fout, S.h.upload(x, 1 - dagger, M.F16), dagger)
    got, xr = S.h.download(fout), rounded(S.h, x, 1 - dagger, M.F16)
    for r in range(nrhs):
        want = O.dslash_eo(S.oa, S.U, xr[r], dagger, dagger)
        assert site_err(got[r], want) <= SITE_TOL[M.F16], (Ls, nrhs, r, site_err(got[r], want))
