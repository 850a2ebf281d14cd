"""Spatial extents that the order of visit splits into halves (16 to 32, also
those whose half is odd) or leaves whole: the hop against the FP64 CPU oracle,
element by element, and the site map, which is a permutation of the lattice.
"""
import pytest

import oracle as O
from paper_1811_08488_amd import mspcg as M
from tests.gpu_util import SITE_TOL, Setup, require_gpu, site_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [(14, 2, 16, 2), (18, 4, 2, 4), (2, 20, 22, 2), (4, 2, 34, 2), (32, 2, 2, 2)],
                         ids=lambda L: "x".join(map(str, L)))
@pytest.mark.parametrize("parity", [0, 1])
def test_hop_on_split_extents(L, parity):
    require_gpu()
    S = Setup(L, 4, "mobius", mf=0.05, seed=71)
    x = S.rand(1, 72)
    fout = S.h.field(M.F64, 1, parity)
    S.h.dslash_eo(fout, S.h.upload(x, 1 - parity), 0)
    want = O.dslash_eo(S.oa, S.U, x[0], parity, 0)
    assert site_err(S.h.download(fout)[0], want) <= SITE_TOL[M.F64]
