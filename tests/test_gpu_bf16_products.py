"""BF16 hops without M_phi on the input, whose link products run on the matrix
cores (Ls a multiple of four) or in the vector units (other Ls): the daggered
hop on every exchange, with idle lanes, partial waves and several
sources, against the FP64 CPU oracle within the per-application bound of BF16
storage.
"""
import numpy as np
import pytest

import oracle as O
from paper_1811_08488_amd import mspcg as M
from tests.gpu_util import SITE_TOL, Setup, require_gpu, rounded, site_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ls,nrhs", [(4, 1), (4, 3), (5, 1), (6, 2), (8, 1), (10, 3), (12, 1), (12, 5), (16, 3),
                                     (20, 1), (24, 3), (28, 1), (32, 2)])
@pytest.mark.parametrize("parity", [0, 1])
def test_bf16_daggered_hop_every_width(Ls, nrhs, parity):
    require_gpu()
    S = Setup((4, 2, 6, 4), Ls, "mobius", mf=0.05, seed=91)
    x = S.rand(nrhs, 92)
    fout = S.h.field(M.BF16, nrhs, parity)
    S.h.dslash_eo(fout, S.h.upload(x, 1 - parity, M.BF16), 1)
    got, xr = S.h.download(fout), rounded(S.h, x, 1 - parity, M.BF16)
    for r in range(nrhs):
        want = O.dslash_eo(S.oa, S.U, xr[r], parity, 1)
        assert site_err(got[r], want) <= SITE_TOL[M.BF16], (Ls, nrhs, r, site_err(got[r], want))


def test_bf16_hop_wide_norm_range_and_zero_sites():
    """Slices of very different magnitude and an all-zero one keep their own accuracy."""
    require_gpu()
    Ls = 12
    S = Setup((4, 4, 2, 4), Ls, "shamir", mf=0.05, seed=93)  # (c = 0: no M_phi mixing of the slices)
    prof = 10.0 ** np.linspace(-15, 15, Ls)
    prof[Ls // 3] = 0.0
    x = S.rand(1, 94) * prof[None, None, :, None, None]
    fout = S.h.field(M.BF16, 1, 0)
    S.h.dslash_eo(fout, S.h.upload(x, 1, M.BF16), 1)
    got, want = S.h.download(fout)[0], O.dslash_eo(S.oa, S.U, rounded(S.h, x, 1, M.BF16)[0], 0, 1)
    for s in range(Ls):
        assert np.all(np.isfinite(got[:, s])) and site_err(got[:, s], want[:, s]) <= SITE_TOL[M.BF16], s
