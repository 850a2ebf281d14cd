"""Conversions, M_5^{-1} and the block kernels at fifth dimensions on both sides of the rules that choose
their stores (rows of Ls x 16 bytes that are whole 128-byte lines, whole 64-byte
segments, or neither; lanes that hold whole sites or are packed).

Conversions: FP64 and FP32 copies are exact, F16 and BF16 round each real to half a
unit in the last place of its site's largest (2^-11, 2^-8, a quarter more for the
reciprocal scale).  M_5^{-1}: the FP64 CPU oracle within the per-application bound.
The rate: a conversion moves its bytes in at most 1.7 times the time of a torch copy of
as many (stores of partial lines took 2.9 times as long as ordinary ones at Ls = 2, and
1.9 times at 5).
"""
import numpy as np
import pytest

import oracle as O
from paper_1811_08488_amd import mspcg as M
from tests.gpu_util import PNAME, PRECS, SITE_TOL, Setup, require_gpu, rounded, site_err

pytestmark = pytest.mark.gpu

ROWS = [(2, 1), (3, 1), (4, 1), (5, 2), (7, 1), (8, 1), (11, 1), (12, 1), (13, 3), (14, 1), (18, 1), (20, 1), (24, 1)]
ROUND = {M.F64: 0, M.F32: 2.0**-24, M.F16: 1.25 * 2.0**-11, M.BF16: 1.25 * 2.0**-8}


@pytest.mark.parametrize("Ls,nrhs", ROWS)
def test_conversions_and_m5inv_every_row(Ls, nrhs):
    require_gpu()
    S = Setup((4, 2, 6, 4), Ls, "mobius", mf=0.05, seed=121)
    x = S.rand(nrhs, 122)
    most = np.abs(x.view(np.float64)).reshape(*x.shape[:3], 24).max(-1)[..., None, None]
    f = {p: S.h.upload(x, 1, p) for p in PRECS}
    for a in PRECS:
        for b in PRECS:
            g = S.h.field(b, nrhs, 1)
            S.h.convert(g, f[a])
            err = np.abs(S.h.download(g) - x)
            assert np.all(err <= 1.5 * (ROUND[a] + ROUND[b]) * most), (PNAME[a], PNAME[b])
    for p in PRECS:
        xr, out = rounded(S.h, x, 1, p), S.h.field(p, nrhs, 1)
        for dagger in (0, 1):
            S.h.m5inv(out, f[p], dagger)
            got = S.h.download(out)
            for r in {0, nrhs - 1}:
                want = O.op5(S.oa, xr[r], O.M5INV_DAG if dagger else O.M5INV, 1)
                assert site_err(got[r], want) <= SITE_TOL[p], (PNAME[p], dagger)


def time(torch, f):
    """Median time of ten calls."""
    f()
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    out = []
    for _ in range(7):
        e[0].record()
        for _ in range(10):
            f()
        e[1].record()
        torch.cuda.synchronize()
        out.append(e[0].elapsed_time(e[1]))
    return sorted(out)[3]


def big_handle(Ls):
    A = M.Action((24, 24, 24, 48), Ls, M5=1.8, mf=0.05, b=1.5, c=0.5)
    return M.Handle(A, np.broadcast_to(np.eye(3, dtype=np.complex128), (A.V, 4, 3, 3)))


@pytest.mark.parametrize("Ls", [2, 5, 24])
def test_conversion_rate(Ls):
    torch = require_gpu()
    h = big_handle(Ls)
    a, b = h.field(M.F64, 1, 0), h.field(M.F64, 1, 0)
    assert time(torch, lambda: h.convert(b, a)) <= 1.7 * time(torch, lambda: b.data.copy_(a.data))


def test_block_gather_and_scatter_rate():
    """Without inner iterations the preconditioner gathers and scatters: per 5D site at
    most 1.55 times the time at Ls = 16 (1.2 to 1.3; stores of partial lines 1.7 to 2.2)."""
    torch = require_gpu()
    per_site = {}
    for Ls in (2, 5, 16):
        h = big_handle(Ls)
        r, z = h.field(M.F64, 1, 0), h.field(M.F64, 1, 0)
        r.data.normal_()
        per_site[Ls] = time(torch, lambda: h.local_block_cg(z, r, (2, 2, 2, 2), 0, M.F32)) / Ls
    assert per_site[2] <= 1.55 * per_site[16] and per_site[5] <= 1.55 * per_site[16], per_site
