"""Cutoffs of bfloat16 rows from the counts of their values: rows that a workgroup holds in its registers (4, 8 or 16
vectors a lane) and rows read again from cache, at the edges of the counters and of those sizes, against the oracle."""
import numpy as np
import pytest
import torch

import harness as H
from test_gpu_deep_nucleus import _rows
from test_gpu_warp import _compare

pytestmark = pytest.mark.gpu


def _more_rows(V, seed):
    n = np.random.default_rng(seed).standard_normal((6, V))
    z = 3.0 * n
    z[1] = 1e-30 * n[1]                                       # every value shares a counter with zero
    z[2] = np.where(n[2] > 0.3, n[2], 0.0)                    # zeros at most cutoffs
    z[3] = 0.0
    z[3, : min(V, 3)] = 40.0                                  # far above the rest
    z[4] = -1e6 + 1e4 * n[4]
    z[5, 0] = np.nan
    return z


# 7 to 9: lists, however short; 65, 71: the shortest that are held; 16384, 32768, 65536: 4, 8, 16 vectors for every one of 512 lanes; odd ones: a row's first
# entries at any alignment and up to seven behind the last vector
@pytest.mark.parametrize("V", [7, 8, 9, 65, 71, 4097, 16384, 16391, 32768, 32769, 65536, 65541])
def test_against_the_oracle(V):
    ties = n = 0
    for z in (_rows(max(V, 4), V)[:, :V], _more_rows(V, V)):
        t = torch.from_numpy(z).to(torch.bfloat16)
        for T, K, Pp in ((0.7, 0, 0.9), (1.0, 0, 0.999), (50.0, 0, 0.4), (1.0, 513, 1.0), (1.0, 2000, 0.9), (0.3, 60000, 0.95)):
            ties += _compare(t, T, K, Pp)
            n += t.shape[0]
    assert ties <= n // 4, (ties, n)                          # (flat rows and the far tail sit within the band: test_gpu_deep_nucleus)


@pytest.mark.parametrize("V, rows", [(24576, 1627), (24577, 512), (32768, 512)])
def test_both_sides_of_the_line_agree(V, rows):
    """The most rows of a length that are held in registers, and one more: which are read again from cache."""
    P = H.sv()
    g = torch.Generator(device="cuda").manual_seed(V)
    z = (2.0 * torch.randn((rows + 1, V), generator=g, device="cuda")).to(torch.bfloat16)
    for T, Pp in ((0.8, 0.9), (0.3, 0.9)):
        out = []
        for n in (rows, rows + 1):
            cut, fl = torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
            P.sv_warp_cutoffs(z[:n], T, 0, Pp, cut, fl)
            out.append((cut[:rows], fl[:rows]))
        torch.cuda.synchronize()
        near = (out[0][1] | out[1][1]) != 0
        assert ((out[0][0] == out[1][0]) | near).all()
        assert int(near.sum()) <= rows // 20


# One value and 65534 equal ones, 10.6 to 11.6 T below it, about as heavy together; one entry out of the K largest.  P lies 2 to
# 4 % inside or outside the band of a near tie around the top value's share, and the fp32 exponent's rounding
# of the lower value, up to 5e-7 of its mass, is 4 to 10 % of that band: the masses have to be better than fp32.
EDGE = [(1.4409691095352173, 31.875, 15.625, 0.54656982421875, False), (1.4184449911117554, 24.375, 8.4375, 0.5363317728042603, False),
        (0.7103328704833984, 29.0, 21.0, 0.5428975224494934, True), (0.6587724089622498, 36.5, 29.0, 0.5730973482131958, True),
        (1.4334756135940552, 27.125, 11.4375, 0.46340182423591614, True), (0.7185483574867249, 16.625, 8.6875, 0.4890678822994232, True),
        (0.7185483574867249, 16.625, 8.6875, 0.4890618920326233, False), (1.4334756135940552, 27.125, 11.4375, 0.46340784430503845, False)]


@pytest.mark.parametrize("V", [65536, 65600])                 # held in registers, read again from cache
@pytest.mark.parametrize("T,top,low,Pp,near", EDGE)
def test_masses_of_the_counters_are_not_rounded_to_fp32(V, T, top, low, Pp, near):
    share = 1.0 / (1.0 + 65534 * np.exp((low - top) / T))
    assert (abs(share - Pp) < 3e-6) == near and abs(abs(share - Pp) - 3e-6) > 6e-8
    z = torch.full((1, V), -1e4)
    z[0, V - 65534:] = low
    z[0, 0] = top
    cut, fl = torch.zeros(1, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    H.sv().sv_warp_cutoffs(z.to(torch.bfloat16).cuda(), T, 65535, Pp, cut, fl)
    assert float(cut[0]) == (top if share >= Pp else low)
    assert bool(int(fl[0]) & 2) == near
