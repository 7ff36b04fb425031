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


# 7: no whole vector; 16384, 32768, 65536: 4, 8, 16 vectors for every one of 512 lanes; odd ones: a row's first
# entries at any alignment and up to seven behind the last vector
@pytest.mark.parametrize("V", [7, 8, 9, 4097, 16384, 16391, 32768, 32769, 65536, 65541])
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
