"""The draw of short rows, one workgroup per sequence: rows that end at, before and past every size of its kernel and its
runs, on and off eight entries, as many sequences as each form takes and one more; the token in the last entries and in
the first; residuals without mass, and rows without any."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O

import harness as H

pytestmark = pytest.mark.gpu

SIZES = [(7, 3), (8, 3), (9, 40), (15, 5), (511, 9), (513, 9), (4095, 12), (4096, 33), (4097, 12), (8191, 9), (8192, 5), (8193, 40),
         (16383, 6), (16384, 6), (16385, 32), (16385, 33), (20003, 34), (32767, 33), (32768, 34), (32769, 33), (1003, 513), (17001, 383), (17001, 384), (16391, 513)]
# the most sequences that a length is drawn at once for, and one more
SIZES += [(2001, 2048), (2001, 2049), (4097, 1280), (4097, 1281), (17001, 1), (17001, 2), (17001, 256), (17001, 257), (25001, 257), (9001, 1025)]


@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,B", SIZES)
def test_the_token_of_short_rows(V, B, dtype, chained):
    n, k = min(B, 9), 2                                  # a few different sequences, in turn
    cfg = svgen.make_config(1, seed=V + B, B=n, k=k, V=V, dtype=dtype)
    z_t, z_d, x = cfg["z_t"], cfg["z_d"], cfg["x"]
    for i in range(k + 1):                               # nearly all of the mass at one end of the row
        z_t[0, i, V - 1] = 20.0
        z_t[1 % n, i, 0] = 20.0
        z_t[2 % n, i, V - 1 - V % 8] = 20.0
    if n > 3:                                            # equal rows, the drafted token in neither: no residual
        z_t[3, 0, int(x[3, 0])] = float("-inf")
        z_d[3, 0] = z_t[3, 0]
    if n > 4:
        z_t[4, :] = float("-inf")                        # nothing to draw from
    at = torch.arange(B) % n
    z_t, z_d, x = z_t[at].contiguous(), z_d[at].contiguous(), x[at].contiguous()
    ref = H.oracle_verify(svgen.to_numpy_bits(z_t), svgen.to_numpy_bits(z_d), x.numpy(), seed=V, step=2)
    if chained:
        got = H.gpu_verify_chained(z_t.cuda(), z_d.cuda(), z_d.cuda(), x.cuda(), seed=V, step=2)
    else:
        got = H.gpu_verify(z_t.cuda(), z_d.cuda(), x.cuda(), seed=V, step=2)
    ties, edges = H.assert_verify(got, ref, k)
    assert ties + edges <= max(2, B // 8) + (B + n - 1) // n           # (the sequences without residual count as unresolved)
    if n > 4:
        assert (got["flags"][4::n] & O.FLAG_BAD_ROW).all()
