"""The draw of short rows, one workgroup per sequence: rows that end at, before and past every size of its kernel and its
runs, on and off eight entries, as many sequences as each form takes and one more; the token in the last entries and in
the first; residuals without mass, and rows without any."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O

import harness as H
from test_gpu_sampling_granules import _check_nuclei

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


# the forms that weigh all of their runs at once and one at a time, the latter a second time for the token
@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("V,B,dtype", [(4001, 20, "bf16"), (8001, 20, "f32"), (12001, 20, "bf16"), (12001, 20, "f32"), (17001, 40, "bf16"), (17001, 40, "f32"),
                                       (17001, 385, "bf16"), (17001, 257, "f32"), (32768, 257, "bf16")])
def test_the_token_of_short_rows_under_cutoffs(V, B, dtype, chained):
    """Equal nuclei, which leave no residual, and nuclei of which the draft lacks a token."""
    _check_nuclei(V, torch.float32 if dtype == "f32" else torch.bfloat16, B, chained, range(1))


@pytest.mark.parametrize("V,B,dtype", [(4097, 40, "bf16"), (17001, 400, "bf16"), (17001, 300, "f32")])
def test_the_token_of_packed_target_rows(V, B, dtype):
    n, k = 9, 3
    cfg = svgen.make_config(1, seed=V, B=n, k=k, V=V, dtype=dtype)
    at = torch.arange(B) % n
    gamma = (at * 7 + torch.arange(B) // n) % (k + 1)                    # every length, the empty prefix included
    offs = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(gamma + 1, 0)]).int()
    packed = torch.cat([cfg["z_t"][a, : g + 1] for a, g in zip(at.tolist(), gamma.tolist())])
    z_d, x, gamma = cfg["z_d"][at].contiguous(), cfg["x"][at].contiguous(), gamma.int()
    got = H.gpu_verify(packed.cuda(), z_d.cuda(), x.cuda(), gamma=gamma, t_offsets=offs, seed=V, step=4)
    few = slice(0, 4 * n)                                # (the oracle on the first of them)
    ref = H.oracle_verify(svgen.to_numpy_bits(packed[: int(offs[4 * n])]), svgen.to_numpy_bits(z_d[few]), x[few].numpy(), gamma=gamma[few].numpy(),
                          t_offsets=offs[: 4 * n + 1].numpy(), seed=V, step=4)
    H.assert_verify({m: v[few] for m, v in got.items()}, ref, k)
    again = H.gpu_verify_chained(packed.cuda(), z_d.cuda(), z_d.cuda(), x.cuda(), gamma=gamma, t_offsets=offs, seed=V, step=4)
    near = ((got["flags"] | again["flags"]) & (O.FLAG_NEAR_TIE | O.FLAG_NEAR_CDF_EDGE)) != 0
    np.testing.assert_array_equal(got["tokens"][~near], again["tokens"][~near])
    # (at most V edges, each flagged 1e-6 W + 1e-6 to either side: 4e-6 V of the draws where W is 1; four standard deviations of B draws)
    share = 4e-6 * V
    assert near.mean() <= share + 4 * np.sqrt(share * (1 - share) / B) + 1 / B
