"""sv_row_stats at the edges of its workgroup shapes: as many pairs as compute units and one more,
rows that end inside, at and past the register share, the LDS share and the limits of the rule,
on and off 16 bytes, with and without the sums of KL and entropy; and the error of the sums of flat rows."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O
from oracle import warp_oracle as W

import harness as H
from test_gpu_warped import _cut32, _gpu_row_stats_warped, _t32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs,V,dtype", [
    (257, 1, "f32"), (257, 4096, "bf16"),                       # less than a vector; one vector per lane
    (256, 8192, "bf16"), (256, 8200, "bf16"), (256, 8193, "bf16"),
    (257, 16384, "bf16"), (257, 29184, "bf16"), (257, 29192, "bf16"),
    (3, 35840, "bf16"), (3, 35848, "bf16"), (2, 36001, "f32"),
    (257, 26000, "f32"), (257, 26004, "f32"),
    (257, 104000, "bf16"), (257, 104008, "bf16"), (257, 104001, "bf16"),
    # three workgroups to a compute unit: registers full (3 or 4 vectors per lane) and one more, LDS full (1600) and one more,
    # the lines of the rule and one vector past them, off 16 bytes
    (1536, 1536 * 8, "bf16"), (1537, 1537 * 8, "bf16"), (1537, 2048 * 8, "bf16"), (1537, 2049 * 8 + 1, "bf16"),
    (1537, 3136 * 8, "bf16"), (1537, 3137 * 8, "bf16"), (1537, 3584 * 8, "bf16"), (1537, 3585 * 8 + 3, "bf16"),
    (4096, 3648 * 8, "bf16"), (4096, 3649 * 8 + 5, "bf16"), (4096, 4608 * 8, "bf16"), (4096, 4609 * 8, "bf16"),
    (1537, 1536 * 4, "f32"), (1537, 1537 * 4, "f32"), (1537, 2560 * 4, "f32"), (4096, 3648 * 4 + 1, "f32"), (4096, 4608 * 4, "f32"),
    (4096, 4609 * 4, "f32"), (300, 5632 * 4, "f32"), (300, 5633 * 4, "f32"), (300, 7169 * 4 + 2, "f32"), (300, 10240 * 4, "f32"),
    # two, whose registers (8 or 10 vectors per lane) and LDS (2432) are full far below the rows that take it
    (300, 10241 * 4, "f32"), (390, 10241 * 4 + 3, "f32"), (391, 10241 * 4, "f32"), (300, 24001 * 4, "f32"), (341, 24001 * 4, "f32"),
    (257, 20000 * 8, "bf16"), (257, 20001 * 8, "bf16"), (400, 20001 * 8 + 5, "bf16"), (401, 20001 * 8, "bf16"),
    # a pair per compute unit with 1024 lanes: its shortest rows, off 16 bytes, one pair more than it takes
    (128, 16896 * 8, "bf16"), (128, 16897 * 8, "bf16"), (3, 16897 * 8 + 1, "bf16"), (129, 16897 * 8, "bf16"), (96, 16896 * 4, "f32"),
    (96, 16897 * 4 + 1, "f32"), (97, 16897 * 4 + 1, "f32"), (128, 16897 * 4 + 1, "f32"), (2, 70001 * 4, "f32")])
@pytest.mark.parametrize("with_kl", [True, False])
def test_row_stats_at_the_edges_of_the_shapes(pairs, V, dtype, with_kl):
    # a few sequences' rows, repeated over the pairs: every workgroup of a launch has its turn
    n = min(pairs, 5 if V < 130000 else 3)
    cfg = svgen.make_config(1, seed=V + pairs, B=n, k=1, V=V, dtype=dtype)
    inp = H.oracle_inputs(cfg)
    ref = O.row_stats(inp["z_d"], inp["z_c"], inp["x"])
    at = np.arange(pairs) % n
    ref = {name: np.asarray(v)[at] for name, v in ref.items()}
    t = torch.from_numpy(at)
    got = H.gpu_row_stats(cfg["z_d"][t].cuda(), cfg["z_c"][t].cuda(), cfg["x"][t].cuda(), with_kl)
    H.assert_row_stats(got, ref, with_kl)


@pytest.mark.parametrize("with_kl", [True, False])
def test_the_sums_of_rows_off_16_bytes_do_not_drift(with_kl):
    """Equal terms round the same way in every lane, so the float32 sum of a lane drifts with the number of its
    additions.  Flat rows of this size over 512 lanes drift by 4.3e-6 entry by entry, by less than 1e-8 vector
    by vector, and by 1.3e-7 entry by entry over 1024 lanes (float32 additions replayed for every value the
    exponential can have here); S of a row with itself is 1."""
    V, pairs = 151869, 260
    z = torch.zeros((pairs, 1, V), dtype=torch.bfloat16, device="cuda")
    got = H.gpu_row_stats(z, z, torch.zeros((pairs, 1), dtype=torch.int32, device="cuda"), with_kl)
    # the drift, one rounding of the exponential (1.2e-7) and one of the result
    worst = float(np.abs(got["S"] - 1.0).max())
    assert worst < 4e-7


@pytest.mark.parametrize("V,dtype", [(1500 * 8, "bf16"), (3000 * 8, "bf16"), (3000 * 4 + 1, "f32"), (6001 * 4, "f32"), (9216 * 8, "bf16"), (16001 * 8, "bf16"),
                                     (9000 * 4, "f32"), (16897 * 8, "bf16"), (16897 * 4 + 1, "f32")])
@pytest.mark.parametrize("pairs", [100, 300, 770, 3072])
@pytest.mark.parametrize("with_kl", [True, False])
def test_warped_rows_in_every_shape(pairs, V, dtype, with_kl):
    """Neighbouring pairs have different cutoffs, the two rows different temperatures; 300 and 770 pairs are more than
    one for every workgroup that walks, one and two to a compute unit."""
    if pairs * V > 200_000_000:
        pairs = 512
    n = 5
    cfg = svgen.make_config(1, seed=V + pairs, B=n, k=1, V=V, dtype=dtype)
    inp = H.oracle_inputs(cfg)
    Td, Tc = _t32(0.7), _t32(1.4)
    warped, cuts = {}, {}
    for name, T, P in (("z_d", Td, (0.9, 0.5, 1.0, 0.99, 0.8)), ("z_c", Tc, (0.7, 1.0, 0.9, 0.6, 0.95))):
        rows = [W.warp_rows(inp[name][b:b + 1], T, 0, P[b]) for b in range(n)]
        warped[name], cuts[name] = np.concatenate([r[0] for r in rows]), np.concatenate([r[1] for r in rows])
    ref = O.row_stats(warped["z_d"], warped["z_c"], inp["x"])
    at = np.arange(pairs) % n
    t = torch.from_numpy(at)
    got = _gpu_row_stats_warped(cfg["z_d"][t].cuda(), cfg["z_c"][t].cuda(), cfg["x"][t].cuda(), Td, _cut32(cuts["z_d"][at]), Tc,
                                _cut32(cuts["z_c"][at]), with_kl)
    H.assert_row_stats(got, {name: np.asarray(v)[at] for name, v in ref.items()}, with_kl)
    for name, v in got.items():                          # a pair's results do not depend on whose turn it was
        if v is not None:
            np.testing.assert_array_equal(v, v[:n][at], err_msg=name)


@pytest.mark.parametrize("pairs,V,dtype,bound", [(200, 152064, "f32", 2.8e-7), (300, 152064, "f32", 2.8e-7), (200, 262144, "bf16", 2.4e-7),
                                                 (24, 1 << 20, "f32", 4.8e-7)])
def test_the_normalisers_of_flat_rows_do_not_drift(pairs, V, dtype, bound):
    """A flat row's terms are equal, and their float32 sums drift with the number of additions (one sum per lane and
    row over 512 lanes: 1.1e-6, 9.5e-7 and 5.2e-6 off here).  `bound` is the largest drift of sums that are put
    aside every 16 vectors, replayed in float32 for every value the terms can have."""
    z = torch.linspace(-300, 300, pairs).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    z = z.cuda().view(pairs, 1, 1).expand(pairs, 1, V).contiguous()
    got = H.gpu_row_stats(z, z, torch.zeros((pairs, 1), dtype=torch.int32, device="cuda"), False)
    # P_d(x) = 1 / V; beside the drift one rounding of the exponential (1.2e-7) and one of the result (6e-8)
    worst = float(np.abs(got["pd_x"].astype(np.float64) * V - 1.0).max())
    assert worst < bound + 1.8e-7, worst
