"""sv_row_stats at the edges of its workgroup shapes: as many pairs as compute units and one more,
rows that end inside, at and past the register share, the LDS share and the limits of the rule,
on and off 16 bytes, with and without the sums of KL and entropy."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O

import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs,V,dtype", [
    (257, 1, "f32"), (257, 4096, "bf16"),                       # less than a vector; one vector per lane
    (256, 8192, "bf16"), (256, 8200, "bf16"), (256, 8193, "bf16"),   # 1024 vectors and one more: wide from there on
    (257, 16384, "bf16"), (257, 29184, "bf16"), (257, 29192, "bf16"),   # three: registers full, LDS full, one over
    (3, 35840, "bf16"), (3, 35848, "bf16"), (2, 36001, "f32"),  # wide: LDS full, one over; off 16 bytes
    (257, 26000, "f32"), (257, 26004, "f32"),                   # three / two in float32
    (257, 104000, "bf16"), (257, 104008, "bf16"), (257, 104001, "bf16")])
@pytest.mark.parametrize("with_kl", [True, False])
def test_row_stats_at_the_edges_of_the_shapes(pairs, V, dtype, with_kl):
    # a few sequences' rows, repeated over the pairs: every workgroup of a launch has its turn
    n = min(pairs, 5)
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
