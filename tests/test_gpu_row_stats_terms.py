"""sv_row_stats of short rows, whose exponentials stay in registers: rows that end at, before and past every number of places,
on and off 16 bytes, less than a wavefront's worth included; a pair per workgroup, several, a workgroup with one pair less,
more pairs than workgroups have records for; bad rows, and rows whose lanes start far below the maximum."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O
from oracle import warp_oracle as W

import harness as H
from test_gpu_warped import _cut32, _gpu_row_stats_warped, _t32

pytestmark = pytest.mark.gpu

# 512 lanes of 8 bf16 or 4 fp32 entries: a place is 4096 or 2048 entries
ROWS = [(8, "bf16"), (9, "bf16"), (511, "bf16"), (513, "bf16")]
ROWS += [(p * 4096 + d, "bf16") for p in (1, 2, 4, 6, 8) for d in (-7, 0, 1)] + [(7 * 4096 + 520, "bf16"), (10 * 4096, "bf16"),
                                                                              (10 * 4096 + 1, "bf16"), (12 * 4096, "bf16"), (12 * 4096 + 3, "bf16")]
ROWS += [(3 * 4096 + d, "bf16") for d in (-7, 0, 1)]
ROWS += [(4, "f32"), (5, "f32"), (255, "f32")]
ROWS += [(p * 2048 + d, "f32") for p in (1, 2, 4, 7, 8, 12) for d in (-3, 0, 1)] + [(16 * 2048 + 1, "f32"), (20 * 2048, "f32"), (20 * 2048 + 1, "f32")]


def _pairs(V, dtype, n=7):
    """Logits of n pairs: ordinary rows and rows that strain the sums."""
    cfg = svgen.make_config(1, seed=V, B=n, k=1, V=V, dtype=dtype)
    t = cfg["z_d"].dtype
    cfg["z_d"][2, 0, V // 3] = float("nan")
    cfg["z_c"][3, 0, V - 1] = float("inf")
    cfg["z_d"][4, 0, : V // 2] = float("-inf")
    cfg["z_c"][4, 0, V - 1] = -1e30
    ramp = torch.linspace(-300.0, 60.0, V)               # every lane begins 2^-500 below the maximum
    cfg["z_d"][5, 0] = ramp.to(t)
    cfg["z_c"][5, 0] = (ramp.flip(0) * 0.25).to(t)
    cfg["z_c"][6, 0] = cfg["z_d"][6, 0]
    return cfg


@pytest.mark.parametrize("V,dtype", ROWS)
@pytest.mark.parametrize("pairs", [3, 256, 257, 600, 1100])
def test_rows_whose_terms_stay_in_registers(V, dtype, pairs):
    cfg = _pairs(V, dtype)
    n = cfg["x"].shape[0]
    inp = H.oracle_inputs(cfg)
    at = np.arange(pairs) % n
    t = torch.from_numpy(at)
    z_d, z_c, x = cfg["z_d"][t].cuda(), cfg["z_c"][t].cuda(), cfg["x"][t].cuda()
    ref = O.row_stats(inp["z_d"], inp["z_c"], inp["x"])
    got = H.gpu_row_stats(z_d, z_c, x, with_kl=False)
    H.assert_row_stats(got, {name: np.asarray(v)[at] for name, v in ref.items()}, with_kl=False)
    same = slice(0, min(pairs, n))
    for name, v in got.items():                          # a pair's results do not depend on whose turn it was
        if v is not None:
            v = np.asarray(v).reshape(pairs, -1)
            np.testing.assert_array_equal(v, v[same][at], err_msg=name)
    if V < 64:
        return
    ok = [0, 1, 4, 5, 6]                                 # (the oracle warps finite rows)
    T = _t32(0.7)
    y_d, cut_d, _ = W.warp_rows(inp["z_d"][ok], T, 0, 0.9)
    y_c, cut_c, _ = W.warp_rows(inp["z_c"][ok], T, 40, 1.0)
    at = np.arange(pairs) % len(ok)
    t = torch.from_numpy(np.asarray(ok)[at])
    ref = O.row_stats(y_d, y_c, inp["x"][ok])
    got = _gpu_row_stats_warped(cfg["z_d"][t].cuda(), cfg["z_c"][t].cuda(), cfg["x"][t].cuda(), T, _cut32(np.asarray(cut_d)[at]), T,
                                _cut32(np.asarray(cut_c)[at]), with_kl=False)
    H.assert_row_stats(got, {name: np.asarray(v)[at] for name, v in ref.items()}, with_kl=False)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_more_pairs_than_the_workgroups_hold_records_for(dtype):
    V, n, pairs = 24, 6, 400000                          # 512 records for each of 256 to 768 workgroups
    cfg = svgen.make_config(1, seed=5, B=n, k=1, V=V, dtype=dtype)
    inp = H.oracle_inputs(cfg)
    ref = O.row_stats(inp["z_d"], inp["z_c"], inp["x"])
    at = np.arange(pairs) % n
    t = torch.from_numpy(at)
    got = H.gpu_row_stats(cfg["z_d"][t].cuda(), cfg["z_c"][t].cuda(), cfg["x"][t].cuda(), with_kl=False)
    H.assert_row_stats(got, {name: np.asarray(v)[at] for name, v in ref.items()}, with_kl=False)
