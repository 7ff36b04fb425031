"""sv_row_stats where a workgroup walks through several pairs: one pair for every workgroup of the chip, one
more, several rounds; rows that end at, one vector before and one past the ends of the register share and of the
LDS share of every shape, on and off 16 bytes, bad rows among good ones, with and without KL and entropy."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O

import harness as H

pytestmark = pytest.mark.gpu

# 512 lanes of 8 bf16 or 4 fp32 entries; register shares of 2, 4, 6, 8 places (4 more in LDS), of 12, 16, 24 (9 more)
ROWS = [(r * 512 + d, "bf16", 0) for r in (3, 5, 7, 11, 15) for d in (0, 1)]          # lines of the rule
ROWS += [(2 * 512, "bf16", 8 - 1), (6 * 512 - 1, "f32", 0), (6 * 512 + 1, "f32", 3), (10 * 512 + 1, "bf16", 0), (12 * 512, "bf16", 0),
         (12 * 512 + 1, "bf16", 5), (12 * 512, "f32", 0), (14 * 512 + 1, "f32", 0), (21 * 512 + 1, "f32", 0),
         (23 * 512 + 1, "bf16", 0), (33 * 512, "bf16", 1), (34 * 512 + 3, "f32", 0), (36 * 512 + 5, "bf16", 7)]


@pytest.mark.parametrize("vecs,dtype,extra", ROWS)
@pytest.mark.parametrize("pairs,with_kl", [(256, True), (257, False), (770, False), (1290, True)])
def test_row_stats_of_several_pairs_per_workgroup(vecs, dtype, extra, pairs, with_kl):
    V = vecs * (8 if dtype == "bf16" else 4) + extra
    if pairs > 770 and vecs > 6000:
        pairs = 420
    n = 7                                                # a few different pairs, in turn
    cfg = svgen.make_config(1, seed=V + pairs, B=n, k=1, V=V, dtype=dtype)
    cfg["z_d"][2, 0, 5] = float("nan")
    cfg["z_c"][4, 0, V - 1] = float("inf")
    cfg["z_d"][5, 0, : V // 2] = float("-inf")
    inp = H.oracle_inputs(cfg)
    ref = O.row_stats(inp["z_d"], inp["z_c"], inp["x"])
    at = np.arange(pairs) % n
    ref = {name: np.asarray(v)[at] for name, v in ref.items()}
    t = torch.from_numpy(at)
    got = H.gpu_row_stats(cfg["z_d"][t].cuda(), cfg["z_c"][t].cuda(), cfg["x"][t].cuda(), with_kl)
    H.assert_row_stats(got, ref, with_kl)
    for name, v in got.items():                          # a pair's results do not depend on whose turn it was
        if v is None:
            continue
        v = np.asarray(v).reshape(pairs, -1)
        np.testing.assert_array_equal(v, v[:n][at], err_msg=name)
