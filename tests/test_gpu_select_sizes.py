"""sv_select_length at the sizes where its sort changes: one wavefront, runs of one workgroup, the
step to merges by runs of two, four and eight values per lane, with list lengths that do not divide
them; distinct and tied products; latencies whose peak comes at once, midway, at the end."""
import numpy as np
import pytest

from oracle import sv_oracle as O

import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k", [(1, 1), (64, 1), (13, 5), (8, 8), (9, 7), (43, 3), (64, 8), (73, 7), (171, 3), (512, 1),
                                 (513, 1), (1, 1000), (128, 8), (205, 5), (1025, 1), (147, 7), (256, 8), (293, 7),
                                 (1, 3000), (4096, 1), (241, 17), (512, 16), (8192, 1), (1170, 7), (2, 4096)])
def test_selection_at_every_size_class(B, k):
    rng = np.random.default_rng(B * 10007 + k)
    n = B * k
    p_any = (0.3 + 0.7 * rng.random((B, k))).astype(np.float32)
    p_tied = rng.choice(np.float32([0.0, 0.25, 0.5, 0.5, 1.0, 1.0]), size=(B, k))
    p_odd = p_any.copy()
    p_odd.flat[::5] = [np.nan, 1.5, -0.25, 1.0, 0.0][n % 5]
    M = np.arange(n + 1)
    flat = np.ones(n + 1, dtype=np.float32)                                # the peak is at the last positive product
    ramp = (30.0 + 0.08 * M).astype(np.float32)
    steep = (1.0 + M.astype(np.float64) ** 2).astype(np.float32)           # the peak is at the first
    jump = ramp.copy()
    jump[n // 2 + 1:] += 1000.0                                            # a wall midway
    for p in (p_any, p_tied, p_odd):
        for lat in (flat, ramp, steep, jump):
            rg, ro, rm = O.select_length(p, lat)
            gg, go, gm = H.gpu_select_length(p, lat, O.MODE_BATCH_GREEDY)
            assert gm == rm and np.array_equal(gg, rg) and np.array_equal(go, ro), (B, k, rm, gm)
