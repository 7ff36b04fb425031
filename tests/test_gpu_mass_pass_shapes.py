"""sv_verify_sample on both sides of the lines between its ways to a token: the mass pass's two workgroup shapes (512 pairs of a
sequence and a granule of 4096 entries, 256 in bfloat16 with several granules to a row), and the one kernel that draws short rows at once.  What
one more sequence turns over must leave the others' results where they are, and both agree with the oracle."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O
from oracle import warp_oracle as W

import harness as H
from test_gpu_warped import _t32

pytestmark = pytest.mark.gpu


T_T, T_D, P_T, P_D = _t32(0.8), _t32(1.3), 0.9, 0.7         # temperatures and nuclei of the target and the draft


def _verify(cfg, B, chained, warped=False):
    P = H.sv()
    z_t, z_d, z_c, x = (cfg[n][:B].contiguous().cuda() for n in ("z_t", "z_d", "z_c", "x"))
    k, V = z_d.shape[1:]
    ws = P.alloc_workspace(B, k, V, P.binding._dtype_tag(z_d))
    f = lambda: torch.empty((B, k), dtype=torch.float32, device="cuda")
    tok = torch.empty((B, k + 1), dtype=torch.int32, device="cuda")
    n, fl = (torch.empty(B, dtype=torch.int32, device="cuda") for _ in range(2))
    if warped:
        cut_t, cut_d = (torch.empty(z.shape[:2], dtype=torch.float32, device="cuda") for z in (z_t, z_d))
        P.sv_warp_cutoffs(z_t, T_T, 0, P_T, cut_t)
        P.sv_warp_cutoffs(z_d, T_D, 0, P_D, cut_d)
        if chained:
            P.sv_row_stats_warped(z_d, z_c, x, T_D, cut_d, 1.0, None, f(), f(), f(), f(), None, None, ws)
        (P.sv_verify_sample_warped_chained if chained else P.sv_verify_sample_warped)(
            z_t, None, z_d, x, None, T_T, cut_t, T_D, cut_d, 11, 3, tok, n, fl, None, ws)
        return tok.cpu().numpy(), n.cpu().numpy(), fl.cpu().numpy()
    if chained:
        P.sv_row_stats(z_d, z_c, x, f(), f(), f(), f(), None, None, ws)
    (P.sv_verify_sample_chained if chained else P.sv_verify_sample)(z_t, None, z_d, x, None, 11, 3, tok, n, fl, None, ws)
    return tok.cpu().numpy(), n.cpu().numpy(), fl.cpu().numpy()


# (the mass pass: a granule to a workgroup, two, or what the one becomes with one sequence more)
MASS = [(28, 36000, "bf16"), (56, 36000, "f32"), (512, 7, "bf16"), (512, 7, "f32")]
# (one kernel on both sides, and on one side only)
DRAW = [(512, 4096, "bf16"), (512, 4001, "f32"), (256, 4097, "bf16"), (170, 8200, "f32"), (64, 32000, "bf16"),
                                       (128, 4097, "bf16"), (85, 8200, "bf16"), (32, 32000, "bf16"), (40, 17001, "bf16"), (40, 17001, "f32"), (400, 17001, "bf16"), (256, 17001, "f32"), (2048, 1999, "bf16"),
        (1280, 4099, "bf16"), (1024, 8201, "f32"), (512, 17001, "bf16")]


@pytest.mark.parametrize("B,V,dtype", MASS + DRAW)
@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("warped", [False, True])
def test_mass_pass_shapes_agree(B, V, dtype, chained, warped):
    k = 2
    cfg = svgen.make_config(1, seed=V, B=B + 1, k=k, V=V, dtype=dtype)
    wide, narrow = _verify(cfg, B, chained, warped), _verify(cfg, B + 1, chained, warped)
    near = ((wide[2] | narrow[2][:B]) & (2 | 16)) != 0          # a decision or an edge within rounding
    for a, b in zip(wide, narrow):
        np.testing.assert_array_equal(a[~near], b[:B][~near])
    assert near.mean() < 0.05
    inp = H.oracle_inputs({n: (v[:6] if torch.is_tensor(v) else v) for n, v in cfg.items()})
    if warped:
        inp["z_t"], inp["z_d"] = (W.warp_rows(inp[n], T, 0, P)[0] for n, T, P in (("z_t", T_T, P_T), ("z_d", T_D, P_D)))
    ref = O.verify_sample(inp["z_t"], inp["z_d"], inp["x"], seed=11, step=3, cdf_abs_band=H.GPU_CDF_ABS_BAND)
    for b in range(6):
        if not near[b]:
            assert wide[1][b] == ref["n_accept"][b]
            np.testing.assert_array_equal(wide[0][b], ref["tokens"][b])
