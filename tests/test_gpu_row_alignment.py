"""Rows that start on any element: vocabularies around whole vectors and around the
workgroup-wide steps of the sweeps, and tensors whose first row is off a 16-byte boundary."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O

import harness as H
from test_gpu_warp import _compare

pytestmark = pytest.mark.gpu


def _shifted(t, n):
    """A contiguous device copy of t that starts n elements into its allocation."""
    flat = torch.zeros(t.numel() + n, dtype=t.dtype, device="cuda")
    flat[n:] = t.reshape(-1).cuda()
    return flat[n:].reshape(t.shape)


@pytest.mark.parametrize("V,dtype,shift", [(7, "bf16", 1), (8, "bf16", 3), (9, "bf16", 0), (5, "f32", 1), (4095, "bf16", 0),
                                           (4097, "f32", 2), (8191, "bf16", 1), (8192, "bf16", 1), (8200, "bf16", 5),
                                           (32001, "bf16", 0), (20001, "f32", 0), (50003, "bf16", 7)])
def test_rows_on_any_element(V, dtype, shift):
    B, k = 3, 3
    cfg = svgen.make_config(1, seed=V, B=B, k=k, V=V, dtype=dtype)
    n = H.oracle_inputs(cfg)
    z_t, z_d, z_c = (_shifted(cfg[name], shift) for name in ("z_t", "z_d", "z_c"))
    x = cfg["x"].cuda()
    H.assert_row_stats(H.gpu_row_stats(z_d, z_c, x), O.row_stats(n["z_d"], n["z_c"], n["x"]))
    for seed in range(3):
        ref = H.oracle_verify(n["z_t"], n["z_d"], n["x"], seed=seed, step=1)
        H.assert_verify(H.gpu_verify(z_t, z_d, x, seed=seed, step=1), ref, k)
        H.assert_verify(H.gpu_verify_chained(z_t, z_d, z_c, x, seed=seed, step=1), ref, k)
    for T, K, Pp in ((0.7, 20, 0.8), (0.9, 0, 0.7)):
        _compare(z_t, T, K, Pp)
    # the largest entry behind the last whole vector
    z_t[:, :, V - 1] = 40.0
    _compare(z_t, 0.7, 5, 0.9)
    assert np.isfinite(H.gpu_row_stats(z_d, z_c, x)["S"]).all()
