"""The sampling stage at the edges of its 4096-entry granules: vocabularies around one lane's run,
a granule and a chunk, more granules than a wavefront has lanes, all mass in one granule, and a
residual without mass, for which the granules of the target row are summed on the spot."""
import numpy as np
import pytest
import torch

import svgen

import harness as H

pytestmark = pytest.mark.gpu


def _check(z_t, z_d, x, k, seeds, fallback=False):
    n_t, n_d = svgen.to_numpy_bits(z_t), svgen.to_numpy_bits(z_d)
    seen = set()
    for seed in seeds:
        ref = H.oracle_verify(n_t, n_d, x.numpy(), seed=seed, step=3)
        got = H.gpu_verify(z_t.cuda(), z_d.cuda(), x.cuda(), seed=seed, step=3)
        H.assert_verify(got, ref, k)
        if fallback:
            assert (got["flags"] & H.O.FLAG_RESIDUAL_FALLBACK).all()
        seen |= {int(t) // 4096 for row in got["tokens"] for t in row if t >= 0}
    return seen


@pytest.mark.parametrize("V,dtype", [(1, "f32"), (15, "bf16"), (17, "f32"), (4095, "bf16"), (4096, "f32"), (4097, "bf16"),
                                     (8193, "f32"), (12288, "bf16"), (12305, "bf16"), (270001, "bf16"), (300000, "f32")])
def test_vocabularies_around_a_granule(V, dtype):
    cfg = svgen.make_config(1, seed=V + 1, B=4, k=2, V=V, dtype=dtype)
    _check(cfg["z_t"], cfg["z_d"], cfg["x"], 2, range(6))


@pytest.mark.parametrize("lo,hi", [(0, 3), (4095, 4097), (8190, 8192), (40000, 40009)])
def test_all_mass_in_a_few_entries(lo, hi):
    """Target mass on entries lo..hi-1 only (the last granule is a partial one)."""
    V = 40009
    cfg = svgen.make_config(1, seed=77, B=6, k=2, V=V, dtype="f32")
    z_t = cfg["z_t"]
    z_t[:, :, :lo] = -np.inf
    z_t[:, :, hi:] = -np.inf
    seen = _check(z_t, cfg["z_d"], cfg["x"], 2, range(4))
    assert {lo // 4096, (hi - 1) // 4096} >= seen - {int(t) // 4096 for t in cfg["x"].reshape(-1)}


@pytest.mark.parametrize("V,dtype", [(20, "f32"), (9001, "bf16"), (30000, "f32"), (270001, "bf16")])
def test_residual_without_mass(V, dtype):
    """Equal rows, and the drafted token at -inf in both (ratio 0/0, rejected): the residual is empty."""
    cfg = svgen.make_config(1, seed=V, B=4, k=1, V=V, dtype=dtype)
    z_t = cfg["z_t"]
    x = cfg["x"]
    for b in range(4):
        z_t[b, 0, int(x[b, 0])] = -np.inf
    z_d = z_t[:, :1].clone()
    seen = _check(z_t, z_d, x, 1, range(6), fallback=True)
    assert V < 9000 or len(seen) > 1


@pytest.mark.parametrize("offset", [0.0, 600.0, -700.0, 708.0, 712.0, -712.0, 5000.0, 1e6])
def test_probabilities_on_either_side_of_the_short_form(offset):
    """The short form of the probabilities holds while |log2 of the normaliser| < 1024 (logits near 710);
    residuals of nearly equal rows, whose mass is what both forms have to leave unbiased."""
    V = 9001
    cfg = svgen.make_config(1, seed=int(abs(offset)) + 5, B=6, k=2, V=V, dtype="f32")
    z_t = cfg["z_t"] + offset
    z_d = z_t[:, :2] + 0.05 * torch.randn(z_t[:, :2].shape, generator=torch.Generator().manual_seed(3))
    _check(z_t, z_d.contiguous(), cfg["x"], 2, range(8))
