"""The profile kernels at the sizes where their routes change: equal-count edges of one wavefront, one value per
lane, more values than lanes; tables whose cells do and do not fit in LDS."""
import numpy as np
import pytest
import torch

import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 2, 63, 64, 65, 511, 512, 513, 1023, 1024, 1025, 2048, 8191, 8192])
def test_edges_at_every_size_class(n):
    P = H.sv()
    rng = np.random.default_rng(n)
    for kind in range(3):
        v = rng.random(n).astype(np.float32)
        if kind == 1:
            v = np.round(v * 8) / 8                     # ties, zeros and ones
        if kind == 2 and n:
            v[rng.random(n) < 0.3] = np.nan
            v[0] = np.inf
        v = v.astype(np.float32)
        for bins in (1, 7, 100):
            out = torch.full((bins + 1,), -3.0, dtype=torch.float32, device="cuda")
            P.sv_quantile_edges(H.dev(v, torch.float32), bins, 0.0, 1.0, out)
            s = np.sort(v[~np.isnan(v)])
            ref = np.zeros(bins + 1, dtype=np.float32)
            for j in range(1, bins):
                ref[j] = s[(j * len(s)) // bins] if len(s) else 0.0
            ref[bins] = 1.0
            assert np.array_equal(out.cpu().numpy(), ref), (n, kind, bins)


@pytest.mark.parametrize("n_s,n_a,n_x", [(1, 1, 1), (1, 1, 1024), (64, 64, 3), (64, 65, 3), (10, 10, 10)])
def test_finalize_with_cells_in_and_beyond_lds(n_s, n_a, n_x):
    P = H.sv()
    rng = np.random.default_rng(n_s * n_a + n_x)
    counts = rng.integers(0, 50, size=(n_s, n_a, n_x)).astype(np.int64)
    counts[rng.random((n_s, n_a)) < 0.2] = 0
    big = np.minimum(counts * 90_000_000, 2 ** 32 - 1)   # a cell's total beyond 32 bits
    for cnt in (counts, big, np.zeros_like(counts)):
        cell = cnt.sum(-1).astype(np.float64)
        sums = cell * rng.random((n_s, n_a))
        table = torch.empty((n_s, n_a), dtype=torch.float32, device="cuda")
        info = torch.empty(3, dtype=torch.float64, device="cuda")
        P.sv_profile_finalize(torch.from_numpy(cnt.astype(np.uint32).view(np.int32)).cuda(), H.dev(sums), table, info)
        N = cell.sum()
        glob = sums.sum() / N if N else 0.0
        ref = np.where(cell > 0, sums / np.maximum(cell, 1), glob)
        plogp = lambda p: np.where(p > 0, -p * np.log2(np.maximum(p, 1e-300)), 0.0)
        h_x = plogp(cnt.sum((0, 1)) / N).sum() if N else 0.0
        h_c = (cell / max(N, 1) * plogp(cnt / np.maximum(cell, 1)[..., None]).sum(-1)).sum()
        np.testing.assert_allclose(table.cpu().numpy(), ref, rtol=2e-7, atol=0)          # one fp32 rounding
        np.testing.assert_allclose(info.cpu().numpy(), [h_x, h_c, h_x - h_c], rtol=1e-12, atol=1e-12)
