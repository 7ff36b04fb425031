"""Top-p cutoffs whose nucleus is deeper than any candidate list: found through mass bins that are
even in the exponent and the list of the one bin that holds the cutoff.  Against the oracle: the
kept set, row by row, at the edges of the bins, of the list and of the number range."""
import numpy as np
import pytest
import torch

import harness as H
from test_gpu_warp import _compare

pytestmark = pytest.mark.gpu


def _rows(V, seed):
    rng = np.random.default_rng(seed)
    n = rng.standard_normal((7, V))
    z = 3.0 * n
    z[1] = 2.0 * n[1] - 50.0                                  # all negative
    z[2] = 3e4 + 3.0 * n[2]                                   # far from zero (few distinct bfloat16 values)
    z[3] = np.round(n[3] * 4) / 4                             # groups of ties larger than a list
    z[4, V // 3:] = -np.inf                                   # masked vocabulary
    z[5] = np.where(rng.random(V) < 0.5, -1e30, 2.0 * n[5])   # a finite stand-in for -inf
    z[6] = np.linspace(-6.0, 6.0, V)                          # even density over every bin
    return z


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [2049, 4096, 20011, 131072])
def test_cutoffs_of_deep_nuclei(V, dtype):
    t = torch.from_numpy(_rows(V, V)).to(dtype)
    ties = n = 0
    for T, Pp in ((1.0, 0.9), (0.6, 0.95), (4.0, 0.5), (1.0, 0.9999), (30.0, 0.02), (1000.0, 0.8)):
        ties += _compare(t, T, 0, Pp)
        n += t.shape[0]
    # The flagged band spans 6e-6 of the mass: where the entries at the cutoff are no heavier, a
    # decision is flagged more often than not.  That is the rule for three of the six parameter
    # sets at V = 131072 (1 / V = 7.6e-6: T = 30 and 1000, nearly flat; P = 0.9999, the far tail).
    assert ties <= n // 2, (ties, n)


def test_cutoffs_and_supports_do_not_depend_on_the_route():
    """A support call (list first) and a cutoff call (bins where a list looks hopeless) agree on the
    cutoff of rows on either side of that line."""
    P = H.sv()
    V, cap = 9001, 64
    rng = np.random.default_rng(4)
    z = torch.from_numpy(rng.standard_normal((48, V)) * np.linspace(0.2, 6.0, 48)[:, None]).float().cuda()
    f32 = lambda: torch.full((48,), -3.0, dtype=torch.float32, device="cuda")
    c1, c2 = f32(), f32()
    fl1, fl2 = (torch.zeros(48, dtype=torch.int32, device="cuda") for _ in range(2))
    P.sv_warp_cutoffs(z, 1.0, 0, 0.9, c1, fl1)
    P.sv_warp_compact(z, 1.0, 0, 0.9, P.Supports(48, cap), c2, fl2)
    torch.cuda.synchronize()
    same = (c1 == c2) | ((fl1 | fl2) != 0)
    assert same.all() and (fl1 != 0).sum() <= 4
