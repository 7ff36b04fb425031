"""Top-p cutoffs whose nucleus is deeper than any candidate list: found through counts over equal
steps of the exponent and the list of the few steps that hold the cutoff.  Against the oracle: the
kept set, row by row, at the edges of the steps, of the list and of the number range; and the row
total that P is a share of."""
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


def _between_the_bounds(z, T, Pp, steps=8192):
    """Entries in the steps between which the kernel's bounds on the running mass place P: counts over equal steps of
    z / T, an entry's mass known to within its step."""
    depth = (z.max() - z) / T * np.log2(np.e)
    width = (np.log2(z.size / (1 - Pp)) + 1) / steps
    at = np.floor(depth / width)
    count = np.bincount(at[at < steps].astype(int), minlength=steps)
    upper = np.cumsum(count * np.exp2(-width * np.arange(steps)))
    target = Pp * np.exp2(-depth).sum()
    first, last = np.searchsorted(upper, target), min(np.searchsorted(upper, target * np.exp2(width)), steps - 1)
    return int(count[first:last + 1].sum())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [2049, 4096, 20011, 131072])
def test_cutoffs_of_deep_nuclei(V, dtype):
    t = torch.from_numpy(_rows(V, V)).to(dtype)
    ties = n = recounts = 0
    for T, Pp in ((1.0, 0.9), (0.6, 0.95), (4.0, 0.5), (1.0, 0.9999), (30.0, 0.02), (1000.0, 0.8)):
        ties += _compare(t, T, 0, Pp)
        n += t.shape[0]
        recounts += sum(_between_the_bounds(row, T, Pp) > 2048 for row in t.double().numpy())
    # more entries than the list holds: the steps are counted again, finer (10 and more of the 42 rows here)
    assert recounts >= 10 or V < 20000, recounts
    # The flagged band spans 6e-6 of the mass: where the entries at the cutoff are no heavier, a
    # decision is flagged more often than not.  That is the rule for the seven rows at P = 0.9999, the far
    # tail, and at V = 131072 (1 / V = 7.6e-6) for the nearly flat rows of T = 30 and 1000 as well; at
    # V = 20011 such a row is flagged one time in eight.
    assert ties <= (n // 2 if V > 100000 else 7 + 4), (ties, n)


def test_cutoffs_and_supports_do_not_depend_on_the_route():
    """A support call (list first) and a cutoff call (steps where a list looks hopeless) agree on the
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


def _check_cutoffs(z, groups, offset):
    """Cutoffs of one row of tied values at P = the end of a group of ties (counted from the top) + offset."""
    P = H.sv()
    vals, counts = np.unique(z, return_counts=True)
    vals, counts = vals[::-1].astype(np.float64), counts[::-1]
    share = np.cumsum(counts * np.exp(vals))
    share /= share[-1]
    row = torch.from_numpy(z)[None].cuda()
    cut, flags = torch.empty(1, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
    for g in groups:
        top_p = float(np.float32(share[g] + offset))
        want = vals[np.searchsorted(share, top_p)]                           # the first group whose end reaches P
        assert np.abs(share - top_p).min() > 7e-6                            # (the flagged band: 3e-6)
        P.sv_warp_cutoffs(row, 1.0, 0, top_p, cut, flags)
        torch.cuda.synchronize()
        assert int(flags[0]) == 0 and float(cut[0]) == want, (g, float(cut[0]), want)


@pytest.mark.parametrize("offset", [-1e-5, 1e-5])
def test_the_row_total_of_a_deep_nucleus_of_ties(offset):
    """Millions of equal terms round the same way in every lane: float32 lane sums of the first sweep are
    2e-5 too large on this row, and a P that lies 1e-5 from the end of a group of ties has to be
    decided by better than that.  A large entry for every lane, a tied value with most of the mass, and
    below it groups of ties down to half its weight."""
    V, per = 1 << 22, 500
    n_low = 1200 * per
    z = np.full(V, -3.7)                                                     # (exponents of two)
    z[:2048:4] = 0.0                                                         # (512 lanes, vectors of four)
    z[V - n_low:] = np.repeat(np.linspace(-4.3, -5.0, 1200), per)
    _check_cutoffs((z * np.log(2.0)).astype(np.float32), (50, 300, 700, 1000), offset)


@pytest.mark.parametrize("offset", [-9e-6, 9e-6])
def test_the_row_total_of_a_short_nucleus_over_ties(offset):
    """The same where a few entries are the nucleus and the ties are the rest: float32 lane sums are 2.9e-5
    too small."""
    z = np.full(1 << 24, -20.0)
    z[:2048:4] = -18.6
    z[:160:4] = np.linspace(0.0, -0.6, 40)
    _check_cutoffs((z * np.log(2.0)).astype(np.float32), (20, 30, 35), offset)
