"""sv_select_length above 1024 positions, where the 1024 largest products are searched first: as many large
products as fit, one less, one more; the peak at the last of them and behind; ties that fill one step of the
histogram; products that are all below its floor of 1/64, on it, and just under a step."""
import numpy as np
import pytest

from oracle import sv_oracle as O

import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1025, 2049])
@pytest.mark.parametrize("large", [0, 1, 1023, 1024, 1025])
@pytest.mark.parametrize("kind", ["spread", "one step", "floor"])
def test_peak_about_the_last_of_the_largest(n, large, kind):
    rng = np.random.default_rng(n * 7 + large)
    small = 0.01 * rng.random(n)                          # below the floor: never among the largest
    top = {"spread": 0.5 + 0.5 * rng.random(large), "one step": np.full(large, 1000 / 2048),
           "floor": rng.choice([1 / 64, np.nextafter(np.float32(33 / 2048), np.float32(0)), 33 / 2048], large)}[kind]
    p = small.astype(np.float32)
    p[rng.permutation(n)[:large]] = top.astype(np.float32)
    p = p.reshape(n, 1)
    for peak in (large - 1, large, large + 1):
        if not 1 <= peak <= n:
            continue
        lat = np.ones(n + 1, dtype=np.float32)            # a wall behind the peak
        lat[peak + 1:] = 1e6
        rg, ro, rm = O.select_length(p, lat)
        gg, go, gm = H.gpu_select_length(p, lat, O.MODE_BATCH_GREEDY)
        assert rm == peak
        assert gm == rm and np.array_equal(gg, rg) and np.array_equal(go, ro), (peak, gm)
