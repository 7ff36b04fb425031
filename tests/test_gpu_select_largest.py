"""sv_select_length above 1024 positions, and above 2048, where the 1024 largest products are searched first if the
peak lies among them: as many large products as fit, one less, one more; the peak at the last of them and behind; ties that
fill one step of the histogram; products that are all below its floor of 1/64, on it, and just under a step; latencies
that rise, stay, fall, jump and dip."""
import numpy as np
import pytest
import torch

import svgen
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


@pytest.mark.parametrize("B,k", [(2049, 1), (331, 7), (512, 16)])
@pytest.mark.parametrize("latency", ["table", "flat", "steep", "falling", "jump", "dip"])
def test_either_way_finds_the_peak(B, k, latency):
    n = B * k
    rng = np.random.default_rng(n + len(latency))
    lat = {"table": svgen.latency_table(n), "flat": np.ones(n + 1), "steep": 1.0 + np.arange(n + 1),
           "falling": np.linspace(2.0, 1.0, n + 1), "jump": 10.0 + 0.01 * np.arange(n + 1) + 5.0 * (np.arange(n + 1) > 700),
           "dip": np.where(np.arange(n + 1) == 900, 0.5, 1.0)}[latency].astype(np.float32)
    for lo, hi, levels in ((0.3, 1.0, 0), (0.95, 1.0, 0), (0.9, 1.0, 8), (1.0, 1.0, 0), (0.0, 0.1, 0), (0.0, 1.0, 3)):
        p = rng.uniform(lo, hi, (B, k))
        if levels:                                       # few different estimates: the products tie
            p = np.round(p * levels) / levels
        p = p.astype(np.float32)
        rg, ro, rm = O.select_length(p, lat)
        gg, go, gm = H.gpu_select_length(p, lat, O.MODE_BATCH_GREEDY)
        assert gm == rm and np.array_equal(gg, rg) and np.array_equal(go, ro), (lo, hi, levels, gm, rm)


@pytest.mark.parametrize("B", [128, 129, 300, 1024])
def test_the_estimates_take_no_launch_of_their_own(B):
    P = H.sv()
    k, n = 8, B * 8
    es, ea, table = (H.dev(a) for a in svgen.profile_table(10, 10))
    f = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda")
    i = lambda *s: torch.empty(s, dtype=torch.int32, device="cuda")
    before, after = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    before.record()
    torch.cuda._sleep(30_000_000)                        # 10 ms and more between the two, unless they are recorded again
    after.record()
    P.sv_set_timing_events(P.binding.SV_KERNEL_ACCEPT_ESTIMATE, before.cuda_event, after.cuda_event)
    try:
        P.sv_estimate_select(f(B, k), f(B, k), es, ea, table, H.dev(svgen.latency_table(n), torch.float32), P.SV_BATCH_GREEDY,
                             f(B, k), i(B), i(B + 1), i(1))
    finally:
        P.sv_set_timing_events(P.binding.SV_KERNEL_ACCEPT_ESTIMATE, None, None)
    torch.cuda.synchronize()
    assert before.elapsed_time(after) > 5.0
