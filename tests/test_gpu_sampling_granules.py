"""The sampling stage at the edges of its 4096-entry granules: vocabularies around one lane's run,
a granule and a chunk, more granules than a wavefront has lanes, all mass in one granule, and a
residual without mass, with and without support cutoffs, where the target's masses are drawn from."""
import numpy as np
import pytest
import torch

import svgen
from oracle import sv_oracle as O
from oracle import warp_oracle as W

import harness as H
from test_gpu_warped import _cut32, _gpu_verify_warped

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


# long rows, and more sequences of short ones than are drawn at once
LARGE = [(33000, "f32", 60), (36001, "bf16", 30), (9001, "f32", 1032), (5000, "bf16", 1284)]


@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("V,dtype,B", [(4097, "f32", 260), (8193, "bf16", 130), (12305, "bf16", 90), (9001, "f32", 180)] + LARGE)
def test_residual_without_mass_in_large_batches(V, dtype, B, chained):
    """More than 512 (bfloat16: 256) pairs of a sequence and a granule: a workgroup of the mass pass takes two granules
    where short rows are not drawn at once, LARGE, and one kernel does it all where they are.
    Every third sequence has a residual, in one granule only."""
    n = 6                                                # a few different sequences, in turn
    cfg = svgen.make_config(1, seed=V + 3, B=n, k=1, V=V, dtype=dtype)
    z_t, x = cfg["z_t"], cfg["x"]
    for b in range(n):
        z_t[b, 0, int(x[b, 0])] = -np.inf
    z_d = z_t[:, :1].clone()
    for b in range(0, n, 3):
        v = (V - 1, V // 2)[b // 3]
        z_t[b, 0, v] = z_t[b, 0].max()                   # the target's mass there is the residual
        z_d[b, 0, v] = -np.inf
    at = torch.arange(B) % n
    z_t, z_d, x = z_t[at], z_d[at], x[at]
    ref = H.oracle_verify(svgen.to_numpy_bits(z_t), svgen.to_numpy_bits(z_d), x.numpy(), seed=1, step=3)
    args = [t.contiguous().cuda() for t in ((z_t, z_d, z_d, x) if chained else (z_t, z_d, x))]
    got = (H.gpu_verify_chained if chained else H.gpu_verify)(*args, seed=1, step=3)
    H.assert_verify(got, ref, 1)
    empty, fell_back = (np.arange(B) % 3) != 0, (got["flags"] & O.FLAG_RESIDUAL_FALLBACK) != 0
    # (chained, the two normalisers are sums in different orders: a residual of rounding noise may be found)
    assert fell_back[empty].any() if chained else fell_back[empty].all()
    assert not fell_back[~empty].any()
    assert len({int(t) // 4096 for t in got["tokens"][fell_back, 0]}) > 1


@pytest.mark.parametrize("offset", [0.0, 600.0, -700.0, 708.0, 712.0, -712.0, 5000.0, 1e6])
def test_probabilities_on_either_side_of_the_short_form(offset):
    """The short form of the probabilities holds while |log2 of the normaliser| < 1024 (logits near 710);
    residuals of nearly equal rows, whose mass is what both forms have to leave unbiased."""
    V = 9001
    cfg = svgen.make_config(1, seed=int(abs(offset)) + 5, B=6, k=2, V=V, dtype="f32")
    z_t = cfg["z_t"] + offset
    z_d = z_t[:, :2] + 0.05 * torch.randn(z_t[:, :2].shape, generator=torch.Generator().manual_seed(3))
    _check(z_t, z_d.contiguous(), cfg["x"], 2, range(8))


def _nuclei(V, dtype, B, peaks_t, peaks_d, seed):
    """Flat rows under a few peaks of mass: z_t [B, 2, V], z_d [B, 1, V], a drafted token under all peaks, and
    the cutoffs and warped rows at P = 0.9, where the peaks are the nucleus."""
    g = torch.Generator().manual_seed(seed)
    z_t = torch.randn((B, 2, V), generator=g)
    z_d = z_t[:, :1].clone()
    for j, v in enumerate(peaks_t):
        z_t[:, :, v] = 24.0 + 0.25 * j
    for j, v in enumerate(peaks_d):
        z_d[:, :, v] = 24.0 + 0.25 * j
    z_t, z_d = z_t.to(dtype), z_d.to(dtype)
    y_t, cut_t, _ = W.warp_rows(svgen.to_numpy_bits(z_t), 1.0, 0, 0.9)
    y_d, cut_d, _ = W.warp_rows(svgen.to_numpy_bits(z_d), 1.0, 0, 0.9)
    assert np.isfinite(y_t[:, 0]).sum() == B * len(peaks_t) and np.isfinite(y_d).sum() == B * len(peaks_d)
    x = torch.full((B, 1), (set(range(len(peaks_t) + len(peaks_d) + 1)) - set(peaks_t) - set(peaks_d)).pop(),
                   dtype=torch.int32)
    return z_t, z_d, x, y_t, y_d, _cut32(cut_t), _cut32(cut_d)


@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("V,dtype", [(300, torch.float32), (9001, torch.float32), (12290, torch.bfloat16),
                                     (40000, torch.bfloat16), (270001, torch.bfloat16), (280003, torch.float32)])
def test_residual_without_mass_under_cutoffs(V, dtype, chained):
    """Equal nuclei of one token and of several, in one granule and in different ones, the drafted token outside
    both: no residual, the target distribution instead.  Then a draft nucleus that lacks one of the target's
    tokens, or has another one's place: a residual in one granule, none in the others."""
    _check_nuclei(V, dtype, 6, chained, range(3))


@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("V,dtype,B", [(4097, torch.float32, 260), (8193, torch.bfloat16, 130), (12290, torch.bfloat16, 90),
                                       (9001, torch.float32, 180)]
                         + [(V, torch.float32 if d == "f32" else torch.bfloat16, B) for V, d, B in LARGE])
def test_residual_without_mass_under_cutoffs_in_large_batches(V, dtype, B, chained):
    """The same where a workgroup takes two granules, the last of them alone in its chunk or with a partner (LARGE), and in one kernel."""
    _check_nuclei(V, dtype, B, chained, range(1))


def _check_nuclei(V, dtype, B, chained, seeds):
    P = H.sv()
    far = [V - 1, 2, V // 2, V // 3]
    for peaks_t, peaks_d, empty in (([V // 2], [V // 2], True), ([7, 9, 30], [7, 9, 30], True), (far, far, True),
                                    (far, far[:3], False), ([V - 1], [2], False)):
        z_t, z_d, x, y_t, y_d, cut_t, cut_d = _nuclei(V, dtype, B, peaks_t, peaks_d, V)
        z_t, z_d = z_t.cuda(), z_d.cuda()
        for seed in seeds:
            ref = H.oracle_verify(y_t, y_d, x.numpy(), seed=seed, step=4)
            if chained:
                f32 = lambda: torch.empty((B, 1), dtype=torch.float32, device="cuda")
                i32 = lambda *s: torch.full(s, -5, dtype=torch.int32, device="cuda")
                ws = P.alloc_workspace(B, 1, V, P.binding._dtype_tag(z_d))
                xd, tokens, n_acc, flags, ratio = x.cuda(), i32(B, 2), i32(B), i32(B), f32()
                P.sv_row_stats_warped(z_d, z_d, xd, 1.0, cut_d, 1.0, cut_d, f32(), f32(), f32(), f32(), None, None, ws)
                P.sv_verify_sample_warped_chained(z_t, None, z_d, xd, None, 1.0, cut_t, 1.0, cut_d, seed, 4, tokens,
                                                  n_acc, flags, ratio, ws)
                torch.cuda.synchronize()
                got = dict(tokens=tokens.cpu().numpy(), n_accept=n_acc.cpu().numpy(),
                           flags=flags.cpu().numpy().astype(np.uint32), ratio=ratio.cpu().numpy())
            else:
                got = _gpu_verify_warped(z_t, z_d, x.cuda(), 1.0, cut_t, 1.0, cut_d, seed=seed, step=4)
            assert (got["n_accept"] == 0).all() and (ref["n_accept"] == 0).all()
            assert (((got["flags"] & O.FLAG_RESIDUAL_FALLBACK) != 0) == empty).all()
            assert np.isin(got["tokens"][:, 0], peaks_t).all()
            clear = ((got["flags"] | ref["flags"]) & O.FLAG_NEAR_CDF_EDGE) == 0
            assert clear.sum() >= B - max(1, B // 50) and np.array_equal(got["tokens"][clear], ref["tokens"][clear])


@pytest.mark.parametrize("warped", [False, True])
def test_an_empty_residual_costs_the_token_pick_no_walk(warped):
    """The pick reads one granule of the row whether the residual has mass or not.  At 2^20 entries a walk over
    the row by its one workgroup takes more than ten times as long as that."""
    P = H.sv()
    V = 1 << 20
    mid = V // 2 + 5
    times = []
    for peaks_d in ([mid], [3]):
        z_t, z_d, x, _, _, cut_t, cut_d = _nuclei(V, torch.bfloat16, 1, [mid], peaks_d, 1)
        if not warped:
            z_t[:, :, int(x[0, 0])] = z_d[:, :, int(x[0, 0])] = -np.inf
        z_t, z_d, x = z_t.cuda(), z_d.cuda(), x.cuda()
        i32 = lambda *s: torch.empty(s, dtype=torch.int32, device="cuda")
        tokens, n_acc, flags = i32(1, 2), i32(1), i32(1)
        ws = P.alloc_workspace(1, 1, V, P.SV_BF16)
        best = np.inf
        for _ in range(20):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(), e1.record()                       # (the handles exist from here on)
            P.sv_set_timing_events(P.binding.SV_KERNEL_VERIFY_PICK, e0.cuda_event, e1.cuda_event)
            if warped:
                P.sv_verify_sample_warped(z_t, None, z_d, x, None, 1.0, cut_t, 1.0, cut_d, 0, 0, tokens, n_acc, flags,
                                          None, ws)
            else:
                P.sv_verify_sample(z_t, None, z_d, x, None, 0, 0, tokens, n_acc, flags, None, ws)
            P.sv_set_timing_events(P.binding.SV_KERNEL_VERIFY_PICK, None, None)
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1) * 1e3)
        assert bool(int(flags[0]) & O.FLAG_RESIDUAL_FALLBACK) == (peaks_d == [mid]) and int(tokens[0, 0]) == mid
        times.append(best)
    assert times[0] < 3.0 * times[1], times
