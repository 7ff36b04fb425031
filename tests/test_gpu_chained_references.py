"""A chained verification sums the target rows as the statistics summed the draft rows, over c(m) or over the next whole
number: equal rows of a few tokens, the drafted token outside, have equal normalisers and no residual, whatever
kernel the statistics took."""
import numpy as np
import pytest
import torch

import harness as H
from oracle import sv_oracle as O

pytestmark = pytest.mark.gpu


def _equal_rows(V, dtype, B, k, n):
    """z_t [B, k + 1, V], z_d [B, k, V], x: n tokens a row in neighbouring vectors, which are different lanes'."""
    g = np.random.default_rng(V + B + n)
    per_vec = 1 if V < 8 else 4 if dtype == "f32" else 8
    z_t = torch.full((B, k + 1, V), float("-inf"))
    x = torch.zeros((B, k), dtype=torch.int32)
    for b in range(B):
        at = 1 + g.integers(V - 1 - (n - 1) * per_vec) + per_vec * np.arange(n)
        z_t[b, :, torch.from_numpy(at)] = torch.from_numpy(g.normal(0.0, 2.0, n).astype(np.float32))
    z_t = z_t.to(torch.float32 if dtype == "f32" else torch.bfloat16)
    return z_t.cuda(), z_t[:, :k].contiguous().cuda(), x.cuda()          # (the drafted token is 0: -inf in both)


def _chained(z_t, z_d, x, form, warped_call=False):
    P = H.sv()
    B, k, V = z_d.shape
    f32 = lambda: torch.empty((B, k), dtype=torch.float32, device="cuda")
    i32 = lambda *s: torch.full(s, -5, dtype=torch.int32, device="cuda")
    ws = P.alloc_workspace(B, k, V, P.binding._dtype_tag(z_d))
    kl = f32() if "kl" in form else None
    ent = f32() if "entropy" in form else None
    if "warped" in form:
        P.sv_row_stats_warped(z_d, z_d, x, 1.0, None, 1.0, None, f32(), f32(), f32(), f32(), kl, None, ws)
    else:
        P.sv_row_stats(z_d, z_d, x, f32(), f32(), f32(), f32(), kl, None, ws, None, ent, None)
    tokens, n_acc, flags = i32(B, k + 1), i32(B), i32(B)
    if warped_call:
        P.sv_verify_sample_warped_chained(z_t, None, z_d, x, None, 1.0, None, 1.0, None, 5, 2, tokens, n_acc, flags, None, ws)
    else:
        P.sv_verify_sample_chained(z_t, None, z_d, x, None, 5, 2, tokens, n_acc, flags, None, ws)
    return tokens.cpu().numpy(), n_acc.cpu().numpy(), flags.cpu().numpy()


def _assert_no_residual(z_t, z_d, x, form, warped_call=False):
    tokens, n_acc, flags = _chained(z_t, z_d, x, form, warped_call)
    assert (n_acc == 0).all()
    assert not (flags & (O.FLAG_BAD_ROW | H.sv().binding.FLAG_NO_CHAIN)).any()
    assert ((flags & O.FLAG_RESIDUAL_FALLBACK) != 0).all(), ((flags & O.FLAG_RESIDUAL_FALLBACK) != 0).mean()
    drawn = z_t[torch.arange(len(tokens)), 0, torch.from_numpy(tokens[:, 0]).long()]
    assert torch.isfinite(drawn).all()


# two tokens, so that sums over c(m) too are the same in every order
@pytest.mark.parametrize("form", ["plain", "kl", "entropy", "warped", "warped kl"])
@pytest.mark.parametrize("V,dtype,B,k", [(4096, "bf16", 96, 1), (32000, "bf16", 48, 2), (40000, "bf16", 48, 1), (8000, "f32", 96, 1), (30000, "f32", 48, 1),
                                         (50000, "bf16", 24, 1)])
def test_equal_rows_have_no_residual_after_any_statistics(V, dtype, B, k, form):
    z_t, z_d, x = _equal_rows(V, dtype, B, k, 2)
    _assert_no_residual(z_t, z_d, x, form)
    _assert_no_residual(z_t, z_d, x, form, warped_call=True)


# plain statistics that keep c(m): few fp32 entries of more pairs than compute units, fp32 rows of more than 14336
# entries of more pairs than two to a compute unit; rows shorter than a vector
@pytest.mark.parametrize("V,dtype,B", [(1000, "f32", 300), (16000, "f32", 600), (7, "bf16", 64), (3, "f32", 64)])
def test_equal_rows_have_no_residual_where_plain_statistics_keep_c_of_m(V, dtype, B):
    _assert_no_residual(*_equal_rows(V, dtype, B, 1, 2), "plain")


# sums over whole references are exact in any order
@pytest.mark.parametrize("V,dtype,B", [(4096, "bf16", 128), (32000, "bf16", 64), (8000, "f32", 128), (30000, "f32", 64), (45056, "bf16", 64)])
@pytest.mark.parametrize("n", [3, 20])
def test_equal_rows_of_more_tokens_have_no_residual_after_plain_statistics(V, dtype, B, n):
    _assert_no_residual(*_equal_rows(V, dtype, B, 1, n), "plain")


# the entries past a row's last whole vector, as the statistics add them: rows whose only tokens are these
@pytest.mark.parametrize("form", ["plain", "kl"])
@pytest.mark.parametrize("V,dtype,n", [(4103, "bf16", 2), (4103, "bf16", 7), (4097, "bf16", 2), (9, "bf16", 2), (15, "bf16", 7), (32007, "bf16", 5), (4099, "f32", 2),
                                       (4099, "f32", 3), (7, "f32", 3), (30001, "f32", 2)])
def test_equal_rows_of_tokens_past_the_last_vector_have_no_residual(V, dtype, n, form):
    g = np.random.default_rng(V + n)
    B = 96
    z_t = torch.full((B, 2, V), float("-inf"))
    z_t[:, :, V - n:] = torch.from_numpy(g.normal(0.0, 2.0, (B, 1, n)).astype(np.float32))
    z_t = z_t.to(torch.float32 if dtype == "f32" else torch.bfloat16).cuda()
    x = torch.zeros((B, 1), dtype=torch.int32, device="cuda")
    _assert_no_residual(z_t, z_t[:, :1].contiguous(), x, form)


# the draft as it is, the target warped: the statistics' sum is over whole references, the target's over c(m)
@pytest.mark.parametrize("cutoffs", [False, True])
@pytest.mark.parametrize("V,dtype,B", [(4096, "bf16", 8), (32000, "bf16", 40), (30001, "f32", 8), (16391, "bf16", 270)])
def test_a_warped_target_after_plain_statistics(V, dtype, B, cutoffs):
    import svgen
    P, k, T = H.sv(), 3, float(np.float32(0.7))
    cfg = svgen.make_config(1, seed=V, B=B, k=k, V=V, dtype=dtype)
    z_t, z_d, x = (cfg[n].cuda() for n in ("z_t", "z_d", "x"))
    f32 = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")
    i32 = lambda *s: torch.full(s, -5, dtype=torch.int32, device="cuda")
    cut_t = None
    if cutoffs:
        cut_t = f32(B, k + 1)
        P.sv_warp_cutoffs(z_t, T, 40, 1.0, cut_t)
    ws = P.alloc_workspace(B, k, V, P.binding._dtype_tag(z_d))
    out = []
    for chained in (True, False):
        o = dict(tokens=i32(B, k + 1), n=i32(B), flags=i32(B), ratio=f32(B, k))
        if chained:
            P.sv_row_stats(z_d, z_d, x, f32(B, k), f32(B, k), f32(B, k), f32(B, k), None, None, ws)
        (P.sv_verify_sample_warped_chained if chained else P.sv_verify_sample_warped)(
            z_t, None, z_d, x, None, T, cut_t, 1.0, None, 5, 2, o["tokens"], o["n"], o["flags"], o["ratio"], ws)
        out.append({n: v.cpu().numpy() for n, v in o.items()})
    a, b = out
    assert not (a["flags"] & P.binding.FLAG_NO_CHAIN).any()
    near = ((a["flags"] | b["flags"]) & (O.FLAG_NEAR_TIE | O.FLAG_NEAR_CDF_EDGE)) != 0
    for n in ("tokens", "n"):
        np.testing.assert_array_equal(a[n][~near], b[n][~near])
    np.testing.assert_allclose(a["ratio"][~near], b["ratio"][~near], rtol=1e-5)
    assert near.mean() <= 4e-6 * V + 0.1
