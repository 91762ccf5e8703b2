"""Attention from per-row key lists and from the FlatCSR tensor where the lists are dense enough for tiles
(bf16, at least 256 blocks of 128 rows): windows of 1024 keys, lists of every length and form, against
the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_01777_amd import synth
from tests.util import TOL, assert_close, oracle_params, to_np64

pytestmark = pytest.mark.gpu


def _lists(B, H, T, L, density, seed):
    """Ascending lists: row (.., t) draws from the keys 0 .. t; every eighth row is empty, short or full."""
    rng = np.random.default_rng(seed)
    idx = np.full((B, H, T, L), -1, dtype=np.int32)
    cnt = np.zeros((B, H, T), dtype=np.int32)
    for b in range(B):
        for h in range(H):
            for t in range(T):
                p = (density, density, density, 0.0, 1.0, density, density / 50, density)[t % 8]
                keys = np.flatnonzero(rng.random(t + 1) < p)[:L]
                idx[b, h, t, :len(keys)] = keys
                cnt[b, h, t] = len(keys)
    return idx, cnt


@pytest.mark.parametrize("T,N,L,density", [(1100, 30, 1100, 0.4), (2080, 16, 2080, 0.9), (513, 52, 200, 0.2),
                                           (1024, 32, 40, 0.03), (1100, 60, 1100, 0.5), (513, 104, 513, 0.5)])
def test_dense_lists(T, N, L, density):
    from paper_2310_01777_amd import binding as sea
    B, H = 2, N // 2
    wl = synth.Workload("lists", B, H, T, 64, 32, 16, 4, 0, True, "bf16", 4)
    x = synth.make_inputs(wl)
    idx, cnt = _lists(B, H, T, L, density, T)
    # the last keys are nobody's (and hold what an unused row may hold); odd lists in a few tiles:
    # entries out of order, repeated, outside [0, T)
    idx[idx >= T - 3] = -1
    cnt[:] = (idx >= 0).sum(-1)
    for k in "KV":
        x[k][:, :, T - 3:] = float("nan")
    order = np.argsort(np.where(idx < 0, 1 << 30, idx), axis=-1, kind="stable")
    idx = np.take_along_axis(idx, order, -1)
    clean_idx, clean_cnt = idx.copy(), cnt.copy()
    r = T // 2
    n = int(cnt[0, 0, r])
    if n > 2:
        idx[0, 0, r, :n] = idx[0, 0, r, :n][::-1]                 # descending
        idx[0, 1, r + 1, 1] = T + 5                               # invalid in the middle
        keep = [v for v in idx[0, 1, r + 1, :cnt[0, 1, r + 1]] if v < T]
        clean_idx[0, 1, r + 1] = -1
        clean_idx[0, 1, r + 1, :len(keep)] = keep
        clean_cnt[0, 1, r + 1] = len(keep)
        idx[1, 0, r, 1] = idx[1, 0, r, 0]                         # listed twice: counts twice
        clean_idx[1, 0, r] = idx[1, 0, r]
    d = {k: x[k].cuda() for k in "QKV"}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=32, K=16, k_hat=4, causal=True, scale=wl.scale, dtype="bf16")
    O = torch.full((B, H, T, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    print(f"[case] lists T{T} N{N} L{L} density {density}", flush=True)
    sea.sea_sparse_attn(p, d["Q"], d["K"], d["V"], torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda(), L, O)
    torch.cuda.synchronize()
    po = oracle_params(wl)
    c = {k: to_np64(torch.nan_to_num(x[k])) for k in "QKV"}
    want = oracle.sparse_attn(po, c["Q"], c["K"], c["V"], clean_idx, clean_cnt)
    assert_close(to_np64(O), want, TOL["bf16"], "O from lists")

    # the FlatCSR tensor of ordinary lists: bit-identical to the lists
    idx, cnt = np.take_along_axis(clean_idx, np.argsort(np.where(clean_idx < 0, 1 << 30, clean_idx), -1), -1), clean_cnt
    idx[1, 0, r], cnt[1, 0, r] = -1, 0
    idx_d, cnt_d = torch.from_numpy(np.ascontiguousarray(idx)).cuda(), torch.from_numpy(cnt).cuda()
    crow = torch.empty(B * T + 1, dtype=torch.int64, device="cuda")
    col = torch.empty(int(cnt.sum()), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(256, sea.sea_flatcsr_workspace_bytes(p)), dtype=torch.uint8, device="cuda")
    O1, O2 = torch.empty_like(O), torch.empty_like(O)
    sea.sea_flatcsr(p, idx_d, cnt_d, L, crow, col, ws)
    sea.sea_flatcsr_attn(p, d["Q"], d["K"], d["V"], crow, col, O1)
    sea.sea_sparse_attn(p, d["Q"], d["K"], d["V"], idx_d, cnt_d, L, O2)
    torch.cuda.synchronize()
    crow_o, col_o = oracle.flatcsr(po, idx, cnt)
    assert np.array_equal(crow.cpu().numpy(), crow_o) and np.array_equal(col.cpu().numpy(), col_o)
    assert torch.equal(O1, O2)
    assert_close(to_np64(O1), oracle.sparse_attn(po, c["Q"], c["K"], c["V"], idx, cnt), TOL["bf16"], "O from the tensor")


def test_lists_astray_in_later_windows():
    """Lists that stop ascending, repeat or leave the sequence behind the first 1024 keys, in blocks of dense lists."""
    from paper_2310_01777_amd import binding as sea
    B, H, T = 1, 16, 2080
    wl = synth.Workload("lists", B, H, T, 64, 32, 16, 4, 0, True, "bf16", 4)
    x = synth.make_inputs(wl)
    L = T + 1
    idx = np.full((B, H, T, L), -1, dtype=np.int32)
    for t in range(T):
        idx[:, :, t, :t + 1] = np.arange(t + 1)
    cnt = np.broadcast_to(np.arange(1, T + 1, dtype=np.int32), (B, H, T)).copy()
    idx[0, 0, 2000, [1499, 1500]] = [1500, 1499]                        # out of order
    idx[0, 1, 1900, 1025:1901] = 1024                                   # 1024 many times, at the window's edge
    idx[0, 2, 2079, 2079] = T + 7                                       # outside, at the end
    idx[0, 3, 1030, 1026] = -5                                          # outside, among the last
    idx[0, 4, 2079, 2080], cnt[0, 4, 2079] = 3, T + 1                   # back to the first window
    idx[0, 5, 1200, 600:1200] = np.arange(600)                          # the first half twice
    idx[0, 6, 1500, 1:1501] = np.concatenate([np.arange(1030, 1501), np.arange(1, 1030)])  # windows exchanged
    d = {k: x[k].cuda() for k in "QKV"}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=32, K=16, k_hat=4, causal=True, scale=wl.scale, dtype="bf16")
    O = torch.full((B, H, T, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    print("[case] lists astray", flush=True)
    sea.sea_sparse_attn(p, d["Q"], d["K"], d["V"], torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda(), L, O)
    ok_idx, ok_cnt = idx.copy(), cnt.copy()
    for h, t, bad in ((2, 2079, T + 7), (3, 1030, -5)):
        keep = idx[0, h, t, :cnt[0, h, t]]
        keep = keep[keep != bad]
        ok_idx[0, h, t], ok_cnt[0, h, t] = -1, len(keep)
        ok_idx[0, h, t, :len(keep)] = keep
    want = oracle.sparse_attn(oracle_params(wl), to_np64(x["Q"]), to_np64(x["K"]), to_np64(x["V"]), ok_idx, ok_cnt)
    assert_close(to_np64(O), want, TOL["bf16"], "O from lists")


@pytest.mark.parametrize("B,H,T,L", [(1, 1, 5, 1), (2, 3, 70, 4), (1, 7, 300, 63), (2, 5, 257, 64), (1, 4, 130, 65),
                                     (1, 67, 40, 30), (1, 66, 150, 128), (2, 3, 140, 129)])
def test_flatcsr_of_short_lists(B, H, T, L):
    """Lists of any length up to L, the tensor whole and cut inside a list."""
    from paper_2310_01777_amd import binding as sea
    rng = np.random.default_rng(L)
    cnt = rng.integers(0, min(L, T) + 1, (B, H, T)).astype(np.int32)
    idx = np.full((B, H, T, L), -1, dtype=np.int32)
    for at in np.ndindex(B, H, T):
        idx[at][:cnt[at]] = np.sort(rng.choice(T, cnt[at], replace=False))
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=32, K=1, k_hat=1)
    po = oracle.Params(B=B, H=H, T=T, d=64, m=32, K=1, k_hat=1)
    crow_o, col_o = oracle.flatcsr(po, idx, cnt)
    idx_d, cnt_d = torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda()
    ws = torch.empty(max(256, sea.sea_flatcsr_workspace_bytes(p)), dtype=torch.uint8, device="cuda")
    print(f"[case] flatcsr {(B, H, T, L)}", flush=True)
    for cut in (len(col_o), max(len(col_o) // 2, 1), max(len(col_o) - 1, 1)):
        crow = torch.full((B * T + 1,), -7, dtype=torch.int64, device="cuda")
        col = torch.full((len(col_o) + 8,), -7, dtype=torch.int32, device="cuda")
        sea.sea_flatcsr(p, idx_d, cnt_d, L, crow, col[:cut], ws)
        assert np.array_equal(crow.cpu().numpy(), crow_o)
        assert np.array_equal(col[:cut].cpu().numpy(), col_o[:cut]) and bool((col[cut:] == -7).all())


@pytest.mark.parametrize("B,H,T,k_hat", [(1, 12, 2048, 96), (1, 13, 2048, 64), (1, 14, 2048, 64), (2, 12, 2048, 48),
                                         (1, 16, 2048, 64), (1, 17, 2048, 64)])
def test_lists_past_the_caches(B, H, T, k_hat):
    """Lists and the tensor built from them on both sides of the size at which they bypass the caches (33.6 M entries),
    against torch's own selection: every score distinct, whole columns of 16 keys."""
    from paper_2310_01777_amd import binding as sea
    K, w = 128, T // 128
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=64, K=K, k_hat=k_hat, causal=False)
    g = torch.Generator(device="cuda").manual_seed(T + k_hat)
    A_hat = torch.rand(B, H, T, K, generator=g, device="cuda").argsort(-1).float() / K
    out = sea.alloc_outputs(p)
    print(f"[case] lists past the caches {(B, H, T, k_hat)}", flush=True)
    sea.sea_topk_mask(p, A_hat, out["sel"], out["idx"], out["cnt"])
    sel = A_hat.topk(k_hat, -1).indices.sort(-1).values.int()
    idx = (sel[..., None] * w + torch.arange(w, dtype=torch.int32, device="cuda")).flatten(-2)
    assert torch.equal(out["sel"], sel) and torch.equal(out["idx"], idx) and bool((out["cnt"] == k_hat * w).all())
    crow = torch.empty(B * T + 1, dtype=torch.int64, device="cuda")
    col = torch.empty(idx.numel(), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(256, sea.sea_flatcsr_workspace_bytes(p)), dtype=torch.uint8, device="cuda")
    sea.sea_flatcsr(p, out["idx"], out["cnt"], sea.sea_row_stride(p), crow, col, ws)
    heads = torch.arange(H, dtype=torch.int32, device="cuda")[:, None, None] * T
    assert torch.equal(col, (idx + heads).transpose(1, 2).flatten())
    assert torch.equal(crow, torch.arange(B * T + 1, device="cuda") * (H * k_hat * w))
