"""Tensors that start anywhere in memory: at whole 4-byte words and, for bf16, between two of them, where some stages
take another kernel.  Same results as with tensors at the start of an allocation."""
import numpy as np
import pytest
import torch

from paper_2310_01777_amd import synth
from tests.util import TOL, assert_close, to_np64

pytestmark = pytest.mark.gpu

# dtype, B, H, T, m, K, k_hat, k_budget, causal, geometry
LAYERS = [
    ("bf16", 1, 3, 512, 64, 64, 16, 0, True, 0),    # columns of a power of two of keys
    ("bf16", 1, 2, 512, 256, 256, 32, 0, False, 0),
    ("bf16", 1, 2, 4096, 64, 64, 1, 16, False, 0),  # one column a row: buckets
    ("bf16", 1, 2, 601, 64, 100, 60, 0, True, 0),   # columns of any width, tiles
    ("bf16", 1, 2, 700, 64, 64, 16, 0, True, 1),    # per-row widths
    ("f32", 1, 2, 512, 64, 64, 16, 0, True, 0),
]


def _shifted(t, by):
    """A copy of t that starts `by` elements into its allocation."""
    at = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda")[by:].view(t.shape)
    return at.copy_(t)


@pytest.mark.parametrize("by", [1, 2])
@pytest.mark.parametrize("case", LAYERS, ids=lambda c: "_".join(str(v) for v in c))
def test_layers(case, by):
    from paper_2310_01777_amd import binding as sea
    dtype, B, H, T, m, K, kh, kb, causal, geometry = case
    wl = synth.Workload("anywhere", B, H, T, 64, m, K, kh, kb, causal, dtype, 4)
    d = {k: v.cuda() for k, v in synth.make_inputs(wl).items() if v is not None}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, k_budget=kb, causal=causal, scale=wl.scale, dtype=dtype,
                      geometry=geometry)
    ws, O = sea.alloc_workspace(p), torch.empty_like(d["Q"])
    print(f"[case] tensors {by} elements in {case}", flush=True)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O, workspace=ws)
    s = {k: _shifted(d[k], by) for k in "QKVW"}
    O_s = _shifted(torch.empty_like(O), by)
    sea.sea_forward(p, s["Q"], s["K"], s["V"], s["W"], O_s, workspace=ws)
    # (weights of 8 or 24 significant bits: two outputs within the tolerance of the definition each)
    assert_close(to_np64(O_s), to_np64(O), TOL[dtype], "O of tensors elsewhere")


@pytest.mark.parametrize("by", [1, 2])
def test_dense(by):
    from paper_2310_01777_amd import binding as sea
    wl = synth.Workload("anywhere", 1, 2, 300, 64, 32, 10, 4, 0, True, "bf16", 4)
    d = {k: v.cuda() for k, v in synth.make_inputs(wl).items() if v is not None}
    p = sea.SeaParams(B=1, H=2, T=300, d=64, m=32, K=10, k_hat=4, causal=True, scale=wl.scale, dtype="bf16")
    O = torch.empty_like(d["Q"])
    print(f"[case] dense, tensors {by} elements in", flush=True)
    sea.sea_dense_attn(p, d["Q"], d["K"], d["V"], O)
    s = {k: _shifted(d[k], by) for k in "QKV"}
    O_s = _shifted(torch.empty_like(O), by)
    sea.sea_dense_attn(p, s["Q"], s["K"], s["V"], O_s)
    assert torch.equal(O, O_s)


@pytest.mark.parametrize("by", [1, 2])
def test_lists(by):
    from paper_2310_01777_amd import binding as sea
    H, T, L = 30, 1100, 600
    wl = synth.Workload("anywhere", 1, H, T, 64, 32, 16, 4, 0, True, "bf16", 4)
    d = {k: v.cuda() for k, v in synth.make_inputs(wl).items() if v is not None}
    p = sea.SeaParams(B=1, H=H, T=T, d=64, m=32, K=16, k_hat=4, causal=True, scale=wl.scale, dtype="bf16")
    cnt = torch.arange(1, T + 1, dtype=torch.int32).clamp(max=L).expand(1, H, T).contiguous().cuda()
    idx = torch.from_numpy(np.maximum(np.arange(T)[:, None] - np.minimum(np.arange(T)[:, None], L - 1) + np.arange(L), 0).astype(np.int32))
    idx = idx.clamp(max=T - 1).expand(1, H, T, L).contiguous().cuda()
    O = torch.empty_like(d["Q"])
    print(f"[case] lists, tensors {by} elements in", flush=True)
    sea.sea_sparse_attn(p, d["Q"], d["K"], d["V"], idx, cnt, L, O)
    s = {k: _shifted(d[k], by) for k in "QKV"}
    O_s = _shifted(torch.empty_like(O), by)
    sea.sea_sparse_attn(p, s["Q"], s["K"], s["V"], _shifted(idx, by), cnt, L, O_s)
    assert_close(to_np64(O_s), to_np64(O), TOL["bf16"], "O of tensors elsewhere")


# dtype, B, H, T, m, K, k_hat, k_budget, causal, geometry: the splits of a block's waves and the slots of the mask product
SAME_KERNEL = [
    ("bf16", 1, 12, 601, 64, 100, 60, 0, True, 0),    # columns of any width: six sets of waves, 8 slots,
    ("bf16", 1, 52, 601, 64, 100, 60, 0, True, 0),    # three,
    ("bf16", 1, 52, 601, 64, 100, 60, 0, False, 0),   # one
    ("bf16", 1, 2, 385, 64, 128, 100, 0, False, 0),   # 16 slots
    ("bf16", 1, 70, 385, 64, 100, 90, 0, False, 0),
    ("bf16", 2, 2, 129, 64, 128, 100, 0, True, 0),    # 32
    ("bf16", 1, 50, 300, 64, 128, 100, 0, False, 0),
    ("bf16", 1, 90, 300, 64, 128, 100, 0, False, 0),
    ("bf16", 1, 2, 512, 64, 64, 16, 0, True, 0),      # powers of two: 64 rows and four sets of waves,
    ("bf16", 1, 9, 4096, 64, 64, 16, 0, True, 0),     # 128 rows and four,
    ("bf16", 1, 60, 1024, 64, 64, 16, 0, False, 0),   # two,
    ("bf16", 1, 36, 1024, 64, 64, 16, 0, True, 0),    # 64 rows and two,
    ("bf16", 1, 70, 512, 64, 64, 16, 0, True, 0),     # one
    ("bf16", 1, 2, 700, 64, 64, 16, 0, True, 1),      # per-row widths (key bits): the same
    ("bf16", 1, 13, 4096, 64, 64, 16, 0, True, 1),
    ("bf16", 1, 26, 2048, 64, 64, 16, 0, True, 1),
    ("bf16", 1, 100, 512, 64, 64, 16, 0, True, 1),
    ("bf16", 1, 2, 512, 64, 2, 1, 0, False, 0),       # a bucket of 256 keys
]


@pytest.mark.parametrize("case", SAME_KERNEL, ids=lambda c: "_".join(str(v) for v in c))
def test_same_kernel(case):
    """Keys and values between two words take the form that the layer takes: the results are the same bit for bit."""
    from paper_2310_01777_amd import binding as sea
    dtype, B, H, T, m, K, kh, kb, causal, geometry = case
    wl = synth.Workload("anywhere", B, H, T, 64, m, K, kh, kb, causal, dtype, 4)
    d = {k: v.cuda() for k, v in synth.make_inputs(wl).items() if v is not None}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, k_budget=kb, causal=causal, scale=wl.scale, dtype=dtype,
                      geometry=geometry)
    ws, O = sea.alloc_workspace(p), torch.empty_like(d["Q"])
    print(f"[case] same kernel {case}", flush=True)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O, workspace=ws)
    assert torch.isfinite(O).all()
    for which in ("K", "V", "KV"):
        s = {k: _shifted(v, 1) if k in which else v for k, v in d.items()}
        O_s = torch.full_like(O, float("nan"))
        sea.sea_forward(p, s["Q"], s["K"], s["V"], s["W"], O_s, workspace=ws)
        assert torch.equal(O, O_s), which


@pytest.mark.parametrize("flat", [False, True])
def test_lists_same_kernel(flat):
    """The same for lists, as they are and in the FlatCSR tensor: enough blocks and entries for tiles."""
    from paper_2310_01777_amd import binding as sea
    H, T, L = 30, 1100, 600
    wl = synth.Workload("anywhere", 1, H, T, 64, 32, 16, 4, 0, True, "bf16", 4)
    d = {k: v.cuda() for k, v in synth.make_inputs(wl).items() if v is not None}
    p = sea.SeaParams(B=1, H=H, T=T, d=64, m=32, K=16, k_hat=4, causal=True, scale=wl.scale, dtype="bf16")
    t, x = torch.arange(T, device="cuda")[:, None], torch.arange(L, device="cuda")
    # (every second key of the last 1200, the row's own among them)
    n = ((t + 2) // 2).clamp(max=L)
    idx = torch.where(x < n, t - 2 * (n - 1 - x), -1).int().expand(1, H, T, L).contiguous()
    cnt = n.flatten().int().expand(1, H, T).contiguous()
    crow, col = torch.empty(T + 1, dtype=torch.int64, device="cuda"), torch.empty(int(cnt.sum()), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(256, sea.sea_flatcsr_workspace_bytes(p)), dtype=torch.uint8, device="cuda")
    sea.sea_flatcsr(p, idx, cnt, L, crow, col, ws)

    def attend(q, k, v):
        O = torch.full_like(d["Q"], float("nan"))
        if flat:
            sea.sea_flatcsr_attn(p, q, k, v, crow, col, O)
        else:
            sea.sea_sparse_attn(p, q, k, v, idx, cnt, L, O)
        return O

    print(f"[case] lists, same kernel, flat {flat}", flush=True)
    O = attend(d["Q"], d["K"], d["V"])
    assert torch.isfinite(O).all()
    for which in ("K", "V", "KV"):
        s = {k: _shifted(v, 1) if k in which else v for k, v in d.items()}
        assert torch.equal(O, attend(s["Q"], s["K"], s["V"])), which


@pytest.mark.parametrize("by", [1, 2, 4])
@pytest.mark.parametrize("B,H,T,K,causal", [(2, 12, 131, 128, True), (1, 4, 150, 64, False), (1, 2, 300, 258, True)])
def test_decoder_weights(B, H, T, K, causal, by):
    """The decoder's weights and results anywhere in memory: read in pieces of 16 bytes, whatever lies in front of them."""
    from paper_2310_01777_amd import binding as sea
    wl = synth.Workload("anywhere", B, H, T, 64, 64, K, 4, 0, causal, "bf16", 4)
    d = {k: v.cuda() for k, v in synth.make_inputs(wl).items() if v is not None}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=64, K=K, k_hat=4, causal=causal, scale=wl.scale, dtype="bf16")
    ws = torch.empty(sea.sea_decoder_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    weights = {k: v.cuda() for k, v in synth.decoder_weights(H, 64, K).items()}
    out = [torch.empty(B, H, T, K, device="cuda"), torch.empty(B, H, T, device="cuda"), torch.empty(B, H, T, device="cuda")]
    print(f"[case] decoder weights {by} elements in {(B, H, T, K, causal)}", flush=True)
    sea.sea_decoder_estimate(p, weights, d["Q"], d["K"], d["V"], d["W"], out[0], ws, s_mix=out[1], s_prob=out[2])
    got = [_shifted(torch.full_like(o, -1.0), by) for o in out]
    shifted = {k: _shifted(v, by) for k, v in weights.items()}
    sea.sea_decoder_estimate(p, shifted, d["Q"], d["K"], d["V"], d["W"], got[0], ws, s_mix=got[1], s_prob=got[2])
    assert all(torch.equal(a, b) for a, b in zip(out, got))
