"""The output may take the place of the queries: every form of the attention reads a row's query before it writes
the row, and no other row's.  Keys with values that are not finite make the tiled forms compute rows again."""
import numpy as np
import pytest
import torch

from paper_2310_01777_amd import synth
from tests.test_gpu_lists import _lists
from tests.util import TOL, assert_close, to_np64

pytestmark = pytest.mark.gpu

# (dtype, B, H, T, m, K, k^, budget, causal, geometry)
LAYERS = [
    ("bf16", 1, 3, 512, 64, 64, 16, 0, True, 0),      # columns of a power of two of keys
    ("bf16", 1, 2, 4096, 64, 64, 1, 16, False, 0),    # one column a row
    ("bf16", 1, 12, 601, 64, 100, 60, 0, True, 0),    # any width, tiles
    ("bf16", 1, 4, 4001, 64, 128, 2, 0, True, 0),     # row by row
    ("bf16", 1, 2, 700, 64, 64, 16, 0, True, 1),      # per-row widths
    ("f32", 1, 2, 512, 64, 64, 16, 0, True, 0),
    ("f32", 1, 2, 385, 64, 128, 90, 0, True, 0),      # any width, tiles
    ("f32", 1, 2, 700, 64, 60, 2, 0, False, 0),       # row by row
]


@pytest.mark.parametrize("case", LAYERS, ids=lambda c: "_".join(str(v) for v in c))
def test_layers(case):
    from paper_2310_01777_amd import binding as sea
    dtype, B, H, T, m, K, kh, kb, causal, geometry = case
    wl = synth.Workload("in_place", B, H, T, 64, m, K, kh, kb, causal, dtype, 4)
    d = {k: v.cuda() for k, v in synth.make_inputs(wl).items() if v is not None}
    d["V"][:, :, T // 2] = float("nan")
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, k_budget=kb, causal=causal, scale=wl.scale, dtype=dtype,
                      geometry=geometry)
    ws, O = sea.alloc_workspace(p), torch.empty_like(d["Q"])
    print(f"[case] in place {case}", flush=True)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O, workspace=ws)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], d["Q"], workspace=ws)
    assert torch.equal(torch.isnan(O), torch.isnan(d["Q"]))
    assert torch.equal(torch.nan_to_num(O), torch.nan_to_num(d["Q"]))


@pytest.mark.parametrize("T,N,L,density", [(1100, 60, 1100, 0.5), (1024, 32, 40, 0.03)])
def test_lists(T, N, L, density):
    from paper_2310_01777_amd import binding as sea
    B, H = 2, N // 2
    wl = synth.Workload("lists", B, H, T, 64, 32, 16, 4, 0, True, "bf16", 4)
    d = {k: v.cuda() for k, v in synth.make_inputs(wl).items() if v is not None}
    d["V"][:, :, T // 2] = float("nan")
    idx, cnt = _lists(B, H, T, L, density, T)
    idx_d, cnt_d = torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda()
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=32, K=16, k_hat=4, causal=True, scale=wl.scale, dtype="bf16")
    crow = torch.empty(B * T + 1, dtype=torch.int64, device="cuda")
    col = torch.empty(int(cnt.sum()), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(256, sea.sea_flatcsr_workspace_bytes(p)), dtype=torch.uint8, device="cuda")
    O, Q1, Q2 = torch.empty_like(d["Q"]), d["Q"].clone(), d["Q"].clone()
    print(f"[case] lists in place T{T} N{N} L{L}", flush=True)
    sea.sea_flatcsr(p, idx_d, cnt_d, L, crow, col, ws)
    sea.sea_sparse_attn(p, d["Q"], d["K"], d["V"], idx_d, cnt_d, L, O)
    sea.sea_sparse_attn(p, Q1, d["K"], d["V"], idx_d, cnt_d, L, Q1)
    sea.sea_flatcsr_attn(p, Q2, d["K"], d["V"], crow, col, Q2)
    listed = (idx == T // 2).any(-1)
    for q in (Q1, Q2):
        assert np.array_equal(torch.isnan(q).any(-1).cpu().numpy(), listed)
        assert_close(to_np64(torch.nan_to_num(q)), to_np64(torch.nan_to_num(O)), TOL["bf16"], "O in the place of Q")
