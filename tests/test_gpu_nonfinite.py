"""A key that a row does not list is no part of the row's result, whatever its value row holds and however large
its scores are: keys with infinities, NaN and scores beyond fp32 among ordinary ones, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_01777_amd import synth
from tests.test_gpu_lists import _lists
from tests.util import TOL, assert_close, oracle_params, to_np64

pytestmark = pytest.mark.gpu

# (dtype, B, H, T, m, K, k^, budget, causal, pad)
COLUMNS = [
    ("bf16", 1, 2, 601, 64, 100, 20, 0, True, 0.0),     # columns of any width, small launches: row by row
    ("bf16", 1, 2, 385, 64, 128, 17, 0, False, 0.0),
    ("bf16", 2, 1, 129, 64, 128, 31, 0, True, 0.3),
    ("bf16", 1, 26, 601, 64, 100, 30, 0, False, 0.0),   # tiles: three sets of waves,
    ("bf16", 5, 9, 700, 64, 100, 20, 0, False, 0.3),    # one
    ("bf16", 1, 1, 1300, 64, 13, 5, 100, True, 0.0),    # 20 of 100 keys a column
    ("bf16", 1, 4, 4001, 64, 128, 2, 0, True, 0.3),     # few keys per row: row by row
    ("bf16", 1, 12, 601, 64, 100, 60, 0, True, 0.0),    # many: tiles, six sets of waves, 8 slots,
    ("bf16", 1, 4, 385, 64, 128, 90, 0, False, 0.0),    # 16 slots,
    ("bf16", 2, 2, 129, 64, 128, 100, 0, True, 0.3),    # and 32
    ("bf16", 1, 2, 1300, 64, 13, 12, 240, True, 0.0),   # 20 of 100 keys a column
]
F32 = [
    ("f32", 1, 2, 385, 64, 128, 33, 0, True, 0.0),      # columns of any width
    ("f32", 2, 1, 290, 96, 64, 20, 0, False, 0.3),
    ("f32", 1, 1, 1300, 64, 13, 5, 500, True, 0.0),     # 100 of 100 keys a column
    ("f32", 1, 2, 700, 64, 60, 2, 0, False, 0.3),       # few keys per row
    ("f32", 1, 2, 385, 64, 128, 90, 0, True, 0.0),      # many: tiles
    ("f32", 2, 1, 290, 96, 64, 50, 0, False, 0.3),
]


def _check(O, idx, cnt, x, wl, bad, bad_rows_nan):
    """Rows that list none of the keys `bad` hold what they would without those keys' values; rows that list
    one with a NaN value are NaN."""
    po = oracle_params(wl)
    c = {k: to_np64(x[k]).copy() for k in "QKV"}
    c["K"][:, :, bad], c["V"][:, :, bad] = 0.0, 0.0
    want = oracle.sparse_attn(po, c["Q"], c["K"], c["V"], idx, cnt)
    listed = np.isin(idx, bad).any(-1)
    assert not listed.all()
    got = to_np64(O)
    clean = np.where(listed[..., None], 0.0, got)
    assert_close(clean, np.where(listed[..., None], 0.0, want), TOL[wl.dtype], "rows without the keys")
    if bad_rows_nan:
        assert listed.any() and np.isnan(got[..., 5][listed]).all()


@pytest.mark.parametrize("case", COLUMNS + F32, ids=lambda c: "_".join(str(v) for v in c))
def test_unselected_keys_stay_out(case):
    from paper_2310_01777_amd import binding as sea
    dtype, B, H, T, m, K, kh, kb, causal, pad = case
    wl = synth.Workload("nonfinite", B, H, T, 64, m, K, kh, kb, causal, dtype, 4, pad)
    x = synth.make_inputs(wl)
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, k_budget=kb, causal=causal, scale=wl.scale, dtype=dtype,
                      seq_len=None if x["seq_len"] is None else x["seq_len"].cuda())
    last = T if x["seq_len"] is None else int(x["seq_len"].min())
    bad = np.unique([last // 3, last // 2, last - 1])
    out, ws = sea.alloc_outputs(p), sea.alloc_workspace(p)
    for what in ("values", "scores") if dtype == "bf16" else ("values",):
        y = {k: x[k].clone() for k in "QKVW"}
        if what == "values":
            y["V"][:, :, bad] = float("inf")
            y["V"][:, :, bad, 5] = float("nan")
        else:  # finite keys whose features vanish and whose scores overflow
            y["K"][:, :, bad] = 1e37 * torch.sign(y["K"][:, :, bad].float()).to(y["K"].dtype)
        d = {k: v.cuda() for k, v in y.items()}
        print(f"[case] nonfinite {what} {case}", flush=True)
        sea.sea_estimate(p, d["Q"], d["K"], d["W"], out["A_hat"], ws)
        assert torch.isfinite(out["A_hat"]).all()
        sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], out["O"], out["A_hat"], out["sel"], out["idx"], out["cnt"], ws)
        O2 = torch.zeros_like(out["O"])
        sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O2, workspace=ws)
        assert torch.equal(O2.view(torch.uint8), out["O"].view(torch.uint8))
        _check(out["O"], out["idx"].cpu().numpy(), out["cnt"].cpu().numpy(), y, wl, bad, what == "values")


@pytest.mark.parametrize("T,m,K,pad", [(500, 128, 64, 0.0), (129, 64, 128, 0.0), (700, 256, 100, 0.3), (301, 64, 128, 0.0),
                                       (1000, 64, 33, 0.0), (2000, 64, 3, 0.0)])
def test_causal_estimate_before_a_key(T, m, K, pad):
    """Scores of causal rows do not know the keys after them."""
    from paper_2310_01777_amd import binding as sea
    wl = synth.Workload("nonfinite", 1, 3, T, 64, m, K, 2, 0, True, "bf16", 4, pad)
    x = synth.make_inputs(wl)
    seq = x["seq_len"]
    j = (T if seq is None else int(seq[0])) // 2
    clean = {k: to_np64(x[k]) for k in "QKW"}
    x["K"][0, 1, j] = float("nan")
    x["K"][0, 2, j, 3] = float("inf")
    p = sea.SeaParams(B=1, H=3, T=T, d=64, m=m, K=K, k_hat=2, causal=True, scale=wl.scale, dtype="bf16",
                      seq_len=None if seq is None else seq.cuda())
    A = torch.empty(1, 3, T, K, device="cuda")
    print(f"[case] nonfinite estimate {(T, m, K, pad)}", flush=True)
    sea.sea_estimate(p, x["Q"].cuda(), x["K"].cuda(), x["W"].cuda(), A, sea.alloc_workspace(p))
    want = oracle.estimate(oracle_params(wl), clean["Q"], clean["K"], clean["W"], seq_len=None if seq is None else seq.numpy())
    assert_close(to_np64(A)[:, :, :j], want[:, :, :j], TOL["bf16"], "A_hat")
    assert torch.isnan(A[0, 1, j]).any()


def test_unlisted_keys_stay_out():
    from paper_2310_01777_amd import binding as sea
    B, H, T, L = 2, 15, 1100, 1100   # lists dense enough, and blocks enough, for tiles
    wl = synth.Workload("lists", B, H, T, 64, 32, 16, 4, 0, True, "bf16", 4)
    x = synth.make_inputs(wl)
    idx, cnt = _lists(B, H, T, L, 0.4, T)
    bad = np.array([0, 500, 1090])
    x["V"][:, :, bad] = float("inf")
    x["V"][:, :, bad, 5] = float("nan")
    d = {k: x[k].cuda() for k in "QKV"}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=32, K=16, k_hat=4, causal=True, scale=wl.scale, dtype="bf16")
    O = torch.zeros(B, H, T, 64, dtype=torch.bfloat16, device="cuda")
    print("[case] nonfinite lists", flush=True)
    sea.sea_sparse_attn(p, d["Q"], d["K"], d["V"], torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda(), L, O)
    _check(O, idx, cnt, x, wl, bad, True)


@pytest.mark.parametrize("T,m,K,k_hat", [(512, 64, 128, 5), (700, 256, 100, 99), (1024, 128, 64, 40), (2048, 256, 256, 200)])
def test_columns_past_a_row_are_never_selected(T, m, K, k_hat):
    """Rows whose scores are ordinary, all zero, infinite or NaN: no column behind a causal row's own, none of padding."""
    from paper_2310_01777_amd import binding as sea
    wl = synth.Workload("nonfinite", 2, 5, T, 64, m, K, k_hat, 0, True, "bf16", 4)
    x = synth.make_inputs(wl)
    x["K"][:, 1] *= 1e3                              # features vanish: every score zero
    x["Q"][:, 2, 3::7] = float("nan")
    x["K"][:, 3, T // 3] = float("nan")
    x["Q"][:, 4, 3::7, 9], x["K"][:, 4, T // 2, 3] = float("inf"), float("-inf")
    lens = torch.tensor([T, T - T // 3], dtype=torch.int32)
    p = sea.SeaParams(B=2, H=5, T=T, d=64, m=m, K=K, k_hat=k_hat, causal=True, scale=wl.scale, dtype="bf16", seq_len=lens.cuda())
    words = torch.full((2, 5, T, (K + 31) // 32), -1, dtype=torch.int32, device="cuda")
    d = {k: x[k].cuda() for k in "QKVW"}
    print(f"[case] columns past a row {(T, m, K, k_hat)}", flush=True)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], torch.empty_like(d["Q"]), workspace=sea.alloc_workspace(p), mhat=words)
    got = ((words.cpu()[..., None] >> torch.arange(32, dtype=torch.int32)) & 1).flatten(-2)
    t, c = torch.arange(T), torch.arange(got.shape[-1])
    allowed = (c[None] <= (t[:, None] * K) // T) & (c[None] < K)
    allowed = allowed[None] & (t[None, :, None] < lens[:, None, None])
    assert not (got.bool() & ~allowed[:, None]).any()
    quota = torch.minimum(allowed.sum(-1), torch.tensor(k_hat))
    assert torch.equal(got.sum(-1)[:, :2], quota[:, None].expand(2, 2, T))  # rows without NaN take all of their quota
