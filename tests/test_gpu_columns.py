"""Column-selected masks whose columns have any width (K does not divide T, or a column emits a number
of keys that is no power of two): the estimator's key kernel for any width and the tiled attention (bf16: with
the mask taken through the matrix product), at the widths where column groups, column slots, tiles and
list ends change, and the aligned tiled attention at the sizes where its waves are split differently, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_01777_amd import synth
from tests.util import TOL, assert_close, oracle_params, to_np64

pytestmark = pytest.mark.gpu

# (B, H, T, m, K, k^, budget, causal, pad)
CASES = [
    (1, 2, 129, 64, 128, 31, 0, True, 0.0),      # one or two keys per column: 32 slots; a tile of one row
    (2, 1, 383, 64, 128, 40, 0, False, 0.3),     # two or three: still 32 slots
    (1, 2, 385, 128, 128, 17, 0, True, 0.0),     # three or four: 16 slots
    (1, 1, 639, 64, 128, 50, 0, True, 0.3),      # four or five: 16 slots
    (1, 2, 640, 64, 128, 50, 0, True, 0.0),      # exactly five: 8 slots, eight columns in a sub-chunk
    (1, 2, 257, 256, 31, 9, 0, True, 0.0),       # eight or nine, K below one mask word
    (2, 2, 1000, 128, 33, 8, 0, False, 0.3),     # 30 or 31, K just above one mask word
    (1, 1, 2047, 64, 9, 4, 0, True, 0.0),        # columns of more than 64 keys
    (2, 1, 2000, 64, 3, 2, 64, True, 0.3),       # columns of more than 256 keys: one per block on the key side
    (1, 2, 250, 256, 250, 60, 0, True, 0.0),     # K = T, no power of two columns
    (1, 2, 1100, 64, 64, 10, 50, True, 0.0),     # five of the 17 or 18 keys of a column
    (1, 2, 1025, 64, 64, 16, 48, False, 0.3),    # three of 16 or 17
    (1, 1, 1500, 64, 100, 20, 20, True, 0.0),    # one of 15
    (1, 1, 1300, 64, 13, 5, 500, True, 0.0),     # 100 of 100: the cap equals every width
    (1, 1, 1030, 32, 1024, 100, 0, True, 0.0),   # the largest K
    (1, 26, 601, 64, 100, 20, 0, False, 0.3),    # more row blocks than six sets of waves share lists for: 8 slots,
    (1, 34, 500, 64, 128, 30, 0, True, 0.0),     # 16 slots
    (1, 75, 249, 32, 140, 60, 0, True, 0.0),     # and 32
    (5, 9, 700, 64, 100, 20, 0, False, 0.3),     # more than three sets do: 8 slots,
    (2, 33, 401, 64, 128, 30, 0, False, 0.0),    # 16 slots
    (3, 45, 250, 32, 249, 60, 0, False, 0.3),    # and 32
    (1, 1, 37, 64, 5, 5, 0, False, 0.0),         # every column selected, less than one step of keys
    (3, 11, 4001, 64, 65, 1, 3, False, 0.0),     # one column per row: row groups end inside heads, shares between them
    (1, 8, 16384, 128, 128, 1, 4, False, 0.0),   # and with full tiles, as few groups as the row kernel takes
    # most columns selected: tiles, six sets of waves
    (1, 2, 129, 64, 128, 120, 0, True, 0.0),     # 32 slots
    (2, 1, 383, 64, 128, 110, 0, False, 0.3),
    (1, 1, 1030, 32, 1024, 900, 0, True, 0.0),
    (1, 4, 385, 128, 128, 100, 0, True, 0.0),    # 16 slots
    (1, 2, 1025, 64, 64, 60, 180, False, 0.3),   # three of 16 or 17 keys
    (1, 2, 257, 256, 31, 28, 0, True, 0.0),      # 8 slots
    (1, 2, 1100, 64, 64, 50, 250, True, 0.0),    # five of the 17 or 18 keys of a column
    (2, 1, 2000, 64, 3, 3, 192, True, 0.3),      # 64 of more than 256
]

# aligned columns: how waves share the key list depends on the number of row blocks and the list's length
ALIGNED_CASES = [
    (1, 2, 1024, 64, 256, 60, 0, True, 0.0),     # four sets of two waves; early rows give three of them nothing
    (2, 1, 2048, 64, 1024, 100, 100, True, 0.3), # one key per column
    (2, 1, 1536, 64, 512, 50, 100, False, 0.3),  # two of three
    (1, 3, 1000, 64, 125, 30, 0, True, 0.0),     # a list that ends inside a chunk
    (3, 4, 640, 64, 64, 20, 80, False, 0.5),     # the shortest list for sets, sequences of half a tile
    (1, 1, 4224, 64, 128, 16, 256, True, 0.0),   # 16 of 33
    (2, 2, 4096, 64, 64, 9, 0, True, 0.3),       # one column per chunk
    (2, 17, 1000, 64, 250, 60, 0, True, 0.3),    # two sets of two waves: a list that ends inside a chunk,
    (2, 17, 1024, 64, 256, 60, 0, True, 0.3),    # four keys per column,
    (3, 23, 512, 64, 512, 100, 0, True, 0.3),    # one: the shortest list for them,
    (2, 19, 960, 64, 15, 4, 0, False, 0.3),      # 64, sequences of half a tile
    (2, 26, 1024, 64, 256, 60, 0, False, 0.3),   # two sets of four waves
    (1, 9, 4096, 64, 128, 16, 0, True, 0.0),     # four
    (1, 2, 128, 64, 128, 31, 0, True, 0.0),      # one set, one key per column
    (2, 1, 200, 64, 100, 25, 0, False, 0.3),     # two
    (1, 2, 240, 64, 60, 20, 0, True, 0.0),       # four
    (1, 1, 192, 64, 3, 2, 0, True, 0.0),         # 64
]


F32_CASES = [CASES[0], CASES[3], CASES[5], CASES[6], CASES[8], CASES[10], (1, 1, 33, 32, 7, 3, 0, True, 0.0),
             (1, 2, 700, 64, 300, 40, 0, True, 0.0), (2, 1, 290, 96, 64, 9, 0, False, 0.3)]


@pytest.mark.parametrize("dtype,case", [("bf16", c) for c in CASES + ALIGNED_CASES] + [("f32", c) for c in F32_CASES],
                         ids=lambda v: v if isinstance(v, str) else "_".join(str(x) for x in v))
def test_any_column_width(dtype, case):
    from paper_2310_01777_amd import binding as sea
    B, H, T, m, K, kh, kb, causal, pad = case
    wl = synth.Workload("columns", B, H, T, 64, m, K, kh, kb, causal, dtype, 4, pad)
    x = synth.make_inputs(wl)
    seq = None if x["seq_len"] is None else x["seq_len"].clone()
    if seq is not None:
        seq[-1] = 0 if B > 1 else T // 2         # a sequence without keys
        for k in "KV" if case not in ALIGNED_CASES else "":  # what lies behind a sequence's end is never read
            for b in range(B):
                x[k][b, :, int(seq[b]):] = float("nan")
    d = {k: x[k].cuda() for k in "QKVW"}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, k_budget=kb, causal=causal, scale=wl.scale,
                      dtype=dtype, seq_len=None if seq is None else seq.cuda())
    out, ws = sea.alloc_outputs(p), sea.alloc_workspace(p)
    print(f"[case] columns {dtype} {case}", flush=True)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], out["O"], out["A_hat"], out["sel"], out["idx"], out["cnt"], ws,
                    mhat=out["mhat"])
    O2 = torch.full_like(out["O"], float("nan"))   # and without any intermediate
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O2, workspace=ws)
    torch.cuda.synchronize()
    po = oracle_params(wl)
    sl = None if seq is None else seq.numpy()
    clean = {k: torch.nan_to_num(x[k]) for k in "QKV"}
    A = out["A_hat"].cpu().numpy().astype(np.float64)
    assert_close(A, oracle.estimate(po, to_np64(clean["Q"]), to_np64(clean["K"]), to_np64(x["W"]), seq_len=sl),
                 TOL[dtype], "A_hat")
    sel, idx, cnt = oracle.topk_mask(po, A, seq_len=sl)
    assert np.array_equal(out["sel"].cpu().numpy(), sel)
    assert np.array_equal(out["idx"].cpu().numpy(), idx)
    assert np.array_equal(out["cnt"].cpu().numpy(), cnt)
    want = oracle.sparse_attn(po, to_np64(clean["Q"]), to_np64(clean["K"]), to_np64(clean["V"]), idx, cnt)
    assert_close(to_np64(out["O"]), want, TOL[dtype], "O")
    assert torch.equal(O2, out["O"])


# few keys per row: a wavefront per row reads them from the mask words, where that is faster than tiles
# (dtype, B, H, T, m, K, k^, budget, causal, pad, grouping)
FEW_CASES = [
    ("bf16", 1, 3, 4001, 64, 128, 2, 60, False, 0.0, 0),    # 30 of 31 or 32 keys
    ("bf16", 2, 2, 3001, 64, 1000, 1, 0, False, 0.3, 0),    # three or four, 32 mask words
    ("bf16", 1, 2, 5003, 64, 100, 1, 40, True, 0.0, 0),     # 40 of 50 or 51, rows that end inside
    ("bf16", 2, 1, 9001, 64, 64, 1, 100, True, 0.5, 0),     # more slots than lanes
    ("bf16", 1, 2, 4001, 64, 128, 1, 0, True, 0.0, 0),      # whole columns
    ("bf16", 1, 3, 3001, 64, 100, 1, 0, True, 0.0, 1),      # heads share the quota
    ("bf16", 1, 1, 2041, 64, 64, 16, 0, False, 0.0, 0),     # 512 keys of 2041: rows; 544: tiles
    ("bf16", 1, 1, 2041, 64, 64, 17, 0, False, 0.0, 0),
    ("bf16", 1, 2, 100, 64, 100, 1, 0, False, 0.3, 1),      # K = T, heads share the quota
    ("f32", 2, 2, 333, 64, 64, 2, 0, True, 0.3, 0),
    ("f32", 1, 1, 130, 32, 128, 1, 0, False, 0.0, 0),       # one or two keys
    ("f32", 1, 2, 1300, 64, 13, 1, 50, False, 0.0, 0),
    ("f32", 1, 1, 5003, 64, 1000, 20, 20, False, 0.3, 0),   # one of five or six
    ("f32", 1, 3, 700, 64, 60, 2, 0, True, 0.0, 1),
    ("f32", 1, 2, 1000, 64, 62, 18, 0, False, 0.0, 0),      # 306 keys of 1000: rows; 323: tiles
    ("f32", 1, 2, 1000, 64, 62, 19, 0, False, 0.0, 0),
]


@pytest.mark.parametrize("case", FEW_CASES, ids=lambda v: "_".join(str(x) for x in v))
def test_few_keys_per_row(case):
    from paper_2310_01777_amd import binding as sea
    dtype, B, H, T, m, K, kh, kb, causal, pad, grouping = case
    wl = synth.Workload("columns", B, H, T, 64, m, K, kh, kb, causal, dtype, 4, pad, grouping=grouping)
    x = synth.make_inputs(wl)
    d = {k: x[k].cuda() for k in "QKVW"}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, k_budget=kb, causal=causal, scale=wl.scale, dtype=dtype,
                      grouping=grouping, seq_len=None if x["seq_len"] is None else x["seq_len"].cuda())
    out, ws = sea.alloc_outputs(p), sea.alloc_workspace(p)
    print(f"[case] few keys {case}", flush=True)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], out["O"], out["A_hat"], out["sel"], out["idx"], out["cnt"], ws)
    O2 = torch.full_like(out["O"], float("nan"))
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O2, workspace=ws)
    lists = torch.full_like(out["O"], float("nan"))
    sea.sea_sparse_attn(p, d["Q"], d["K"], d["V"], out["idx"], out["cnt"], sea.sea_row_stride(p), lists)
    torch.cuda.synchronize()
    po = oracle_params(wl)
    idx, cnt = out["idx"].cpu().numpy(), out["cnt"].cpu().numpy()
    _, idx_o, cnt_o = oracle.topk_mask(po, out["A_hat"].cpu().numpy().astype(np.float64),
                                       seq_len=None if x["seq_len"] is None else x["seq_len"].numpy())
    assert np.array_equal(idx, idx_o) and np.array_equal(cnt, cnt_o)
    want = oracle.sparse_attn(po, to_np64(x["Q"]), to_np64(x["K"]), to_np64(x["V"]), idx, cnt)
    assert_close(to_np64(out["O"]), want, TOL[dtype], "O")
    assert torch.equal(O2, out["O"])
    if kb:  # a fixed number of keys per column: the rows' keys in the order of the lists, so the same sums
        assert torch.equal(out["O"], lists)


@pytest.mark.parametrize("m,T,K", [(64, 1000, 60), (96, 1025, 33), (128, 1000, 125)])
def test_f32_features_of_many_rows(m, T, K):
    """fp32 scores where one wave takes the features of 16 rows (3072 row tiles, queries and keys, and more)."""
    from paper_2310_01777_amd import binding as sea
    wl = synth.Workload("features", 2, 13, T, 64, m, K, 4, 0, True, "f32", 4, 0.3)
    x = synth.make_inputs(wl)
    p = sea.SeaParams(B=2, H=13, T=T, d=64, m=m, K=K, k_hat=4, causal=True, scale=wl.scale, dtype="f32",
                      seq_len=x["seq_len"].cuda())
    A = torch.full((2, 13, T, K), float("nan"), device="cuda")
    print(f"[case] f32 features {(m, T, K)}", flush=True)
    sea.sea_estimate(p, x["Q"].cuda(), x["K"].cuda(), x["W"].cuda(), A, sea.alloc_workspace(p))
    want = oracle.estimate(oracle_params(wl), to_np64(x["Q"]), to_np64(x["K"]), to_np64(x["W"]), seq_len=x["seq_len"].numpy())
    assert_close(to_np64(A), want, TOL["f32"], "A_hat")
