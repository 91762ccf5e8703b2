"""Per-row widths, bf16: the estimate that selects its rows' columns and writes the key bits itself, at the sizes
where its column parts, row tiles and key-bit words change, against the selection made from the scores in
memory (itself checked against the oracle) and the oracle's attention on it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_01777_amd import synth
from tests.util import TOL, assert_close, oracle_params, to_np64

pytestmark = pytest.mark.gpu


# (B, H, T, m, K, k^, budget, pad)
@pytest.mark.parametrize("case", [
    (1, 2, 40, 64, 40, 3, 0, 0.0),         # every row narrower than K but the last
    (2, 2, 65, 64, 33, 9, 0, 0.3),         # two parts of 17 and 16 columns
    (1, 3, 129, 128, 128, 40, 0, 0.0),     # rows of K - 1, K and K + 1 keys
    (1, 2, 500, 128, 100, 30, 60, 0.0),    # parts of 25 columns; two keys of up to five
    (2, 1, 700, 64, 250, 60, 250, 0.5),    # eight parts, four keys of up to three: every key
    (1, 2, 300, 256, 128, 128, 0, 0.0),    # m = 256: 64-row blocks; every column
    (1, 1, 1025, 256, 200, 1, 0, 0.3),     # seven parts, one column
    (1, 1, 2049, 64, 64, 20, 0, 0.0),      # two parts share two waves' room
    (1, 1, 4100, 128, 128, 20, 0, 0.0),    # rows of 129 words
    # a 64-row block per CU: where the estimate selects
    (4, 64, 40, 64, 40, 3, 0, 0.0),
    (4, 32, 65, 64, 33, 9, 0, 0.3),
    (2, 43, 129, 128, 128, 40, 0, 0.0),
    (4, 8, 500, 128, 100, 30, 60, 0.0),
    (2, 12, 700, 64, 125, 30, 250, 0.5),   # eight keys of up to six: every key
    (3, 18, 300, 256, 128, 128, 0, 0.0),
    (1, 16, 1025, 256, 128, 1, 0, 0.3),
    (1, 8, 2049, 64, 64, 20, 0, 0.0),
    (1, 4, 4100, 128, 128, 20, 0, 0.0),
    (3, 28, 130, 64, 129, 40, 0, 0.0),     # K above 128: not there
    (1, 12, 4200, 64, 64, 4, 0, 0.0),      # attention: four sets of four waves (385 to 512 blocks of 128 rows)
    (1, 25, 2050, 64, 64, 4, 0, 0.0),      # 64 rows and two sets of two waves (385 to 896)
    (1, 11, 4100, 256, 64, 4, 0, 0.3),     # all heads together, each on all XCDs
    (1, 17, 2050, 128, 128, 4, 0, 0.3),    # head after head: an odd number
    (1, 12, 4100, 256, 250, 4, 0, 0.3),    # groups of 8 and 4 heads
    (1, 20, 2050, 256, 64, 4, 0, 0.3),     # all heads together, more than an L2's share
    (1, 12, 1601, 64, 128, 4, 0, 0.3),     # all heads together, on two XCDs each
    (1, 36, 1024, 64, 100, 4, 0, 0.3),     # head after head: a little more than one round
    (3, 12, 640, 64, 64, 4, 0, 0.0),       # few tiles
], ids=lambda c: "_".join(str(x) for x in c))
def test_selection_in_the_estimate(case):
    from paper_2310_01777_amd import binding as sea
    B, H, T, m, K, kh, kb, pad = case
    wl = synth.Workload("row_width", B, H, T, 64, m, K, kh, kb, True, "bf16", 4, pad, geometry=1)
    x = synth.make_inputs(wl)
    d = {k: x[k].cuda() for k in "QKVW"}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, k_budget=kb, causal=True, scale=wl.scale, dtype="bf16",
                      geometry=1, seq_len=None if x["seq_len"] is None else x["seq_len"].cuda())
    out, ws = sea.alloc_outputs(p), sea.alloc_workspace(p)
    print(f"[case] row width {case}", flush=True)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], out["O"], out["A_hat"], out["sel"], out["idx"], out["cnt"], ws,
                    mhat=out["mhat"])
    O2, O3 = torch.full_like(out["O"], float("nan")), torch.full_like(out["O"], float("nan"))
    mhat, A = torch.full_like(out["mhat"], -1), torch.full_like(out["A_hat"], float("nan"))
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O2, workspace=ws)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O3, A_hat=A, mhat=mhat, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(mhat, out["mhat"]) and torch.equal(A, out["A_hat"])
    assert torch.equal(O2, out["O"]) and torch.equal(O3, out["O"])
    want = oracle.sparse_attn(oracle_params(wl), to_np64(x["Q"]), to_np64(x["K"]), to_np64(x["V"]),
                              out["idx"].cpu().numpy(), out["cnt"].cpu().numpy())
    assert_close(to_np64(out["O"]), want, TOL["bf16"], "O")
