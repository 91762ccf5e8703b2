"""Sequences that end at, just before and just behind the edge of a tile, or are empty: row and key tiles with nothing but
padding are not computed, and leave zeros where something may have been before."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_01777_amd import synth
from tests.util import TOL, assert_close, oracle_params, to_np64

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 16, 63, 64, 65, 128, 129, 255, 256]  # of 512 or 500 tokens

# (T, m, K, k^, budget): two, four, eight, sixteen, 32 and 128 keys per column; 256; columns of other widths
SHAPES = [(512, 64, 256, 40, 0), (512, 64, 128, 40, 0), (512, 128, 64, 20, 0), (512, 64, 32, 12, 0), (512, 256, 16, 9, 64),
          (512, 64, 4, 2, 0), (512, 64, 2, 2, 128), (512, 64, 512, 60, 0), (500, 64, 128, 40, 0), (500, 128, 33, 12, 0)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "_".join(map(str, s)))
def test_tiles_of_padding(dtype, shape, causal):
    from paper_2310_01777_amd import binding as sea
    T, m, K, kh, kb = shape
    B, H = len(LENGTHS), 2
    wl = synth.Workload("padding", B, H, T, 64, m, K, kh, kb, causal, dtype, 4)
    x = synth.make_inputs(wl)
    seq = torch.tensor(LENGTHS, dtype=torch.int32)
    d = {k: x[k].cuda() for k in "QKVW"}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, k_budget=kb, causal=causal, scale=wl.scale, dtype=dtype,
                      seq_len=seq.cuda())
    out, ws = sea.alloc_outputs(p), sea.alloc_workspace(p)
    for o in list(out.values()) + [ws]:  # (bytes that are NaN in every type)
        o.view(torch.uint8).fill_(255)
    print(f"[case] padding {dtype} {shape} causal={causal}", flush=True)
    O2 = torch.full_like(out["O"], float("nan"))
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], O2, workspace=ws)
    ws.fill_(255)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], out["O"], out["A_hat"], out["sel"], out["idx"], out["cnt"], ws)
    assert torch.equal(O2, out["O"])
    po, sl = oracle_params(wl), seq.numpy()
    A = out["A_hat"].cpu().numpy().astype(np.float64)
    assert_close(A, oracle.estimate(po, to_np64(x["Q"]), to_np64(x["K"]), to_np64(x["W"]), seq_len=sl), TOL[dtype], "A_hat")
    sel, idx, cnt = oracle.topk_mask(po, A, seq_len=sl)
    assert np.array_equal(out["cnt"].cpu().numpy(), cnt)
    want = oracle.sparse_attn(po, to_np64(x["Q"]), to_np64(x["K"]), to_np64(x["V"]), idx, cnt)
    assert_close(to_np64(out["O"]), want, TOL[dtype], "O")
    for b, n in enumerate(LENGTHS):
        assert not out["O"][b, :, n:].any() and not A[b, :, n:].any()
