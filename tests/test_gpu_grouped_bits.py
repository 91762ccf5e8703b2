"""Causal-per-batch selection when only the mask words are wanted (K a power of two): the counting passes, the
ranked bin and the tie walk, against the oracle's selection applied to the GPU's own scores."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_01777_amd import synth
from tests.test_gpu_parity import _sel_to_mask, _unpack_mhat
from tests.util import oracle_params

pytestmark = pytest.mark.gpu


# (B, H, T, m, K, k^, causal, pad), factor on Q and K
@pytest.mark.parametrize("case,factor", [
    ((2, 2, 200, 64, 32, 5, True, 0.3), 1.0),      # a slab of less than one group of every thread
    ((1, 12, 300, 128, 128, 100, True, 0.0), 1.0), # heads that end inside a group; most candidates taken
    ((1, 33, 130, 64, 32, 4, False, 0.0), 1.0),    # one head past a whole group
    ((1, 6, 600, 64, 512, 40, True, 0.3), 1.0),
    ((1, 3, 1030, 64, 1024, 200, True, 0.0), 1.0), # a group per head
    ((1, 32, 257, 64, 256, 64, True, 0.0), 1.0),   # 32 keys per thread
    ((1, 12, 300, 64, 128, 100, True, 0.0), 4.0),  # scores far below 2^-15 decide
    ((1, 8, 256, 64, 64, 60, False, 0.0), 6.0),    # and underflow to equal zeros
    ((1, 12, 256, 64, 128, 9, True, 0.0), 0.0),    # every score of a row the same: more ties than are ranked
    ((1, 1, 96, 64, 32, 7, True, 0.0), 0.0),       # fewer
], ids=lambda v: "_".join(str(x) for x in v) if isinstance(v, tuple) else str(v))
def test_grouped_bits(case, factor):
    from paper_2310_01777_amd import binding as sea
    B, H, T, m, K, kh, causal, pad = case
    wl = synth.Workload("grouped_bits", B, H, T, 64, m, K, kh, 0, causal, "bf16", 4, pad, grouping=1)
    x = synth.make_inputs(wl)
    d = {k: (x[k] * factor if k in "QK" else x[k]).cuda() for k in "QKVW"}
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=kh, causal=causal, scale=wl.scale, dtype="bf16", grouping=1,
                      seq_len=None if x["seq_len"] is None else x["seq_len"].cuda())
    out, ws = sea.alloc_outputs(p), sea.alloc_workspace(p)
    print(f"[case] grouped bits {case} {factor}", flush=True)
    sea.sea_forward(p, d["Q"], d["K"], d["V"], d["W"], out["O"], A_hat=out["A_hat"], workspace=ws, mhat=out["mhat"])
    torch.cuda.synchronize()
    sel, _, _ = oracle.topk_mask(oracle_params(wl), out["A_hat"].cpu().numpy().astype(np.float64),
                                 seq_len=None if x["seq_len"] is None else x["seq_len"].numpy())
    assert np.array_equal(_unpack_mhat(out["mhat"].cpu().numpy(), K), _sel_to_mask(sel, K))
