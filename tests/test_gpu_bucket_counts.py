"""Rows per column for the attention that groups rows by column: the kernels of the estimate zero them (and, for one column
per row, count them).  A workspace full of other numbers, used twice, has to give what a zeroed one gives."""
import pytest
import torch

from paper_2310_01777_amd import binding as sea
from paper_2310_01777_amd import synth

pytestmark = pytest.mark.gpu


# counted by the rows kernel (power-of-two columns and others); zeroed by the key kernel in blocks of four and eight waves, by the
# one of other widths (12 keys, 8 of them kept), with fewer threads than counters, several columns a row, causal and padded
@pytest.mark.parametrize("B,H,T,m,K,k_hat,k_budget,causal,pad", [
    (1, 16, 8192, 128, 128, 1, 16, False, 0.0), (1, 12, 12800, 64, 100, 1, 64, False, 0.0), (1, 2, 96000, 128, 96, 1, 8, False, 0.0),
    (1, 2, 512, 256, 256, 1, 2, True, 0.0), (2, 2, 1024, 64, 16, 1, 64, False, 0.3), (1, 2, 4096, 128, 8, 1, 32, True, 0.0),
    (1, 3, 3072, 64, 256, 1, 8, False, 0.0), (1, 2, 4096, 128, 64, 3, 48, True, 0.0), (2, 1, 8192, 256, 64, 8, 512, False, 0.2)])
def test_workspace_of_other_numbers(B, H, T, m, K, k_hat, k_budget, causal, pad):
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=k_hat, k_budget=k_budget, causal=causal, scale=0.125, dtype="bf16")
    g = torch.Generator().manual_seed(T + K)
    q, k, v = (torch.randn(B, H, T, 64, generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    w = synth.gaussian_orthogonal(m, 64, 1).to(torch.bfloat16).cuda()
    if pad:
        p.seq_len = torch.tensor([T - int(pad * T * i) for i in range(B)], dtype=torch.int32, device="cuda")
    ws = sea.alloc_workspace(p)
    outs = []
    for fill in (0, 0x5a, None):  # (None: as the call before left it)
        if fill is not None:
            ws.fill_(fill)
        o = torch.full_like(q, float("nan"))
        sea.sea_forward(p, q, k, v, w, o, workspace=ws)
        outs.append(o)
    assert not outs[0].isnan().any()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
