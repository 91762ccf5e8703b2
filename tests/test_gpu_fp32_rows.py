"""fp32 attention in tiles: accumulators are rescaled only when some row's maximum rises, chunks of 16 keys alternate
between two sets of registers.  Scores that rise, fall and repeat along the keys, against 64 bits."""
import pytest
import torch

from paper_2310_01777_amd import synth

pytestmark = pytest.mark.gpu


# T: one chunk, two, chunks for some of the four waves, an odd and an even number for all; columns of one and 65 keys
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("T,K", [(16, 16), (32, 32), (80, 16), (144, 16), (1040, 16), (50, 20), (333, 50)])
def test_scores_along_the_keys(T, K, causal):
    from paper_2310_01777_amd import binding as sea
    H, d = 3, 64
    g = torch.Generator(device="cuda").manual_seed(T)
    q = torch.randn(1, H, T, d, generator=g, device="cuda")
    v = torch.randn(1, H, T, d, generator=g, device="cuda")
    # head 0: scores rise by 40 along the keys, head 1: they fall, head 2: all alike
    ramp = torch.linspace(0, 40, T, device="cuda")
    k = torch.zeros(1, H, T, d, device="cuda")
    q[..., 0], k[0, 0, :, 0], k[0, 1, :, 0] = 8.0, ramp, -ramp
    k[0, :2, :, 1:] = 0.1 * torch.randn(2, T, d - 1, generator=g, device="cuda")
    p = sea.SeaParams(B=1, H=H, T=T, d=d, m=64, K=K, k_hat=K, causal=causal, scale=0.125, dtype="f32")
    W = synth.gaussian_orthogonal(64, 64, 3).float().cuda()
    O = torch.empty_like(q)
    print(f"[case] fp32 rows {(T, K, causal)}", flush=True)
    sea.sea_forward(p, q, k, v, W, O, workspace=sea.alloc_workspace(p))
    s = (q.double() @ k.double().transpose(-1, -2).contiguous()) * 0.125
    if causal:
        s = s.masked_fill(torch.ones(T, T, device="cuda", dtype=torch.bool).triu(1), -torch.inf)
    want = torch.softmax(s, -1) @ v.double()
    # weights: argument rounded to 24 bits (|y| <= 60: 2^-19 at most, times ln 2) and the exponential's last bit, on
    # both sides of the quotient; sums of T terms: T 2^-24 of the largest |v| (5) at the very most
    assert float((O.double() - want).abs().max()) <= 5.0 * (2 * 2.0 ** -19 + T * 2.0 ** -24)
