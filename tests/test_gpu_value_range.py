"""bf16 attention whose scores rise, fall, jump or stay along the keys, with values from nearly the smallest to nearly the
largest the type holds: the running reference of the softmax may cost neither end of the range.  Every key is selected."""
import pytest
import torch

from paper_2310_01777_amd import synth

pytestmark = pytest.mark.gpu

T = 512
# scores in log2 units; a jump of 47 in the middle, where half of the keys share the largest weight
SCORES = {"flat": torch.zeros(T), "rise": torch.linspace(0, 90, T), "fall": torch.linspace(0, -90, T),
          "jump": 47.0 * (torch.arange(T) >= T // 2)}

# how, heads, K, k^, geometry: 64-row blocks and 128-row blocks of tiles, key bits, a bucket of 512 keys, the dense kernel,
# columns of any width
LAYERS = [("layer", 2, 64, 64, 0), ("layer", 70, 16, 16, 0), ("layer", 2, 64, 64, 1), ("layer", 2, 1, 1, 0),
          ("dense", 2, 64, 64, 0), ("layer", 2, 60, 60, 0)]


@pytest.mark.parametrize("exponent", [-125, -118, 0, 106])
@pytest.mark.parametrize("scores", SCORES)
@pytest.mark.parametrize("how,H,K,k_hat,geometry", LAYERS)
def test_values_of_any_size(how, H, K, k_hat, geometry, scores, exponent):
    from paper_2310_01777_amd import binding as sea
    g = torch.Generator(device="cuda").manual_seed(H + K)
    q, k = (torch.zeros(1, H, T, 64, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    q[..., 0] = 8.0
    k[..., 0] = (SCORES[scores] / 1.4426950408889634).bfloat16().cuda()
    v = ((1 + torch.rand(1, H, T, 64, generator=g, device="cuda")).double() * 2.0 ** exponent).bfloat16()
    causal = geometry == 1
    p = sea.SeaParams(B=1, H=H, T=T, d=64, m=64, K=K, k_hat=k_hat, causal=causal, scale=0.125, dtype="bf16", geometry=geometry)
    O = torch.empty_like(q)
    print(f"[case] values {(how, H, K, geometry, scores, exponent)}", flush=True)
    if how == "dense":
        sea.sea_dense_attn(p, q, k, v, O)
    else:
        sea.sea_forward(p, q, k, v, synth.gaussian_orthogonal(64, 64, 3).bfloat16().cuda(), O, workspace=sea.alloc_workspace(p))
    s = (k[0, 0, :, 0].double() * (8.0 * 0.125)).expand(T, T)
    if causal:
        s = s.masked_fill(torch.ones(T, T, device="cuda", dtype=torch.bool).triu(1), -torch.inf)
    want = torch.softmax(s, -1) @ v.double()
    # weights of 8 bits, the same ones in the sum: 2^-9 each; the result rounded: 2^-9; exponents of up to 90 in 24 bits: 2^-17
    assert float(((O.double() - want) / want).abs().max()) <= 2.0 ** -9 * 2 + 2.0 ** -9 + 2.0 ** -17
