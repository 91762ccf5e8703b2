"""bf16 tensors, softmax weights held in fp32: where the key lists are walked in tiles, a weight may not lose bits on
its way into the matrix product.  Checked against 64 bits at the outputs that nearly cancel."""
import pytest
import torch

from paper_2310_01777_amd import synth

pytestmark = pytest.mark.gpu


# (B, H, T, K): 8, 16 and 32 column slots, six, three and one set of waves; lists in tiles
@pytest.mark.parametrize("how,B,H,T,K", [("layer", 1, 24, 601, 100), ("layer", 1, 64, 499, 128), ("layer", 4, 64, 250, 140),
                                         ("layer", 2, 64, 333, 50), ("lists", 1, 64, 601, 100)])
def test_weights_keep_their_bits(how, B, H, T, K):
    from paper_2310_01777_amd import binding as sea
    g = torch.Generator(device="cuda").manual_seed(T)
    # entries of -1, 0, 1: q.k is a whole number, exact in fp32; every key is attended
    q, k = (torch.randint(-1, 2, (B, H, T, 64), generator=g, device="cuda").bfloat16() for _ in range(2))
    v = torch.randn(B, H, T, 64, generator=g, device="cuda").bfloat16()
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=64, K=K, k_hat=K, causal=False, scale=0.125, dtype="bf16")
    O = torch.empty_like(q)
    print(f"[case] weights {how} {(B, H, T, K)}", flush=True)
    if how == "layer":
        W = synth.gaussian_orthogonal(64, 64, 3).bfloat16().cuda()
        sea.sea_forward(p, q, k, v, W, O, workspace=sea.alloc_workspace(p))
    else:
        idx = torch.arange(T, dtype=torch.int32, device="cuda").expand(B, H, T, T).contiguous()
        sea.sea_sparse_attn(p, q, k, v, idx, torch.full((B, H, T), T, dtype=torch.int32, device="cuda"), T, O)
    want = torch.softmax(q.double() @ k.double().transpose(-1, -2).contiguous() * 0.125, -1) @ v.double()
    rms = want.square().mean().sqrt()
    small = want.abs() < rms * 2.0 ** -12
    assert int(small.sum()) >= 100
    # The result's own rounding is at most 2^-21 rms there.  A weight off by a share e moves an output by e rms
    # (the keys' signs are random): fp32 weights are off by 2^-22 (the exponential, |y| <= 6 rounded to 24
    # bits), weights of 16 significant bits by 2^-18.6 in the mean.
    err = (O.double() - want)[small].square().mean().sqrt() / rms
    assert float(err) <= 2.0 ** -20


# (the argument of exp2 against a reference 32 above the scores is off by 2^-21, which reads 2^-20.4 here)
@pytest.mark.parametrize("how,B,H,T,K", [("layer", 1, 64, 2001, 128), ("lists", 1, 64, 601, 100)])
def test_weights_that_count_have_small_arguments(how, B, H, T, K):
    from paper_2310_01777_amd import binding as sea
    g = torch.Generator(device="cuda").manual_seed(T)
    q, k = (torch.randint(-1, 2, (B, H, T, 64), generator=g, device="cuda").bfloat16() for _ in range(2))
    v = torch.randn(B, H, T, 64, generator=g, device="cuda").bfloat16()
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=64, K=K, k_hat=K, causal=False, scale=0.125, dtype="bf16")
    O = torch.empty_like(q)
    print(f"[case] weights, reference {how} {(B, H, T, K)}", flush=True)
    if how == "layer":
        W = synth.gaussian_orthogonal(64, 64, 3).bfloat16().cuda()
        sea.sea_forward(p, q, k, v, W, O, workspace=sea.alloc_workspace(p))
    else:
        idx = torch.arange(T, dtype=torch.int32, device="cuda").expand(B, H, T, T).contiguous()
        sea.sea_sparse_attn(p, q, k, v, idx, torch.full((B, H, T), T, dtype=torch.int32, device="cuda"), T, O)
    want = torch.softmax(q.double() @ k.double().transpose(-1, -2).contiguous() * 0.125, -1) @ v.double()
    rms = want.square().mean().sqrt()
    small = want.abs() < rms * 2.0 ** -12
    # result rounded: at most 2^-21; weights of 24 bits, |argument| <= 8: 2^-22.  Together sqrt(2^-42 + 2^-44).
    err = (O.double() - want)[small].square().mean().sqrt() / rms
    assert float(err) <= 2.0 ** -20.8
