"""Causal decoder layers whose three convolutions run in one launch: strips of a multiple of four rows, whose first rows are
computed twice, so lengths around multiples of four, strips of one and of many steps, several sequences per round of blocks,
sequences that end inside a strip, and every number of channels and columns the kernel is built for."""
import pytest
import torch

import tests.test_gpu_decoder as base
from paper_2310_01777_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    base._wl("chain_4_heads_64_columns", 1, 4, 64, 64, 64, 8),
    base._wl("chain_4_heads_128_columns", 3, 4, 131, 64, 128, 8, pad_frac=0.4),
    base._wl("chain_8_heads_64_columns", 2, 8, 97, 64, 64, 8, pad_frac=0.4),
    base._wl("chain_8_heads_128_columns", 1, 8, 130, 64, 128, 8),
    base._wl("chain_12_heads_64_columns", 2, 12, 257, 64, 64, 8, pad_frac=0.4),
    base._wl("chain_12_heads_128_columns", 1, 12, 129, 64, 128, 8),
    base._wl("chain_long_strips", 20, 4, 399, 64, 64, 8),
    base._wl("chain_more_sequences_than_blocks", 260, 4, 66, 64, 64, 8, pad_frac=0.3),
    base._wl("chain_strips_of_32_rows", 20, 12, 360, 64, 128, 8, pad_frac=0.3),   # all layers at work, rings that wrap
]


@pytest.fixture(scope="module")
def sea():
    from paper_2310_01777_amd import binding
    return binding


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_decoder_sizes(sea, wl):
    base.test_decoder_matches_oracle(sea, wl)


@pytest.mark.parametrize("nonfinite", [False, True])
@pytest.mark.parametrize("K", [64, 128])
@pytest.mark.parametrize("H", [4, 8, 12])
def test_rows_do_not_depend_on_their_strip(sea, H, K, nonfinite):
    """A sequence alone is cut into strips of four rows, among twenty into strips of 36.  Queries and keys of zeros and
    whole values make the sums in front of the image exact, however they are split, so every row comes out the same;
    also where the image holds infinities and NaN."""
    B, T = 20, 399
    g = torch.Generator(device="cuda").manual_seed(H * K)
    q = torch.zeros(B, H, T, 64, dtype=torch.bfloat16, device="cuda")
    v = torch.randint(-2, 3, q.shape, generator=g, device="cuda").bfloat16()
    W = synth.gaussian_orthogonal(64, 64, 3).bfloat16().cuda()
    wd = {k: w.cuda() for k, w in synth.decoder_weights(H, 64, K, seed=H + K).items()}
    if nonfinite:   # channels 1 of column 1 and 2 of column 9
        wd["nu2_b"] = wd["nu2_b"].clone()
        wd["nu2_b"][5], wd["nu2_b"][38] = float("inf"), float("nan")
    seq = torch.randint(T // 2, T + 1, (B,), generator=torch.Generator().manual_seed(K)).int().cuda()

    def estimate(b):
        n = b.stop - b.start
        p = sea.SeaParams(B=n, H=H, T=T, d=64, m=64, K=K, k_hat=8, causal=True, scale=0.125, dtype="bf16", seq_len=seq[b].contiguous())
        A = torch.full((n, H, T, K), -1.0, device="cuda")
        ws = torch.empty(sea.sea_decoder_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        print(f"[case] strips H{H} K{K} nonfinite{int(nonfinite)} sequences {b.start}..{b.stop}", flush=True)
        sea.sea_decoder_estimate(p, wd, q[b].contiguous(), q[b].contiguous(), v[b].contiguous(), W, A, ws)
        return A

    together = estimate(slice(0, B))
    assert (together != 0).any() and torch.isnan(together).any().item() in (False, nonfinite)
    for b in (0, 7, B - 1):
        alone = estimate(slice(b, b + 1))[0]
        assert torch.equal(torch.isnan(alone), torch.isnan(together[b]))
        assert torch.equal(alone.nan_to_num(-2.0), together[b].nan_to_num(-2.0))
