"""The selection inside the estimate's rows kernels against the stand-alone one on the same scores: the same columns, row by
row, where the search for a row's threshold has little to go by -- quotas of one, of all columns but one or two, equal
scores, scores over many octaves and over a few units in the last place -- and at the edges of tiles, stages and sequences."""
import pytest
import torch

from paper_2310_01777_amd import binding as sea
from paper_2310_01777_amd import synth

pytestmark = pytest.mark.gpu

# T, m, K, causal, pad: one key per column; 16-, 8- and 32-key columns; columns of any width; all three numbers of tiles, full
# and not; several heads of a padded batch
SHAPES = [(64, 64, 64, True, 0.0), (2048, 128, 128, True, 0.0), (2048, 256, 256, True, 0.3), (4096, 256, 128, True, 0.0),
          (333, 64, 20, True, 0.3), (1000, 128, 100, False, 0.3), (1000, 128, 200, True, 0.0), (256, 128, 32, False, 0.3),
          (515, 256, 256, False, 0.0), (2000, 256, 256, True, 0.3)]


def _inputs(kind, T, K, seed):
    g = torch.Generator().manual_seed(seed)
    q, k = (torch.randn(2, 3, T, 64, generator=g) for _ in range(2))
    if kind == "peaked":     # scores over dozens of octaves
        q, k = 3.0 * q, 3.0 * k
    elif kind == "close":    # scores that differ in their last bits only
        k = k[:, :, :1] + 2.0 ** -9 * k
    elif kind == "equal":    # seven keys, again and again
        k = k[:, :, (torch.arange(T) % 7)]
    return q, k


@pytest.mark.parametrize("kind", ["plain", "peaked", "close", "equal"])
@pytest.mark.parametrize("T,m,K,causal,pad", SHAPES)
def test_same_columns_as_alone(T, m, K, causal, pad, kind):
    q, k = _inputs(kind, T, K, seed=T + K)
    w = synth.gaussian_orthogonal(m, 64, 1)
    q, k, w = (x.to(torch.bfloat16).cuda() for x in (q, k, w))
    lens = synth.padding_lengths(2, T, pad, 5).cuda() if pad else None
    for k_hat in sorted({1, 2, 3, K // 8, K // 2, K - 2, K - 1, K} - {0}):
        p = sea.SeaParams(B=2, H=3, T=T, d=64, m=m, K=K, k_hat=k_hat, causal=causal, scale=0.125, dtype="bf16", seq_len=lens)
        print(f"[case] selection {(T, m, K, causal, pad, kind, k_hat)}", flush=True)
        words = torch.zeros(2, 3, T, (K + 31) // 32, dtype=torch.int32, device="cuda")
        sea.sea_forward(p, q, k, k, w, torch.empty_like(q), workspace=sea.alloc_workspace(p), mhat=words)
        out = sea.alloc_outputs(p)
        sea.sea_estimate(p, q, k, w, out["A_hat"], sea.alloc_workspace(p))
        sea.sea_topk_mask(p, out["A_hat"], out["sel"], out["idx"], out["cnt"])
        got = ((words[..., None] >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1).flatten(-2)[..., :K]
        sel = out["sel"].long()
        want = torch.zeros(2, 3, T, K + 1, dtype=torch.int32, device="cuda")
        want.scatter_(-1, torch.where(sel < 0, K, sel), 1)
        assert torch.equal(got, want[..., :K])
