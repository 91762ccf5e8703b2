"""fp32 layers whose estimator selects the columns itself: the same mask as with the lists asked for, which takes the selection's own
kernel.  One and, from 112 blocks of 32 rows on, two slots of 64 columns, partial mask words, rows past a multiple of the 32 of a
block, quotas of one, of some and of all columns, rows of equal scores, and values that are not finite."""
import pytest
import torch

from paper_2310_01777_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inputs", ["random", "equal", "nonfinite"])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("T,K,k_hat,pad", [(256, 64, 8, 0.0), (257, 64, 1, 0.3), (320, 128, 128, 0.0), (333, 100, 17, 0.4), (40, 33, 5, 0.0),
                                           (96, 1, 1, 0.0), (700, 128, 128, 0.0), (690, 100, 17, 0.4), (673, 65, 65, 0.0)])
def test_same_mask_as_with_lists(T, K, k_hat, pad, causal, inputs):
    from paper_2310_01777_amd import binding as sea
    B, H = 2, 3
    g = torch.Generator(device="cuda").manual_seed(T + K)
    q, k, v = (torch.randn(B, H, T, 64, generator=g, device="cuda") for _ in range(3))
    if inputs == "equal":
        q, k = torch.zeros_like(q), torch.zeros_like(k)
    elif inputs == "nonfinite":
        q[0, 0, T // 2, 3], k[0, 1, T // 3, 5], k[1, 2, 1, 0] = float("nan"), float("inf"), -float("nan")
    W = synth.gaussian_orthogonal(64, 64, 3).float().cuda()
    seq = synth.padding_lengths(B, T, pad, 1).cuda() if pad else None
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=64, K=K, k_hat=k_hat, causal=causal, scale=0.125, dtype="f32", seq_len=seq)
    print(f"[case] fp32 selection {(T, K, k_hat, pad, causal, inputs)}", flush=True)
    words = (K + 31) // 32
    mask, want = (torch.full((B, H, T, words), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    O, want_O = torch.empty_like(q), torch.empty_like(q)
    cnt = torch.empty(B, H, T, dtype=torch.int32, device="cuda")
    sea.sea_forward(p, q, k, v, W, want_O, cnt=cnt, mhat=want, workspace=sea.alloc_workspace(p))
    sea.sea_forward(p, q, k, v, W, O, mhat=mask, workspace=sea.alloc_workspace(p))
    assert torch.equal(mask, want)
    assert torch.equal(O.view(torch.int32), want_O.view(torch.int32))
    A, want_A = torch.empty(B, H, T, K, device="cuda"), torch.empty(B, H, T, K, device="cuda")
    sea.sea_forward(p, q, k, v, W, want_O, A_hat=want_A, cnt=cnt, workspace=sea.alloc_workspace(p))
    sea.sea_forward(p, q, k, v, W, O, A_hat=A, workspace=sea.alloc_workspace(p))
    assert torch.equal(A.view(torch.int32), want_A.view(torch.int32))
