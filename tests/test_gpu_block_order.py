"""Launches whose blocks are all resident deal their row tiles to the CUs in another order than shorter and longer
ones: a head computed among many has to come out as it does alone.  Column buckets of 1, 2 and 4 keys."""
import numpy as np
import pytest
import torch

from paper_2310_01777_amd import synth
from util import TOL

pytestmark = pytest.mark.gpu


# (dtype, heads, T, K): 296 tiles of 128 rows (two sets of waves, 592 blocks); 352 contraction and 693 attention tiles; 296 tiles of
# ragged columns (three sets, in the ordinary order); 783 tiles with one set of waves, of both kinds of columns: the last
# round that runs backwards has 15 of them; three whole rounds; two groups of heads, 72 and 65, of both kinds of columns
@pytest.mark.parametrize("dtype,H,T,K", [("bf16", 37, 1024, 64), ("f32", 11, 1000, 40), ("f32", 11, 1024, 128),
                                         ("bf16", 37, 999, 60), ("bf16", 87, 1152, 72), ("bf16", 87, 1100, 60), ("bf16", 96, 1024, 128),
                                         ("bf16", 137, 4096, 128), ("bf16", 137, 4000, 120)])
def test_a_head_among_many(dtype, H, T, K):
    from paper_2310_01777_amd import binding as sea
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(T + H)
    q, k, v = (torch.randn(1, H, T, 64, generator=g, device="cuda").to(td) for _ in range(3))
    W = synth.gaussian_orthogonal(64, 64, 3).to(td).cuda()

    def layer(q, k, v):
        p = sea.SeaParams(B=1, H=q.shape[1], T=T, d=64, m=64, K=K, k_hat=K // 4, causal=True, scale=0.125, dtype=dtype)
        O = torch.full_like(q, float("nan"))
        sea.sea_forward(p, q, k, v, W, O, workspace=sea.alloc_workspace(p))
        return O

    print(f"[case] block order {(dtype, H, T, K)}", flush=True)
    many = layer(q, k, v)
    assert torch.isfinite(many).all()  # every tile was written
    for h in (0, 1, H // 2, H - 1):
        alone = layer(*(x[:, h:h + 1].contiguous() for x in (q, k, v)))
        # the same products, perhaps merged from other parts: each within the contract's tolerance
        assert float((many[:, h] - alone[:, 0]).abs().max()) <= 2 * TOL[dtype] * float(alone.abs().max())


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("r,T", [(1, 1024), (2, 1024), (4, 2048)])
def test_buckets_of_few_keys(r, T, causal):
    import oracle
    from paper_2310_01777_amd import binding as sea
    from util import assert_close, oracle_params, to_np64
    K = 512
    g = torch.Generator().manual_seed(T + r)
    q, k, v = (torch.randn(1, 2, T, 64, generator=g).bfloat16() for _ in range(3))
    W = synth.gaussian_orthogonal(64, 64, 3).bfloat16()
    p = sea.SeaParams(B=1, H=2, T=T, d=64, m=64, K=K, k_hat=1, k_budget=r, causal=causal, scale=0.125, dtype="bf16")
    O = torch.empty_like(q).cuda()
    print(f"[case] buckets of few keys {(r, T, causal)}", flush=True)
    args = (p, q.cuda(), k.cuda(), v.cuda(), W.cuda())
    sea.sea_forward(*args, O, workspace=sea.alloc_workspace(p))
    idx, cnt = (torch.full(s, -1, dtype=torch.int32, device="cuda") for s in ((1, 2, T, r), (1, 2, T)))
    sea.sea_forward(*args, torch.empty_like(O), idx=idx, cnt=cnt, workspace=sea.alloc_workspace(p))
    want = oracle.sparse_attn(oracle_params(p), to_np64(q), to_np64(k), to_np64(v), idx.cpu().numpy(), cnt.cpu().numpy())
    assert np.isfinite(want).all()
    assert_close(to_np64(O), want, TOL["bf16"], "O")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("k_hat,H,T", [(1, 64, 1024), (2, 44, 4096)])
def test_buckets_of_many_heads(k_hat, H, T, causal):
    """More and fewer than 8192 chunks of 128 rows (one or four to a block): a head's rows come out alike.  The columns
    differ in the number of their rows, from none to several chunks of them, and some rows have no column."""
    from paper_2310_01777_amd import binding as sea
    K = 128
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn(1, H, T, 64, generator=g, device="cuda").bfloat16() for _ in range(3))
    col = (K * torch.rand(k_hat, 1, H, T, generator=g, device="cuda") ** 4).long()  # (the same one twice is one)
    bits = torch.zeros(1, H, T, K, dtype=torch.bool, device="cuda")
    for c in col:
        bits.scatter_(-1, c[..., None], True)
    bits[:, :, 7::50] = False
    words = (bits.view(1, H, T, K // 32, 32).long() << torch.arange(32, device="cuda")).sum(-1)
    mhat = torch.where(words >= 1 << 31, words - (1 << 32), words).int()

    def attend(h):
        n = h.stop - h.start
        p = sea.SeaParams(B=1, H=n, T=T, d=64, m=64, K=K, k_hat=k_hat, k_budget=k_hat * T // K, causal=causal, scale=0.125, dtype="bf16")
        O = torch.full((1, n, T, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.empty(sea.sea_mask_attn_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        assert ws.numel() > 0  # rows are grouped by column
        sea.sea_mask_attn(p, *(x[:, h].contiguous() for x in (q, k, v, mhat)), O, ws)
        return O

    print(f"[case] buckets of many heads {(k_hat, H, T, causal)}", flush=True)
    many = attend(slice(0, H))
    assert torch.isfinite(many).all() and bool((many[:, :, 7::50] == 0).all())
    for h in range(0, H, 20):
        some = slice(h, min(h + 20, H))
        assert torch.equal(many[:, some], attend(some))
