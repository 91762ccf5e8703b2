"""Layers whose rows select one column each (bidirectional, 65 to 128 columns, from 131072 rows on: the kernel that keeps a
head's whole state in LDS).  Values that name their column make the output name the selected column; it has to be the
first of the row's largest scores."""
import pytest
import torch

from paper_2310_01777_amd import binding as sea
from paper_2310_01777_amd import synth

pytestmark = pytest.mark.gpu


def _layer(B, H, T, m, K, seed):
    p = sea.SeaParams(B=B, H=H, T=T, d=64, m=m, K=K, k_hat=1, k_budget=16, causal=False, scale=0.125, dtype="bf16")
    g = torch.Generator().manual_seed(seed)
    q, k = (torch.randn(B, H, T, 64, generator=g) for _ in range(2))
    w = synth.gaussian_orthogonal(m, 64, seed)
    return p, q, k, w


def _columns(p, q, k, w):
    """The column each row's output names, and the scores."""
    col = (torch.arange(p.T) * p.K) // p.T
    v = col.to(torch.bfloat16)[None, None, :, None].expand(p.B, p.H, p.T, 64).contiguous().cuda()
    q, k, w = (x.to(torch.bfloat16).cuda() for x in (q, k, w))
    o = torch.empty_like(q)
    sea.sea_forward(p, q, k, v, w, o, workspace=sea.alloc_workspace(p))
    a = torch.empty(p.B, p.H, p.T, p.K, device="cuda")
    sea.sea_estimate(p, q, k, w, a, sea.alloc_workspace(p))
    assert torch.equal(o, o[..., :1].expand_as(o))
    # a layer that writes its scores as well comes to the same result
    o2, a2 = torch.full_like(o, float("nan")), torch.full_like(a, float("nan"))
    sea.sea_forward(p, q, k, v, w, o2, a2, workspace=sea.alloc_workspace(p))
    assert torch.equal(o, o2) and torch.equal(a, a2)
    return o[..., 0].float().cpu(), a.cpu()


def _first_largest(a):
    return (a == a.amax(-1, keepdim=True)).int().argmax(-1)


# whole tiles and rows past the last one, columns that fill their tiles and not, both feature counts
@pytest.mark.parametrize("B,H,T,m,K", [(1, 16, 8192, 128, 128), (2, 8, 8195, 64, 100), (1, 2, 65537, 128, 65),
                                       (1, 3, 43723, 64, 127), (1, 1, 131072, 128, 96)])
def test_first_largest_score(B, H, T, m, K):
    p, q, k, w = _layer(B, H, T, m, K, seed=T)
    got, a = _columns(p, q, k, w)
    assert torch.equal(got, _first_largest(a).float())
    # each score against 64 bits, at the tolerance of the estimate (bf16 features: 2e-2 of a row's largest)
    f = lambda x: x.to(torch.bfloat16).double()
    rows = torch.arange(0, T, max(T // 97, 1))
    scale = p.scale ** 0.5
    for h in range(0, B * H, max(B * H // 3, 1)):
        b, hh = divmod(h, H)
        phi = lambda x, s: torch.exp(scale * x @ f(w).T - 0.5 * p.scale * (x * x).sum(-1, keepdim=True) - s)
        fk = phi(f(k[b, hh]), 0.0)
        x = f(q[b, hh])[rows]
        fq = phi(x, (scale * x @ f(w).T - 0.5 * p.scale * (x * x).sum(-1, keepdim=True)).amax(-1, keepdim=True))
        s = fq @ torch.zeros(K, m, dtype=torch.double).index_add_(0, (torch.arange(T) * K) // T, fk).T
        s = s / s.sum(-1, keepdim=True)
        assert ((a[b, hh][rows] - s).abs().amax(-1) / s.amax(-1)).max() <= 2e-2


# keys that repeat from column to column: several columns hold the largest score, the first of them wins
@pytest.mark.parametrize("same", [128, 64, 2])
def test_equal_columns(same):
    p, q, k, w = _layer(1, 16, 8192, 128, 128, seed=same)
    k = k[:, :, : p.T // same].repeat(1, 1, same, 1)  # column c holds the keys of column c mod (128 / same)
    got, a = _columns(p, q, k, w)
    assert (got < 128 // same).all()
    assert torch.equal(got, _first_largest(a).float())


# columns whose scores differ by a few units in the last place, which the row's sum makes equal or not
@pytest.mark.parametrize("T,m,K", [(8192, 128, 128), (8200, 64, 100), (8195, 128, 65)])
def test_nearly_equal_columns(T, m, K):
    p, q, k, w = _layer(1, 16, T, m, K, seed=3)
    g = torch.Generator().manual_seed(4)
    k = k[:, :, :1] + 2.0 ** -6 * (torch.rand(1, 16, T, 64, generator=g) < 2.0 ** -10)
    got, a = _columns(p, q, k, w)
    assert torch.equal(got, _first_largest(a).float())


# A head among few goes to the kernel of all other layers, among many to this one.  The scores before their scaling are the same
# and the sum of a row's at most 128 is taken in another order: 35 and 65 additions in turn, (35 + 65 + 4) 2^-24 < 6.3e-6; two
# roundings each are left between the scores of one row.
@pytest.mark.parametrize("T,m,K", [(8192, 128, 128), (8195, 64, 100), (8200, 128, 65)])
def test_scores_of_a_head_among_many(T, m, K):
    p, q, k, w = _layer(1, 16, T, m, K, seed=5)
    q, k, w = (x.to(torch.bfloat16).cuda() for x in (q, k, w))
    out = []
    for H in (2, 16):
        p.H = H
        a = torch.full((1, H, T, K), float("nan"), device="cuda")
        sea.sea_estimate(p, q[:, :H].contiguous(), k[:, :H].contiguous(), w, a, sea.alloc_workspace(p))
        out.append(a[:, :2].double())
    ratio = out[1] / out[0]
    assert (ratio - 1).abs().max() < 6.3e-6
    assert (ratio.amax(-1) / ratio.amin(-1) - 1).max() < 4 * 2.0 ** -24 * 1.01
