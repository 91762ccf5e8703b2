"""Workloads that stand for what a user of this library runs: whole attention layers through the
public entry points of `binding.py`, from one short sentence to the longest sequences, over every
tensor type, direction and option the layer has.

A case is a dict of plain values.  `kind` says which calls a pass makes:
  forward   sea_forward into an output tensor
  decoder   sea_decoder_estimate (the paper's learned estimator; weights laid out once)
  stages    sea_estimate -> sea_topk_mask -> sea_flatcsr -> sea_flatcsr_attn -> sea_output_mix,
            for callers who want the intermediate tensors in the paper's own format
The other values are those of `SeaParams`, the number of key clusters per head (`centroids`) and the
largest share of right padding (`pad`).
"""
import numpy as np
import torch

from paper_2310_01777_amd import binding as sea
from paper_2310_01777_amd import synth

D = 64  # head dimension of every layer


def _case(kind, B, H, T, m, K, k_hat, k_budget=0, causal=True, dtype="bf16", centroids=16, pad=0.0, grouping=0,
          geometry=0):
    return dict(kind=kind, B=B, H=H, T=T, m=m, K=K, k_hat=k_hat, k_budget=k_budget, causal=causal, dtype=dtype,
                centroids=centroids, pad=pad, grouping=grouping, geometry=geometry)


def listed():
    return [
        # one sentence through a BERT-base-shaped layer (T = 256, K = 32, k = 25): latency
        dict(_case("forward", 1, 12, 256, 128, 32, 3, 25, False, centroids=8), name="bert_one_sentence"),
        # a padded batch of 32 through the same kind of layer (configuration c5)
        dict(_case("forward", 32, 12, 512, 128, 64, 16, 0, False, centroids=8, pad=0.25), name="bert_batch"),
        # OPT-125m-shaped layer on fp32 tensors (configuration c1)
        dict(_case("forward", 1, 12, 1024, 128, 128, 32, dtype="f32"), name="opt125m_fp32"),
        # OPT-125m-shaped layer, bf16 (configuration c2)
        dict(_case("forward", 4, 12, 2048, 128, 128, 64), name="opt125m"),
        # OPT-1.3B-shaped layer (configuration c3)
        dict(_case("forward", 8, 32, 2048, 256, 256, 64, centroids=64), name="opt1b3"),
        # long context, fixed key budget (configuration c4 at its longest)
        dict(_case("forward", 1, 32, 32768, 256, 256, 64, 512, centroids=64), name="long_context"),
        # the paper's efficiency runs: random inputs, k = 64 fixed, longest length of its table (c6)
        dict(_case("forward", 1, 12, 131072, 128, 128, 1, 64, False), name="fixed_k_128k"),
        # a batch of prompts cut at 2000 tokens: no multiple of K, every sequence of its own length
        dict(_case("forward", 8, 32, 2000, 256, 256, 64, centroids=64, pad=0.25), name="prompts_ragged"),
        # c3 with the paper's causal-per-batch selection
        dict(_case("forward", 8, 32, 2048, 256, 256, 64, centroids=64, grouping=1), name="opt1b3_grouped"),
        # c2 in the paper's per-row causal width
        dict(_case("forward", 4, 12, 2048, 128, 128, 64, geometry=1), name="opt125m_row_width"),
        # the paper's MLP + CNN estimator on the c2 layer
        dict(_case("decoder", 4, 12, 2048, 128, 128, 64), name="opt125m_decoder"),
        # c2 stage by stage with the FlatCSR tensor in between and the output mixing at the end
        dict(_case("stages", 4, 12, 2048, 128, 128, 64), name="opt125m_stages"),
    ]


def _row_len(T, K, k_hat, k_budget):
    """Most keys a row of one head can list."""
    w = -(-T // K)
    return k_hat * (w if k_budget == 0 else min(w, max(1, k_budget // k_hat)))


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _length(rng, lo, hi, K):
    """A sequence length, log-uniform: one half multiples of K (callers who pad to the column grid),
    one half any length (callers who do not)."""
    T = max(_log_int(rng, lo, hi), K)
    return max(T // K, 1) * K if rng.random() < 0.5 else min(T | 1, hi)


def _batch(rng, H, T, most, rows, row_len=0):
    """Sequences per batch, log-uniform, within `rows` rows of all heads (and 2^28 listed keys, about what
    prompts_ragged has)."""
    if row_len:
        rows = min(rows, (1 << 28) // row_len)
    return max(1, min(_log_int(rng, 1, most), rows // (H * T)))


def draw(rng):
    family = rng.choice(["opt125m", "opt1b3", "bert", "fixed_k", "f32", "grouped", "row_width", "decoder", "stages"])
    rows = 1 << 19  # rows of all heads: those of the c3 layer
    if family == "opt125m":
        T = _length(rng, 256, 16384, 128)
        k_hat, budget = rng.choice([16, 32, 48, 64]), 512 if T > 4096 else 0
        return _case("forward", _batch(rng, 12, T, 8, rows, _row_len(T, 128, k_hat, budget)), 12, T, 128, 128, k_hat,
                     budget, pad=rng.choice([0.0, 0.25]))
    if family == "opt1b3":
        T = _length(rng, 512, 16384, 256)
        k_hat, budget = rng.choice([32, 64, 96]), 512 if T > 2048 else 0
        return _case("forward", _batch(rng, 32, T, 8, rows, _row_len(T, 256, k_hat, budget)), 32, T, 256, 256, k_hat,
                     budget, centroids=64, pad=rng.choice([0.0, 0.25]))
    if family == "bert":
        K, k = rng.choice([32, 64]), rng.choice([25, 64, 128])
        T = _length(rng, 128, 2048, K)
        k_hat = max(1, (2 * k * K + T) // (2 * T))
        return _case("forward", _batch(rng, 12, T, 64, rows), 12, T, 128, K, min(k_hat, K), k, False, centroids=8,
                     pad=0.25)
    if family == "fixed_k":
        # lengths of the paper's latency table
        T, k = 1 << rng.randint(12, 16), rng.choice([32, 64, 128])
        k_hat = max(1, (2 * k * 128 + T) // (2 * T))
        return _case("forward", rng.randint(1, 2), rng.choice([8, 12, 16]), T, 128, 128, k_hat, k, rng.random() < 0.5)
    if family == "f32":
        T = _length(rng, 256, 4096, 128)
        return _case("forward", _batch(rng, 12, T, 4, 1 << 17), 12, T, 128, 128, rng.choice([16, 32]), 0,
                     rng.random() < 0.7, "f32", pad=rng.choice([0.0, 0.25]))
    if family == "grouped":
        H, K = rng.choice([(12, 128), (32, 256)])
        T = _length(rng, 512, 4096, K)
        return _case("forward", _batch(rng, H, T, 8, 1 << 18), H, T, K, K, rng.choice([32, 64]), 512 if T > 2048 else 0,
                     centroids=64, grouping=1)
    if family == "row_width":
        T = _length(rng, 256, 4096, 128)
        return _case("forward", _batch(rng, 12, T, 4, 1 << 17), 12, T, 128, 128, rng.choice([32, 64]), geometry=1,
                     pad=rng.choice([0.0, 0.25]))
    if family == "decoder":
        K = rng.choice([64, 128])
        T = _length(rng, 256, 2048, K)
        return _case("decoder", _batch(rng, 12, T, 8, 1 << 17), 12, T, 128, K, K // 2, 0, rng.random() < 0.6,
                     pad=rng.choice([0.0, 0.25]))
    T = 1 << rng.randint(8, 11)
    return _case("stages", _batch(rng, 12, T, 8, 1 << 17), 12, T, 128, 128, rng.choice([16, 32, 48, 64]), 0,
                 rng.random() < 0.7)


def _inputs(c, seed):
    """Q, K, V as in `synth.clustered_qkv` (queries and keys of a token share a cluster centroid), drawn on
    the GPU; a Gaussian-orthogonal projection W."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, H, T, n = c["B"], c["H"], c["T"], c["centroids"]
    dt = synth.torch_dtype(c["dtype"])
    mu = torch.randn(B, H, n, D, generator=g, device="cuda")
    z = torch.randint(0, n, (B, H, T), generator=g, device="cuda")
    shift = 2.0 * torch.gather(mu, 2, z[..., None].expand(B, H, T, D))
    x = {"Q": (torch.randn(B, H, T, D, generator=g, device="cuda") + shift).to(dt),
         "K": (torch.randn(B, H, T, D, generator=g, device="cuda") + shift).to(dt),
         "V": torch.randn(B, H, T, D, generator=g, device="cuda").to(dt),
         "W": synth.gaussian_orthogonal(c["m"], D, seed).to(dt).cuda()}
    x["seq_len"] = synth.padding_lengths(B, T, c["pad"], seed).cuda() if c["pad"] > 0 else None
    x["s_mix"] = torch.rand(B, H, T, generator=g, device="cuda")
    x["s_prob"] = torch.rand(B, H, T, generator=g, device="cuda")
    return x


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    p = sea.SeaParams(B=c["B"], H=c["H"], T=c["T"], d=D, m=c["m"], K=c["K"], k_hat=c["k_hat"], k_budget=c["k_budget"],
                      causal=c["causal"], scale=D ** -0.5, dtype=c["dtype"], seq_len=x["seq_len"],
                      grouping=c["grouping"], geometry=c["geometry"])
    s = dict(kind=c["kind"], p=p, x=x)
    n = (c["B"], c["H"], c["T"])
    if c["kind"] == "forward":
        s["O"] = torch.empty(*n, D, dtype=p.torch_dtype, device="cuda")
        s["ws"] = sea.alloc_workspace(p)
    elif c["kind"] == "decoder":
        s["weights"] = {k: v.cuda() for k, v in synth.decoder_weights(c["H"], D, c["K"], seed=seed).items()}
        s["A_hat"] = torch.empty(*n, c["K"], device="cuda")
        s["s_mix"], s["s_prob"] = torch.empty(*n, device="cuda"), torch.empty(*n, device="cuda")
        s["ws"] = torch.empty(sea.sea_decoder_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    else:
        s.update(sea.alloc_outputs(p))
        s["L"] = sea.sea_row_stride(p)
        s["ws"] = sea.alloc_workspace(p)
        s["crow"] = torch.zeros(c["B"] * c["T"] + 1, dtype=torch.int64, device="cuda")
        s["col"] = torch.zeros(c["B"] * c["H"] * c["T"] * s["L"], dtype=torch.int32, device="cuda")
        s["flat_ws"] = torch.empty(max(sea.sea_flatcsr_workspace_bytes(p), 256), dtype=torch.uint8, device="cuda")
        s["mix_ws"] = torch.empty(max(sea.sea_output_mix_workspace_bytes(p), 256), dtype=torch.uint8, device="cuda")
        s["C"] = torch.empty(*n, D, dtype=p.torch_dtype, device="cuda")
    return s


def run(state):
    s = state
    p, x = s["p"], s["x"]
    if s["kind"] == "forward":
        sea.sea_forward(p, x["Q"], x["K"], x["V"], x["W"], s["O"], workspace=s["ws"])
        return s["O"]
    if s["kind"] == "decoder":
        sea.sea_decoder_estimate(p, s["weights"], x["Q"], x["K"], x["V"], x["W"], s["A_hat"], s["ws"], s_mix=s["s_mix"],
                                 s_prob=s["s_prob"])
        return {"A_hat": s["A_hat"], "s_mix": s["s_mix"], "s_prob": s["s_prob"]}
    sea.sea_estimate(p, x["Q"], x["K"], x["W"], s["A_hat"], s["ws"])
    sea.sea_topk_mask(p, s["A_hat"], s["sel"], s["idx"], s["cnt"])
    sea.sea_flatcsr(p, s["idx"], s["cnt"], s["L"], s["crow"], s["col"], s["flat_ws"])
    sea.sea_flatcsr_attn(p, x["Q"], x["K"], x["V"], s["crow"], s["col"], s["C"])
    sea.sea_output_mix(p, s["C"], x["V"], x["s_mix"], s["O"], s["mix_ws"], s_prob=x["s_prob"],
                       A_hat=None if p.causal else s["A_hat"])
    return {"O": s["O"], "A_hat": s["A_hat"], "sel": s["sel"], "crow": s["crow"], "col": s["col"]}


def _pairs(c):
    """(query, key) pairs the attention of one head attends, and (row, column) cells it estimates; padding
    and the cut of a causal row's own column left out of account."""
    T, K = c["T"], c["K"]
    t = np.arange(T, dtype=np.float64)
    cols = np.full(T, float(K))
    if c["causal"]:
        cols = np.minimum(t + 1, K) if c["geometry"] else np.floor(t * K / T) + 1
    per_column = _row_len(T, K, 1, c["k_budget"] // c["k_hat"])
    keys = np.minimum(np.minimum(cols, c["k_hat"]) * per_column, t + 1 if c["causal"] else T)
    return float(keys.sum()), float(cols.sum())


def work(case):
    c = case
    N, T, m, K, e = c["B"] * c["H"], c["T"], c["m"], c["K"], 2 if c["dtype"] == "bf16" else 4
    rows = N * T
    pairs, cells = _pairs(c)
    estimate = 4.0 * rows * D * m + 2.0 * N * m * cells
    if c["geometry"] == 1:  # no columns shared by the rows: one product per admissible (query, key) pair
        estimate = 4.0 * rows * D * m + 2.0 * N * m * T * (T + 1) / 2
    attention = 4.0 * D * N * pairs
    qkv = 3.0 * rows * D * e + m * D * e
    if c["kind"] == "forward":
        return {"bytes": qkv + rows * D * e, "flops": estimate + attention}
    if c["kind"] == "decoder":
        C, Wd = 4 * c["H"], K // 2
        img = c["B"] * (T if c["causal"] else -(-T // 2)) * 1.0  # rows of the convolutions' images
        flops = 4.0 * rows * D * m + 4.0 * rows * m * (2 * D + 1)              # features, linear attention
        flops += 2.0 * rows * (3 * D * 2 * D + 4 * D * D + 2 * D * 4 * Wd)     # mu, nu
        flops += 2.0 * 9 * C * (2 * img * Wd * C + c["B"] * T * K * c["H"])    # three convolutions
        weights = 2.0 * (2 * D * 3 * D + 4 * D * D + 4 * Wd * 2 * D + 9 * C * (2 * C + c["H"]))
        return {"bytes": qkv + weights + rows * (K + 2) * 4.0, "flops": flops}
    # the lists and the tensor are results; the mixing reads V and the scalers again only if they left the chip
    lists = rows * (c["k_hat"] + _row_len(T, K, c["k_hat"], c["k_budget"])) * 4.0 + N * pairs * 4.0
    return {"bytes": qkv + rows * D * e + rows * (K * 4.0 + 12) + lists, "flops": estimate + attention}


def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    # bf16 tensors.  Scores that differ by less than their rounding may change places in the selection,
    # which exchanges one of a row's columns for another: few rows, large differences in them.  Lists
    # and the tensor built from them follow the selection.
    return {"rel": 1e-2, "max": 0.95, "differ": 1e-3}
