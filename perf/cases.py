"""The work whose speed this library is judged by: its attention calls over the range they are used in.

Every case is one pass through the public entry points on tensors that are already on the GPU: a
forward (`forward`), or a forward with row statistics and table followed by the backward (`train`).
Inputs follow the value structures of the repository's own configurations (near-copies among the
channels, per-channel scales, low rank), made on the GPU from the seed.
"""
import math

import torch

import paper_2507_17245_amd as da


def _case(name, kind, form, dtype, B, H, Hkv, N, Nk, d, causal, Br, Bc, n_groups, n_planes, values):
    return {"name": name, "kind": kind, "form": form, "dtype": dtype, "B": B, "H": H, "Hkv": Hkv, "N": N, "Nk": Nk,
            "d": d, "causal": causal, "Br": Br, "Bc": Bc, "n_groups": n_groups, "n_planes": n_planes, "lsh_seed": 0,
            "values": values}


def listed():
    return [
        # One small float problem: a check of a model's block in float32, all latency.
        _case("tiny_f32", "forward", "distr", "f32", 1, 1, 1, 256, 256, 64, False, 64, 64, 32, 4, "pairs"),
        # Training step of a layer kept in float32 (reference-precision runs).
        _case("f32_train", "train", "distr", "f32", 1, 8, 8, 2048, 2048, 64, False, 128, 64, 32, 16, "pairs"),
        # The mirrored form (samples K, fuses Q) on the same layer.
        _case("f32_mirrored", "forward", "mirrored", "f32", 1, 8, 8, 2048, 2048, 64, False, 128, 64, 32, 16, "pairs"),
        # One attention layer of a ViT-B/16 over a batch of images: 197 tokens, ragged tiles everywhere.
        _case("vit_forward", "forward", "distr", "bf16", 64, 12, 12, 197, 197, 64, False, 64, 64, 32, 16, "copies"),
        # Fine-tuning step of the same layer.
        _case("vit_train", "train", "distr", "bf16", 64, 12, 12, 197, 197, 64, False, 64, 64, 32, 16, "copies"),
        # Prefill of a Llama-1B-shaped layer: causal, grouped heads, d = 64.
        _case("llama_prefill", "forward", "distr", "bf16", 1, 32, 8, 4096, 4096, 64, True, 128, 64, 32, 16, "scales"),
        # The exact kernel on the same prompt: what a user without the approximation runs.
        _case("llama_exact", "forward", "exact", "bf16", 1, 32, 8, 4096, 4096, 64, True, 128, 64, 64, 16, "scales"),
        # Fine-tuning step of that layer.
        _case("llama_train", "train", "distr", "bf16", 1, 32, 8, 4096, 4096, 64, True, 128, 64, 32, 16, "scales"),
        # Decoding: one new token against 16384 cached keys, grouped heads.
        _case("decode", "forward", "distr", "bf16", 1, 32, 8, 1, 16384, 64, True, 64, 64, 32, 16, "scales"),
        # Chunked prefill: a ragged chunk of 200 tokens against a cache of 32768 keys.
        _case("chunk", "forward", "distr", "bf16", 1, 16, 16, 200, 32768, 128, True, 128, 64, 64, 16, "lowrank"),
        # Training step on a batch of medium-length sequences, d = 128: the most arithmetic.
        _case("mid_train", "train", "distr", "bf16", 4, 16, 16, 8192, 8192, 128, False, 128, 64, 64, 16, "rho"),
        # One long causal sequence.
        _case("long_forward", "forward", "distr", "bf16", 1, 16, 16, 32768, 32768, 128, True, 128, 64, 64, 16, "lowrank"),
    ]


def _spread(rng, lo, hi):
    """An integer of [lo, hi], even over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_once(rng):
    family = rng.choice(("f32", "vit", "prefill", "prefill", "decode", "chunk"))
    form = "distr" if rng.random() < 0.75 else "exact"
    values = rng.choice(("pairs", "copies", "scales", "rho", "lowrank"))
    d = rng.choice((64, 128))
    kind, dtype, causal, B, Bc, n_planes = "forward", "bf16", True, 1, 64, 16
    if family == "f32":
        dtype, causal = "f32", rng.random() < 0.5
        kind = rng.choice(("forward", "train"))
        if kind == "forward" and rng.random() < 0.4:
            form, Bc = "mirrored", rng.choice((32, 64, 128))
        H = rng.choice((1, 2, 4, 8))
        Hkv = max(1, H // rng.choice((1, 1, 4)))
        N = Nk = _spread(rng, 64, 2048)
        Br, n_planes = rng.choice((64, 128)), rng.choice((4, 16))
    elif family == "vit":
        kind, causal, d = rng.choice(("forward", "train")), False, 64
        B, H = _spread(rng, 1, 64), 12
        Hkv, N, Br = H, _spread(rng, 50, 577), 64
        Nk = N
    elif family == "prefill":
        kind, causal = rng.choice(("forward", "forward", "train")), rng.random() < 0.7
        B, H = rng.choice((1, 1, 2, 4)), rng.choice((8, 16, 32))
        Hkv = H // rng.choice((1, 4))
        N = Nk = _spread(rng, 512, 32768)
        Br = rng.choice((128, 128, 128, 256))
    elif family == "decode":
        B, H = _spread(rng, 1, 16), rng.choice((16, 32))
        Hkv, N, Nk, Br = H // rng.choice((1, 4, 8)), _spread(rng, 1, 8), _spread(rng, 512, 32768), 64
    else:
        B, H = rng.choice((1, 1, 2)), rng.choice((16, 32))
        Hkv, N, Nk, Br = H // rng.choice((1, 4)), _spread(rng, 16, 1024), _spread(rng, 2048, 32768), rng.choice((64, 128))
    n_groups = d if form == "exact" else d // rng.choice((2, 2, 4))
    case = _case("", kind, form, dtype, B, H, Hkv, N, Nk, d, causal, Br, Bc, n_groups, n_planes, values)
    del case["name"]
    case["lsh_seed"] = rng.randrange(1 << 31)
    return case


def draw(rng):
    """Another case of the same families: float checks and training, image batches, prefill and
    training on prompts, decoding and chunked prefill against a cache."""
    most = {"f32": work(listed()[1])["flops"], "bf16": work(listed()[10])["flops"]}
    most_bytes = max(work(c)["bytes"] for c in listed())
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["flops"] <= most[case["dtype"]] and w["bytes"] <= most_bytes:
            return case


def _values(case, gen):
    """q, k, v as float32 tensors with the channel structure case["values"] names."""
    dev = torch.device("cuda")
    B, H, Hkv, N, Nk, d = (case[x] for x in ("B", "H", "Hkv", "N", "Nk", "d"))
    qs, ks = (B, H, N, d), (B, Hkv, Nk, d)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev)

    pi = torch.randperm(d, generator=gen, device=dev)   # partner channels are no neighbours
    v = normal(*ks)
    if case["values"] == "pairs":        # two noisy copies of each of d/2 latent columns
        def pairs(shape):
            z = normal(*shape[:-1], d // 2)
            x = torch.empty(shape, device=dev)
            x[..., pi[0::2]] = z + 0.1 * normal(*z.shape)
            x[..., pi[1::2]] = z + 0.1 * normal(*z.shape)
            return x
        return pairs(qs), pairs(ks), v
    if case["values"] == "copies":       # a quarter of the channels are noisy copies of others
        def copies(x):
            n = d // 4
            x[..., pi[:n]] = x[..., pi[n:2 * n]] + 0.1 * normal(*x.shape[:-1], n)
            return x
        return copies(normal(*qs)), copies(normal(*ks)), copies(v)
    if case["values"] == "scales":       # log-normal scale per head and channel
        q = normal(*qs) * (1.0 + torch.exp(0.5 * normal(1, H, 1, d)))
        k = normal(*ks) * (1.0 + torch.exp(0.5 * normal(1, Hkv, 1, d)))
        return q, k, v
    if case["values"] == "rho":          # channel pairs with correlation 0.9
        def rho(x):
            x[..., pi[1::2]] = 0.9 * x[..., pi[0::2]] + math.sqrt(1.0 - 0.81) * x[..., pi[1::2]]
            return x
        return rho(normal(*qs)), rho(normal(*ks)), v
    # lowrank: q and k of a kv head share a rank-32 component, plus noise
    w = normal(1, Hkv, 32, d) / math.sqrt(32.0)
    q = torch.matmul(normal(B, H, N, 32), w.repeat_interleave(H // Hkv, dim=1)) + 0.3 * normal(*qs)
    k = torch.matmul(normal(B, Hkv, Nk, 32), w) + 0.3 * normal(*ks)
    return q, k, v


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    q, k, v = (x.to(dtype).contiguous() for x in _values(case, gen))
    s = {"case": case, "q": q, "k": k, "v": v, "o": torch.empty_like(q)}
    options = dict(Br=case["Br"], Bc=case["Bc"], n_groups=case["n_groups"], causal=case["causal"],
                   lsh_seed=case["lsh_seed"], n_planes=case["n_planes"], side=1 if case["form"] == "mirrored" else 0)
    if case["kind"] == "train":
        s["dout"] = torch.randn(q.shape, generator=gen, device=q.device).to(dtype)
        s["dq"], s["dk"], s["dv"] = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
        s["lse"] = torch.empty(q.shape[:3], dtype=torch.float32, device=q.device)
        if case["form"] == "distr":      # the forward leaves its grouping for the backward
            table = torch.empty((case["B"], case["H"], -(-case["N"] // case["Br"]), case["d"]), dtype=torch.uint8,
                                device=q.device)
            s["table"] = table
            s["fwd"] = da.make_params(q, k, v, lse_out=s["lse"], perm_out=table, **options)
            s["bwd"] = da.make_params(q, k, v, perm_in=table, **options)
        else:
            s["fwd"] = da.make_params(q, k, v, lse_out=s["lse"], **options)
            s["bwd"] = da.make_params(q, k, v, **options)
    else:
        s["fwd"] = da.make_params(q, k, v, **options)
    return s


def run(s):
    q, k, v, o = s["q"], s["k"], s["v"], s["o"]
    exact = s["case"]["form"] == "exact"
    (da.distr_attn_exact_fwd_ex if exact else da.distr_attn_fwd_ex)(q, k, v, o, s["fwd"])
    if s["case"]["kind"] == "forward":
        return o
    (da.distr_attn_exact_bwd_ex if exact else da.distr_attn_bwd_ex)(q, k, v, o, s["dout"], s["lse"], s["dq"], s["dk"],
                                                                  s["dv"], s["bwd"])
    return [o, s["lse"], s["dq"], s["dk"], s["dv"]]


def work(case):
    """Products of the method over the visible (query, key) pairs, n_groups wide where it reduces them,
    and the projections of the grouping; every input read and every output written once."""
    B, H, Hkv, N, Nk, d, k = (case[x] for x in ("B", "H", "Hkv", "N", "Nk", "d", "n_groups"))
    size = 4 if case["dtype"] == "f32" else 2
    pairs = B * H * (N * (Nk - N) + N * (N + 1) // 2 if case["causal"] else N * Nk)
    q_bytes, kv_bytes = B * H * N * d * size, B * Hkv * Nk * d * size
    bytes_, flops = 2 * q_bytes + 2 * kv_bytes, 2 * pairs * (k + d)
    if case["form"] != "exact":
        rows = B * Hkv * Nk if case["form"] == "mirrored" else B * H * N
        flops += 2 * rows * d * case["n_planes"]
    if case["kind"] == "train":
        flops += 2 * pairs * (3 * k + 2 * d)             # scores, dQ, dK over the groups; dP, dV over the channels
        bytes_ += 4 * q_bytes + 4 * kv_bytes + 2 * 4 * B * H * N   # q, o, dout, k, v, lse in; lse, dq, dk, dv out
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """About four times the largest distance from the same path in 64 bits over these ranges: float 1e-6 (max
    1.2e-5), bf16 forward 2.4e-3 (max 4.4e-2), bf16 backward 4.9e-3 (max 0.15, llama_train's dq)."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5}
    return {"rel": 2e-2, "max": 0.6} if case["kind"] == "train" else {"rel": 1e-2, "max": 0.18}
