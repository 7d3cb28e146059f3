"""Timing cases of the decode path: one attention call of a serving step, over the shapes it is used with.

Every case is one decode step's attention for a batch of sequences through the public binding: grouped-query
attention (``xattn_decode``), the same behind an append of the step's K/V rows (``xattn_write_kvcache``), or
latent-KV attention (``xattn_mla_decode``).  K/V caches and queries are N(0, 1) in bf16, as the repository's
workloads draw them (latent-KV queries scaled so that the scores have unit variance).
"""
import math
import random

import torch

import paper_2510_14686_amd as xa

HEAD_DIM = 128
D_LATENT, D_ROPE = 512, 64
D_QK = D_LATENT + D_ROPE
MAX_SEQ_LEN = 65536                      # tokens of virtual address space an xTensor range reserves


def _gqa(name, batch, q_len, n_q_heads, n_kv_heads, lens, lo, hi, **more):
    return dict(name=name, op="gqa", batch=batch, q_len=q_len, n_q_heads=n_q_heads, n_kv_heads=n_kv_heads, lens=lens,
                lo=lo, hi=hi, xtensor=False, append=False, **more)


def _mla(name, batch, q_len, n_heads, lo, hi):
    return dict(name=name, op="mla", batch=batch, q_len=q_len, n_heads=n_heads, lens="uniform", lo=lo, hi=hi)


def listed():
    skewed = _gqa("gqa_skewed_lengths", 256, 1, 40, 8, "lognormal", 16, 65536)
    skewed.update(xtensor=True)
    chat = _gqa("gqa_decode_8kv", 64, 1, 32, 8, "uniform", 512, 4096)
    chat.update(xtensor=True)
    append = _gqa("gqa_short_append", 256, 1, 16, 8, "uniform", 16, 512)
    append.update(append=True)
    return [
        # the smallest call of the benchmark (workload "tiny"): latency and launches
        _gqa("gqa_tiny", 4, 1, 8, 2, "uniform", 17, 256),
        # plain decode of an 8B-shaped model, conversations of a few thousand tokens, on xTensor ranges
        chat,
        # long documents, groups of eight query heads: every sequence split over many compute units
        _gqa("gqa_long_context", 16, 1, 64, 8, "uniform", 16384, 32768),
        # verification of three draft tokens: 16 query rows per KV head, a causal mask inside the block
        _gqa("gqa_verify_4_tokens", 128, 4, 32, 8, "uniform", 1024, 8192),
        # a batch of very unequal lengths on xTensor ranges
        skewed,
        # one user's long prompt, nothing else on the GPU
        _gqa("gqa_one_request", 1, 1, 32, 8, "uniform", 30001, 30001),
        # the 8B shape split over four GPUs by KV head: two KV heads are left on this one
        _gqa("gqa_decode_2kv", 64, 1, 8, 2, "uniform", 512, 4096),
        # verification with groups of eight: 32 query rows per KV head
        _gqa("gqa_verify_32_rows", 32, 4, 64, 8, "uniform", 1024, 8192),
        # many short chats of a small model (two query heads per KV head): append the step's rows, then attend
        append,
        # latent-KV decode, all 128 heads on one GPU (data-parallel attention)
        _mla("mla_decode", 64, 1, 128, 1024, 8192),
        # latent-KV verification of one speculated token
        _mla("mla_verify", 64, 2, 128, 1024, 8192),
        # latent-KV decode with the heads split over eight GPUs: 16 are left on this one
        _mla("mla_decode_16_heads", 64, 1, 16, 1024, 8192),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [(8, 2), (4, 4), (5, 1), (7, 1), (16, 2), (12, 2), (6, 2), (32, 16), (32, 8), (64, 8), (40, 8), (16, 8), (16, 4), (8, 1)]
_MAX_TOKENS, _MAX_BYTES, _MAX_FLOPS = 500000, 1.5e9, 1.2e11


def draw(rng):
    """One more case: head counts of the workloads and tests, 1 to 8 new tokens, 1 to 512 sequences of 16 to 32768 tokens."""
    while True:
        hi = _log_uniform(rng, 32, 32768)
        lo = max(1, hi // rng.choice([2, 4, 8, 16]))
        batch = _log_uniform(rng, 1, 512)
        if rng.random() < 0.6:
            hq, hkv = rng.choice(_HEADS)
            q_len = 1 if rng.random() < 0.6 else rng.randint(2, min(8, 64 // (hq // hkv)))
            case = dict(op="gqa", batch=batch, q_len=q_len, n_q_heads=hq, n_kv_heads=hkv, lo=lo, hi=hi,
                        lens=rng.choice(["uniform", "uniform", "lognormal"]), xtensor=rng.random() < 0.25 and batch <= 64,
                        append=rng.random() < 0.25)
            case["append"] = case["append"] and not case["xtensor"]
        else:
            q_len = rng.choice([1, 1, 2, 3])
            case = dict(op="mla", batch=min(batch, 128), q_len=q_len, n_heads=rng.choice([8, 16, 24, 32, 64, 72, 128]), lens="uniform",
                        lo=lo, hi=hi)
        w = work(case)
        if sum(_lengths(case)) <= _MAX_TOKENS and w["bytes"] <= _MAX_BYTES and w["flops"] <= _MAX_FLOPS:
            return case


def _lengths(case, seed=None):
    """KV lengths of the case, the new tokens included; the seed only decides which sequence has which."""
    rng = random.Random("%d %d %d %s" % (case["batch"], case["lo"], case["hi"], case["lens"]))
    if case["lens"] == "lognormal":      # sigma 1.2 around the middle of the range, 1024 at most
        median = min(1024.0, math.sqrt(case["lo"] * case["hi"]))
        lens = [int(round(min(case["hi"], max(case["lo"], median * math.exp(rng.gauss(0.0, 1.2)))))) for _ in range(case["batch"])]
    else:
        lens = [rng.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]
    lens = [n + case["q_len"] - 1 for n in lens]
    if seed is not None:
        random.Random(seed).shuffle(lens)
    return lens


def _normal(seed, stream, shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 8 + stream)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _values(case, seed):
    """Lengths, queries, cached rows of all sequences back to back, and the rows to append (or None)."""
    lens = _lengths(case, seed)
    n = sum(lens)
    if case["op"] == "mla":
        q = _normal(seed, 0, (case["batch"], case["q_len"], case["n_heads"], D_QK)) * math.sqrt(192.0 / D_QK)
        return lens, q, [_normal(seed, 1, (n, D_QK))], None
    hkv = case["n_kv_heads"]
    q = _normal(seed, 0, (case["batch"], case["q_len"], case["n_q_heads"], HEAD_DIM))
    kv = [_normal(seed, s, (n, hkv, HEAD_DIM)) for s in (1, 2)]
    new = [_normal(seed, s, (case["batch"], case["q_len"], hkv, HEAD_DIM)) for s in (3, 4)] if case["append"] else None
    return lens, q, kv, new


class _Ranges:
    """xTensor ranges of a batch's K and V, filled from contiguous tensors; unmapped with the object."""

    def __init__(self, lens, kv, seed):
        self.handles = []
        row = kv[0][0].numel() * 2
        hkv = kv[0].shape[1]
        self.addr = [[], []]
        for b, n in enumerate(lens):
            for which in (0, 1):
                base, handle = xa.xtensor_map(max(MAX_SEQ_LEN, n) * row, n * row, seed * 1000003 + 2 * b + which, 0)
                self.handles.append(handle)
                self.addr[which].append(base)
        self.ptrs = [torch.tensor(a, dtype=torch.int64, device="cuda") for a in self.addr]
        ends = torch.tensor(lens, dtype=torch.int32, device="cuda")
        at = 0
        for b, n in enumerate(lens):
            xa.xattn_write_kvcache(kv[0][at:at + n], kv[1][at:at + n], self.ptrs[0][b:b + 1], self.ptrs[1][b:b + 1],
                                   ends[b:b + 1], 1, n, hkv, HEAD_DIM)
            at += n
        torch.cuda.synchronize()

    def __del__(self):
        torch.cuda.synchronize()
        for handle in self.handles:
            xa.xtensor_unmap(handle)


def _addresses(flat, lens):
    row, at, out = flat[0].numel() * flat.element_size(), flat.data_ptr(), []
    for n in lens:
        out.append(at)
        at += n * row
    return torch.tensor(out, dtype=torch.int64, device="cuda")


def _scale(case):
    """The caller's fp32 softmax scale."""
    return float(torch.tensor(1.0 / math.sqrt(192.0 if case["op"] == "mla" else HEAD_DIM), dtype=torch.float32))


def prepare(case, seed):
    lens, q, kv, new = _values(case, seed)
    rows = q.shape[:3]
    s = dict(case=case, q=q, new=new, kv=kv, scale=_scale(case), stream=torch.cuda.current_stream(),
             lens=torch.tensor(lens, dtype=torch.int32, device="cuda"),
             out=torch.empty(rows + (D_LATENT if case["op"] == "mla" else HEAD_DIM,), dtype=torch.bfloat16, device="cuda"),
             lse=torch.empty(rows, dtype=torch.float32, device="cuda"))
    if case["op"] == "gqa" and case["xtensor"]:
        s["ranges"] = _Ranges(lens, kv, seed)
        s["ptrs"] = s["ranges"].ptrs
        s["kv"] = None
    else:
        s["ptrs"] = [_addresses(flat, lens) for flat in kv]
    return s


def run(s):
    c = s["case"]
    if c["op"] == "mla":
        xa.xattn_mla_decode(s["q"], s["ptrs"][0], s["lens"], c["batch"], c["q_len"], c["n_heads"], D_LATENT, D_ROPE, s["scale"],
                            s["out"], s["lse"], s["stream"])
        return s["out"], s["lse"]
    if c["append"]:
        xa.xattn_write_kvcache(s["new"][0], s["new"][1], s["ptrs"][0], s["ptrs"][1], s["lens"], c["batch"], c["q_len"],
                               c["n_kv_heads"], HEAD_DIM, s["stream"])
    xa.xattn_decode(s["q"], s["ptrs"][0], s["ptrs"][1], s["lens"], c["batch"], c["q_len"], c["n_q_heads"], c["n_kv_heads"],
                    HEAD_DIM, s["scale"], s["out"], s["lse"], s["stream"])
    return (s["out"], s["lse"], s["kv"][0], s["kv"][1]) if c["append"] else (s["out"], s["lse"])


def work(case):
    """Cached rows, queries and appended rows read once, results and appended rows written once; the two products."""
    lens, t = _lengths(case), case["q_len"]
    # key t of the last q_len is seen by the tokens from it on
    pairs = sum(n * t - t * (t - 1) // 2 for n in lens)
    if case["op"] == "mla":
        rows = case["batch"] * t * case["n_heads"]
        return {"bytes": sum(lens) * D_QK * 2 + rows * ((D_QK + D_LATENT) * 2 + 4) + case["batch"] * 12,
                "flops": pairs * case["n_heads"] * 2 * (D_QK + D_LATENT)}
    rows = case["batch"] * t * case["n_q_heads"]
    n_bytes = sum(lens) * case["n_kv_heads"] * HEAD_DIM * 4 + rows * (HEAD_DIM * 4 + 4) + case["batch"] * 20
    if case["append"]:                   # the new rows come from the step, and go to the cache
        n_bytes += case["batch"] * t * case["n_kv_heads"] * HEAD_DIM * 4
    return {"bytes": n_bytes, "flops": pairs * case["n_q_heads"] * 4 * HEAD_DIM}


def tolerance(case):
    """bf16 results of fp32 sums over bf16 inputs: about four times what the path differs from ``exact`` by
    (rel 1.7e-3 and, for one element, 4e-3, which is bf16 rounding; latent-KV 1.9e-3)."""
    return {"rel": 7e-3, "max": 3e-2}


def exact(case, seed):
    lens, q, kv, new = _values(case, seed)
    t, scale = case["q_len"], _scale(case)
    q = q.double()
    out = torch.empty(q.shape[:3] + (D_LATENT if case["op"] == "mla" else HEAD_DIM,), dtype=torch.float64, device="cuda")
    lse = torch.empty(q.shape[:3], dtype=torch.float64, device="cuda")
    at = 0
    for b, n in enumerate(lens):
        if new is not None:
            for flat, rows in zip(kv, new):
                flat[at + n - t:at + n] = rows[b]
        if case["op"] == "mla":
            k = kv[0][at:at + n].double().unsqueeze(0)                               # [1, n, 576]
            v = k[:, :, :D_LATENT].contiguous()
        else:
            k, v = (flat[at:at + n].double().transpose(0, 1).contiguous() for flat in kv)      # [kv heads, n, 128]
        g = k.shape[0]
        qb = q[b].reshape(t, g, -1, q.shape[-1]).transpose(0, 1).reshape(g, -1, q.shape[-1])   # rows (token, head of group)
        s = torch.matmul(qb, k.transpose(1, 2).contiguous()) * scale
        token = torch.arange(qb.shape[1], device="cuda") // (qb.shape[1] // t)
        s.masked_fill_(torch.arange(n, device="cuda")[None, :] > (n - t + token)[:, None], -math.inf)
        z = torch.logsumexp(s, dim=-1)
        o = torch.matmul(torch.exp(s - z.unsqueeze(-1)), v)
        out[b] = o.reshape(g, t, -1, o.shape[-1]).transpose(0, 1).reshape(t, -1, o.shape[-1])
        lse[b] = z.reshape(g, t, -1).transpose(0, 1).reshape(t, -1)
        at += n
    return (out, lse, kv[0], kv[1]) if new is not None else (out, lse)
