"""Performance cases of the AnTKV online path: what a serving or calibration program asks of this package.

Three parts of such a program are covered, one attention layer at a time: a decode step (append the new token behind the
FP16 window, then attend over codes and FP16 anchors), the prompt (attention, Anchor Score selection, encoding, anchor
rows), and one iteration of the offline k-means that learns the codebooks.

    listed()  the fixed cases            prepare(case, seed)  inputs and buffers on the GPU
    draw(rng) one more of their ranges   run(state)           one pass through the public entry points
    work(case), tolerance(case)          what a pass cannot do without, and how closely two results agree
"""
from __future__ import annotations

import math

import torch

import paper_2506_19505_amd as antkv

D = 128                       # head dim
WINDOW = 32                   # FP16 sliding window of recent tokens
STEPS = 256                   # decode steps before a sequence ends and the next one takes its place
ROPE_BASE, ROPE_STYLE = 500000.0, 1


def _case(name, op, B, Hq, Hkv, N, d_sub, C=256, **more):
    return dict(name=name, op=op, B=B, Hq=Hq, Hkv=Hkv, N=N, d_sub=d_sub, C=C, **more)


def listed():
    return [
        # -- decode steps (append_token + decode attention), anchors 1 % of the context plus the window
        # a short chat: launches and latency are all there is
        _case("decode_4k_d8", "decode", 1, 32, 8, 4096, 8),
        # one user with a long document, the most accurate code format
        _case("decode_32k_d4", "decode", 1, 32, 8, 32768, 4),
        # a batch of long contexts at 1 bit per element: the benchmark's headline shape
        _case("decode_128k_b4_d8", "decode", 4, 32, 8, 131072, 8),
        # the longest context, with Anchor Scores of the step and re-selection of the anchor sets
        _case("decode_840k_d16_reselect", "decode", 1, 32, 8, 840000, 16, reselect=True),
        # the same context in the 0.375-bit format (4096 centroids)
        _case("decode_840k_d32m4096", "decode", 1, 32, 8, 840000, 32, C=4096),
        # keys cached before RoPE, an uneven batch size and context length
        _case("decode_prerope_57k_b3_d8", "prerope", 3, 32, 8, 57003, 8),
        # -- prompts: attention with row statistics, selection from them, K and V encoded, anchor rows gathered
        # short requests of uneven length, one KV head per query head
        _case("prompt_1531_b2_mha_d8", "prompt", 2, 32, 32, 1531, 8),
        # a long prompt in one go
        _case("prompt_32k_d8", "prompt", 1, 32, 8, 32768, 8),
        # a very long prompt whose attention ran elsewhere: anchors chosen from the last 32 queries, the whole cache encoded
        _case("ingest_128k_d16", "ingest", 1, 32, 8, 131072, 16),
        # one chunk of a chunked prefill encoded behind an existing cache: K and V rows straight out of the projection
        _case("encode_32k_d8", "encode", 1, 32, 8, 32768, 8),
        _case("encode_9001_d16m4096", "encode", 1, 32, 8, 9001, 16, C=4096),
        # -- codebook learning: one weighted k-means iteration over a calibration set
        _case("kmeans_32k_d8", "kmeans", 1, 32, 8, 32768, 8),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["decode"] * 5 + ["prerope", "prompt", "prompt", "ingest", "encode", "encode", "kmeans"])
    Hq, Hkv = rng.choice([(32, 8)] * 4 + [(32, 32), (16, 8)])
    B = rng.choice([1, 1, 2, 3, 4])
    d_sub, C = rng.choice([(4, 256), (8, 256), (8, 256), (16, 256), (32, 4096), (16, 4096)])
    if op in ("decode", "prerope"):
        most = min(840000, 6_700_000 // (B * Hkv))              # cached rows of all heads: as the longest listed context
        N = _log_uniform(rng, 1000, most)
    elif op == "prompt":
        most = min(32768, int(32768 * math.sqrt(32 / (B * Hq))))  # query-key pairs: as the longest listed prompt
        N = _log_uniform(rng, 500, most)
    elif op == "ingest":
        N = _log_uniform(rng, 4000, 131072 * 8 // (B * Hkv))
    else:
        N = _log_uniform(rng, 500, 32768 * 8 // (B * Hkv))
    case = dict(op=op, B=B, Hq=Hq, Hkv=Hkv, N=N, d_sub=d_sub, C=C)
    if op == "decode" and rng.random() < 0.25:
        case["reselect"] = True
    return case


# ------------------------------------------------------------------------------------------------ inputs

def _anchors(N):
    return max(1, math.ceil(0.01 * N))                          # 1 % of the context


def _normal(gen, shape, scale=None):
    x = torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    return x if scale is None else x.mul_(scale)


def _outliers(gen, Hkv):
    """Per-channel factors of the keys [Hkv, 1, D]: four channels of each KV head are ten times larger."""
    order = torch.rand((Hkv, D), device="cuda", generator=gen).argsort(dim=1)
    factors = torch.ones((Hkv, D), dtype=torch.float16, device="cuda")
    return factors.scatter_(1, order[:, :4], 10.0).view(Hkv, 1, D)


def _codebook(gen, case, scale):
    """fp16 [Hkv, M, C, d_sub]: sub-vectors of rows of the cache's distribution."""
    Hkv, d, C = case["Hkv"], case["d_sub"], case["C"]
    rows = _normal(gen, (Hkv, C, D), scale)
    return rows.view(Hkv, C, D // d, d).transpose(1, 2).contiguous()


def _anchor_sets(gen, B, Hkv, N, k):
    """int32 [B, Hkv, k] ascending positions below N: a quarter at the head, a quarter at the tail, the rest anywhere between."""
    head = tail = k // 4
    rest = k - head - tail
    middle = torch.rand((B, Hkv, N - head - tail), device="cuda", generator=gen)
    idx = middle.argsort(dim=-1, stable=True)[..., :rest] + head
    ends = torch.cat([torch.arange(head, device="cuda"), torch.arange(N - tail, N, device="cuda")]).expand(B, Hkv, -1)
    return torch.cat([idx, ends], dim=-1).sort(dim=-1).values.to(torch.int32).contiguous()


def _prepare_decode(case, gen):
    B, Hq, Hkv, N = case["B"], case["Hq"], case["Hkv"], case["N"]
    geom = antkv.Geometry(B, Hq, Hkv, case["d_sub"], n_centroids=case["C"])
    cap = (N + STEPS + 63) // 64 * 64
    outl = _outliers(gen, Hkv)
    k = _anchors(N)
    s = dict(op=case["op"], geom=geom, scale=1 / math.sqrt(D), N0=N, step=0, resel=k if case.get("reselect") else 0)
    s["cb_k"], s["cb_v"] = _codebook(gen, case, outl), _codebook(gen, case, None)
    shape = (B, Hkv, cap, geom.code_bytes)
    s["codes_k"] = torch.randint(0, 256, shape, dtype=torch.uint8, device="cuda", generator=gen)
    s["codes_v"] = torch.randint(0, 256, shape, dtype=torch.uint8, device="cuda", generator=gen)
    recent = torch.arange(N - WINDOW, N, dtype=torch.int32, device="cuda").expand(B, Hkv, WINDOW)
    for which, f in (("k", outl), ("v", None)):
        s["idx_" + which] = torch.cat([_anchor_sets(gen, B, Hkv, N - WINDOW, k), recent], dim=-1).contiguous()
        s["rows_" + which] = _normal(gen, (B, Hkv, k + WINDOW, D), f)
        s["prompt_" + which] = (s["idx_" + which].clone(), s["rows_" + which].clone())
        s["new_" + which] = list(_normal(gen, (STEPS, B, Hkv, D), None if f is None else f.view(Hkv, D)))
    s["q"] = list(_normal(gen, (STEPS, B, Hq, D)))
    s["out"] = torch.empty((B, Hq, D), dtype=torch.float16, device="cuda")
    if case["op"] == "prerope":
        spaces = (antkv.decode_attn_prerope_workspace(geom, n, k + WINDOW, "cuda") for n in range(N, N + STEPS + 1))
        s["workspace"] = max(spaces, key=lambda w: w.numel())
    else:
        spaces = (antkv.DecodeWorkspace(geom, n, k + WINDOW, k + WINDOW, s["resel"], "cuda") for n in range(N, N + STEPS + 1))
        s["workspace"] = max(spaces, key=lambda w: w.nbytes)
    return s


def _prepare_rows(case, gen):
    B, Hq, Hkv, N, op = case["B"], case["Hq"], case["Hkv"], case["N"], case["op"]
    geom = antkv.Geometry(B, Hq, Hkv, case["d_sub"], n_centroids=case["C"])
    outl = _outliers(gen, Hkv)
    s = dict(op=op, geom=geom, scale=1 / math.sqrt(D), k=_anchors(N))
    s["cb_k"], s["cb_v"] = _codebook(gen, case, outl), _codebook(gen, case, None)
    if op == "encode":                                           # rows as a projection leaves them: token-major, heads inside
        k = _normal(gen, (B, N, Hkv, D), outl.view(Hkv, D))
        s["K"], s["V"] = k.transpose(1, 2), _normal(gen, (B, N, Hkv, D)).transpose(1, 2)
        s["offset"] = 1024                                       # earlier chunks of the prompt
    else:
        s["K"], s["V"] = _normal(gen, (B, Hkv, N, D), outl), _normal(gen, (B, Hkv, N, D))
        s["offset"] = 0
    if op == "kmeans":
        s["w"] = torch.rand((B, Hkv, N), dtype=torch.float32, device="cuda", generator=gen)
        return s
    if op in ("prompt", "ingest"):
        s["Q"] = _normal(gen, (B, Hq, N if op == "prompt" else WINDOW, D))
        s["rows_k"] = torch.empty((B, Hkv, s["k"], D), dtype=torch.float16, device="cuda")
        s["rows_v"] = torch.empty_like(s["rows_k"])
    cap = (s["offset"] + N + 1023) // 1024 * 1024
    s["codes_k"] = torch.zeros((B, Hkv, cap, geom.code_bytes), dtype=torch.uint8, device="cuda")
    s["codes_v"] = torch.zeros_like(s["codes_k"])
    return s


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return (_prepare_decode if case["op"] in ("decode", "prerope") else _prepare_rows)(case, gen)


# ------------------------------------------------------------------------------------------------ one pass

def _run_decode(s):
    g = s["geom"]
    if s["step"] == STEPS:                                       # the sequence is over: its prompt's successor starts
        s["step"] = 0
        for which in ("k", "v"):
            s["idx_" + which].copy_(s["prompt_" + which][0])
            s["rows_" + which].copy_(s["prompt_" + which][1])
    t = s["step"]
    s["step"] = t + 1
    n = antkv.append_token(g, s["new_k"][t], s["new_v"][t], s["N0"] + t, WINDOW, s["cb_k"], s["cb_v"], s["codes_k"], s["codes_v"],
                           s["idx_k"], s["rows_k"], s["idx_v"], s["rows_v"])
    args = (g, s["q"][t], s["scale"], s["codes_k"], s["codes_v"], s["cb_k"], s["cb_v"], s["idx_k"], s["rows_k"], s["idx_v"],
            s["rows_v"])
    if s["op"] == "prerope":
        out = antkv.decode_attn_prerope(*args, rope_base=ROPE_BASE, rope_style=ROPE_STYLE, N=n, out=s["out"], workspace=s["workspace"])
    else:
        out = antkv.decode_attn(*args, N=n, out=s["out"], k_resel=s["resel"], workspace=s["workspace"])
    return {"out": out, "cache": [s[x] for x in ("codes_k", "codes_v", "idx_k", "rows_k", "idx_v", "rows_v")]}


def run(s):
    op, g = s["op"], s["geom"]
    if op in ("decode", "prerope"):
        return _run_decode(s)
    if op == "kmeans":
        return antkv.kmeans_step(g, s["K"], s["w"], s["cb_k"])
    res = {}
    if op == "prompt":
        res["attn"] = antkv.prefill_attn(g, s["Q"], s["K"], s["V"], s["scale"])
        _, row_max, row_sum = res["attn"]
        res["selected"] = antkv.anchor_select(g, s["Q"], s["K"], s["scale"], s["k"], row_max=row_max, row_sum=row_sum)
    elif op == "ingest":
        res["selected"] = antkv.anchor_select(g, s["Q"], s["K"], s["scale"], s["k"], want_scores=False)
    res["codes_k"] = antkv.encode(g, s["K"], s["cb_k"], codes=s["codes_k"], token_offset=s["offset"])
    res["codes_v"] = antkv.encode(g, s["V"], s["cb_v"], codes=s["codes_v"], token_offset=s["offset"])
    if op != "encode":
        idx_k, idx_v = res["selected"][:2]
        res["rows_k"] = antkv.gather_rows(g, s["K"], idx_k, out=s["rows_k"])
        res["rows_v"] = antkv.gather_rows(g, s["V"], idx_v, out=s["rows_v"])
    return res


# ------------------------------------------------------------------------------------------------ work and tolerance

def work(case):
    B, Hq, Hkv, N, C, op = (case[x] for x in ("B", "Hq", "Hkv", "N", "C", "op"))
    M = D // case["d_sub"]
    code_bytes = M if C == 256 else 3 * M // 2
    k, rows = _anchors(N), B * Hkv * N
    codebook = 2 * Hkv * D * C
    if op in ("decode", "prerope"):
        k += WINDOW
        by = 2 * rows * code_bytes + 2 * B * Hkv * k * (2 * D + 4) + 2 * codebook + 4 * B * Hq * D
        by += 2 * B * Hkv * WINDOW * 2 * D                                       # the window moves one place
        fl = B * Hq * (2 * D * C + N * (M + 2 * D) + 2 * k * 2 * D)              # table, scores, values, FP16 rows
        if op == "prerope":
            fl = B * Hq * N * 4 * D + rows * 3 * D                               # every key rotated, scores, values
        if case.get("reselect"):
            by += 2 * 4 * rows + 2 * 4 * B * Hkv * (k - WINDOW)                  # scores written, sets written
            fl += B * Hq * N * 4
        return {"bytes": by, "flops": fl}
    encode = 2 * rows * D * C                                                    # one tensor against its codebook
    if op == "kmeans":
        return {"bytes": rows * (2 * D + 4 + code_bytes) + 2 * codebook, "flops": encode + 2 * rows * D}
    by = 2 * (rows * (2 * D + code_bytes) + codebook)
    fl = 2 * encode
    if op == "prompt":
        pairs = B * Hq * N * (N + 1) // 2
        by += B * Hq * N * (4 * D + 8) + 8 * rows
        fl += pairs * (4 * D + 2 * D)                                            # QK^T and PV, then the scores' own QK^T
    elif op == "ingest":
        by += B * Hq * WINDOW * 2 * D
        fl += B * Hq * WINDOW * N * 2 * D
    if op != "encode":
        by += 4 * B * Hkv * k * 2 * D + 8 * B * Hkv * k
    return {"bytes": by, "flops": fl}


def tolerance(case):
    op = case["op"]
    # Codes are the nearest centroid by fp32 distances: two orders of summation pick another one only between near-equal
    # distances, less than one in ten thousand.  In an ascending list of anchors, one near-tie at the selection threshold
    # that falls the other way moves every entry between the two positions.
    if op in ("prompt", "ingest") or case.get("reselect"):
        return {"rel": 2e-3, "differ": 1e-2}
    if op in ("decode", "prerope"):
        return {"rel": 2e-3, "differ": 1e-4}                     # fp16 weights and centroids, fixed-point scores, fp16 output
    if op == "kmeans":
        return {"rel": 1e-3, "max": 0.1, "differ": 1e-4}         # fp16 centroids; a small cluster can lose a near-tie
    return {"differ": 1e-4}
