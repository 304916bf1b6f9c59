"""Decode-time workloads of the library, for timing: what they are, their inputs, one pass, and the same pass in 64 bits.

A case names one call of the library's Python layer on one paged cache:

``step``   ``DecodeSession.decode_step`` after one token per sequence was appended (statistics of the last page, page
           scores, top-k pages, attention over them) -- what a serving loop does per layer and token.
``calls``  the same work through the separate calls, as a program that also wants the score rows makes it.
``dense``  attention over every page (layers that stay dense, and the first decode steps of short prompts).
``build``  page statistics of whole sequences (after a prefill).
``chunk``  page statistics of the last ``chunk`` tokens of every sequence (after one piece of a chunked prefill).

Sizes are those of the five benchmark configurations and of the paper-shape benchmark, and of the supported ranges
around them (other group sizes, head dimension 64, pages of 8 and 32 tokens, fp32 caches, odd lengths).
"""
from __future__ import annotations

import math
import random
import zlib

import torch

from paper_2605_27740_amd.session import DecodeSession
from paper_2605_27740_amd.workloads import Workload

LAMBDA = 0.5
DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}


def _case(name, op, *, dtype="bf16", stats="fp32", batch=1, q_heads=32, kv_heads=8, head_dim=128, page_size=16,
          context=32768, min_context=0, top_k=128, recent=0, keys="shift", chunk=0):
    case = dict(op=op, dtype=dtype, stats=stats, batch=batch, q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim,
                page_size=page_size, context=context, min_context=min_context or context, top_k=top_k, recent=recent,
                keys=keys, chunk=chunk)
    return dict(case, name=name) if name else case


def listed():
    return [
        # a toy model in fp32: everything is launch latency
        _case("step_tiny_fp32", "step", dtype="fp32", q_heads=8, kv_heads=2, head_dim=64, context=2048, top_k=16, keys="iid"),
        # one chat session of 32K tokens on an 8B-shaped model: the interactive case
        _case("step_one_32k", "step"),
        # one whole-book prompt of a million tokens (the length is odd, the last page partial), the paper's statistics format
        _case("step_one_1m", "step", stats="bf16", context=1_000_003, top_k=1024),
        # a full serving batch at 128K: the headline configuration
        _case("step_batch_128k", "step", batch=16, context=131072, top_k=256),
        # a serving batch of mixed lengths, pages of 32 tokens
        _case("step_ragged", "step", stats="bf16", batch=32, page_size=32, context=131072, min_context=4096, top_k=64),
        # long-form speech: smooth keys, 4 KV heads, the largest page budget
        _case("step_speech_256k", "step", batch=4, q_heads=16, kv_heads=4, context=262144, top_k=1024, keys="smooth"),
        # the paper's throughput setting: 80 sequences of 32K, pages of 8 tokens, 512 tokens attended
        _case("step_batch80_s8", "step", stats="bf16", batch=80, page_size=8, context=32768, top_k=64),
        # a 70B-shaped model (8 query heads per KV head) with the last pages always kept
        _case("step_group8", "step", batch=12, q_heads=64, context=50_001, min_context=30_000, top_k=200, recent=4),
        # multi-head attention (no groups), head dimension 64, fp32 cache, separate calls with the score rows kept
        _case("calls_fp32_mha", "calls", dtype="fp32", batch=6, q_heads=16, kv_heads=16, head_dim=64, page_size=8,
              context=20_000, min_context=1_000, top_k=96, keys="iid"),
        # the dense layers beside the sparse ones
        _case("dense_ragged", "dense", batch=8, context=60_000, min_context=2_000),
        # statistics of a whole batch after its prefill
        _case("build_batch_128k", "build", stats="bf16", batch=16, context=131072, top_k=256),
        # statistics of the 2048 tokens that a chunked prefill has just written
        _case("chunk_2k", "chunk", batch=4, context=24_000, min_context=9_000, chunk=2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """One more case of the ranges above; it moves at most half the bytes of the largest listed case."""
    most = 0.5 * max(work(c)["bytes"] for c in listed())
    while True:
        op = rng.choices(["step", "calls", "dense", "build", "chunk"], [60, 10, 12, 10, 8])[0]
        kv_heads = rng.choices([1, 2, 4, 8, 16, 32], [1, 1, 2, 5, 1, 1])[0]
        group = rng.choices([1, 2, 4, 8], [2, 2, 4, 3])[0]
        context = _log_int(rng, 500, 1_000_000)
        ragged = rng.random() < 0.5
        case = _case(None, op, dtype=rng.choices(["bf16", "fp32"], [4, 1])[0], stats=rng.choice(["bf16", "fp32"]),
                     batch=_log_int(rng, 1, 80), q_heads=kv_heads * group, kv_heads=kv_heads,
                     head_dim=rng.choices([64, 128], [1, 3])[0], page_size=rng.choice([8, 16, 32]), context=context,
                     min_context=max(1, int(context * rng.uniform(0.05, 0.9))) if ragged else context,
                     top_k=_log_int(rng, 8, 1024), recent=rng.choices([0, 4], [4, 1])[0],
                     keys=rng.choice(["iid", "shift", "smooth"]),
                     chunk=_log_int(rng, 1, 4096) if op == "chunk" else 0)
        if case["q_heads"] > 128 or work(case)["bytes"] > most:
            continue
        tokens = case["batch"] * context * kv_heads * case["head_dim"] * (2 if case["dtype"] == "bf16" else 4)
        if 2 * tokens > 9e9:  # K and V of one state
            continue
        return case


def _lengths(case):
    """Sequence lengths, log-uniform between the case's bounds; they belong to the case, not to the seed."""
    lo, hi, n = case["min_context"], case["context"], case["batch"]
    if lo == hi:
        return [hi] * n
    r = random.Random(zlib.crc32(repr((lo, hi, n)).encode()))
    lens = [min(hi, max(lo, round(math.exp(r.uniform(math.log(lo), math.log(hi)))))) for _ in range(n)]
    lens[r.randrange(n)] = hi
    return lens


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    es = 2 if case["stats"] == "bf16" else 4
    B, H, Hkv, D, S = (case[k] for k in ("batch", "q_heads", "kv_heads", "head_dim", "page_size"))
    lens = _lengths(case)
    pages = [-(-n // S) for n in lens]
    record = Hkv * (D * es + 4)
    q_out = B * H * (2 * D * e + 4)
    if case["op"] in ("step", "calls"):
        attended = sum(min(n, case["top_k"] * S) for n in lens) * Hkv
        tail = sum(n - (p - 1) * S for n, p in zip(lens, pages)) * Hkv * D * e + B * record
        b = sum(pages) * (record + 4) + tail + attended * D * 2 * e + q_out + B * Hkv * (case["top_k"] + 1) * 4
        if case["op"] == "calls":
            b += sum(pages) * Hkv * 4
        return {"bytes": b, "flops": sum(pages) * H * 2 * D + attended * (H // Hkv) * 4 * D}
    if case["op"] == "dense":
        t = sum(lens) * Hkv
        return {"bytes": t * D * 2 * e + sum(pages) * 4 + q_out, "flops": t * (H // Hkv) * 4 * D}
    if case["op"] == "build":
        touched, tokens = sum(pages), sum(lens)
    else:
        first = [max(0, n - case["chunk"]) // S for n in lens]
        touched = sum(p - f for p, f in zip(pages, first))
        tokens = sum(n - f * S for n, f in zip(lens, first))
    return {"bytes": tokens * Hkv * D * e + touched * (record + 4), "flops": tokens * Hkv * D * 4}


def tolerance(case):
    """fp32 caches: sums of fp32 numbers in another order. bf16 caches: the output is rounded to bf16 (half an ulp is
    2^-9 of the value), which measures 1.7e-3 against 64 bits. `differ`: the pages of one row in some hundreds may
    change where two scores lie closer than fp32 sums in another order."""
    rel = 1e-5 if case["dtype"] == "fp32" else 7e-3
    return {"rel": rel, "max": 40 * rel, "differ": 0.005}


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _keys(case, n_pages, q_b, g):
    """[n_pages, Hkv, S, D] fp32 keys: iid normal | with a mean vector per (page, head) and a few keys that point along
    the query of their head (1 % of the pages) | smooth along time (an AR(1) walk of unit variance per channel)."""
    Hkv, D, S = case["kv_heads"], case["head_dim"], case["page_size"]
    dev = q_b.device
    if case["keys"] == "smooth":
        rho, L = 0.95, 512
        blocks = -(-n_pages * S // L)
        eps = torch.randn((blocks, L, Hkv * D), generator=g, device=dev) * math.sqrt(1 - rho * rho)
        eps[0, 0] /= math.sqrt(1 - rho * rho)
        i = torch.arange(L, device=dev, dtype=torch.float32)
        T = torch.tril(rho ** (i[:, None] - i[None, :]).clamp(min=0))
        x = torch.matmul(T, eps)
        last = x[:-1, -1:].clone()
        x[1:] += (rho ** (i + 1))[:, None] * last  # what is two blocks back has decayed below 1e-11
        return x.view(-1, Hkv, D)[:n_pages * S].view(n_pages, S, Hkv, D).permute(0, 2, 1, 3)
    k = torch.randn((n_pages, Hkv, S, D), generator=g, device=dev)
    if case["keys"] == "shift":
        k += 0.5 * torch.randn((n_pages, Hkv, 1, D), generator=g, device=dev)
        page = torch.rand((n_pages, Hkv, 1), generator=g, device=dev) < 0.01
        slot = torch.rand((n_pages, Hkv, S), generator=g, device=dev) < 2.0 / S
        p, h, t = torch.nonzero(page & slot, as_tuple=True)
        first = q_b.float().view(Hkv, -1, D)[:, 0]
        first = first / first.norm(dim=-1, keepdim=True) * math.sqrt(D)
        k[p, h, t] = 4.0 * first[h] + torch.randn((p.numel(), D), generator=g, device=dev)
    return k


def _inputs(case, seed):
    dev, dtype = torch.device("cuda"), DTYPES[case["dtype"]]
    B, H, Hkv, D, S = (case[k] for k in ("batch", "q_heads", "kv_heads", "head_dim", "page_size"))
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    lens = _lengths(case)
    pages = [-(-n // S) for n in lens]
    q = torch.randn((B, H, D), generator=g, device=dev).to(dtype)
    ids = torch.randperm(sum(pages), generator=g, device=dev).to(torch.int32)  # a pool that has been in use for a while
    table = torch.zeros((B, max(pages)), dtype=torch.int32, device=dev)
    k_cache = torch.zeros((sum(pages), Hkv, S, D), dtype=dtype, device=dev)
    v_cache = torch.zeros_like(k_cache)
    at = 0
    for b, n in enumerate(pages):
        mine = ids[at:at + n]
        at += n
        table[b, :n] = mine
        k_cache[mine.long()] = _keys(case, n, q[b], g).to(dtype)
        v_cache[mine.long()] = torch.randn((n, Hkv, S, D), generator=g, device=dev).to(dtype)
    return q, k_cache, v_cache, table, torch.tensor(lens, dtype=torch.int32, device=dev)


def _chunk_range(case, seq_lens):
    return (seq_lens - case["chunk"]).clamp(min=0), seq_lens.clone()


def prepare(case, seed):
    q, k_cache, v_cache, table, seq_lens = _inputs(case, seed)
    wl = Workload(name="cases", dtype=DTYPES[case["dtype"]], B=case["batch"], H=case["q_heads"], Hkv=case["kv_heads"],
                  D=case["head_dim"], S=case["page_size"], top_k=case["top_k"], lam=LAMBDA, q=q, k_cache=k_cache,
                  v_cache=v_cache, page_table=table, seq_lens=seq_lens)
    s = DecodeSession(wl, stats_dtype=DTYPES[case["stats"]], force_recent_pages=case["recent"],
                      want_scores=case["op"] == "calls")
    state = {"op": case["op"], "session": s}
    if case["op"] in ("step", "calls"):  # statistics are current up to the token that was appended last
        seq_lens -= 1
        s.update_page_stats()
        seq_lens += 1
    if case["op"] == "calls":
        state["begin"], state["end"], state["touched"] = seq_lens - 1, seq_lens.clone(), 1
    elif case["op"] == "chunk":
        s.page_stats.zero_()
        state["begin"], state["end"] = _chunk_range(case, seq_lens)
        state["touched"] = -(-case["chunk"] // case["page_size"]) + 1
    return state


def run(state):
    s, op = state["session"], state["op"]
    if op == "dense":
        s.dense_paged_decode()
        return {"out": s.out_dense, "lse": s.lse_dense}
    if op == "build":
        s.update_page_stats()
        return {"mean": s.page_mean, "std": s.page_std}
    if op == "chunk":
        s.update_page_stats(state["begin"], state["end"], state["touched"])
        return {"mean": s.page_mean, "std": s.page_std}
    got = {}
    if op == "step":
        s.decode_step(refresh_tail=True)
    else:
        s.update_page_stats(state["begin"], state["end"], state["touched"])
        s.score_select_topk()
        s.sparse_paged_decode()
        got["scores"] = s.scores
    got.update(out=s.out, lse=s.lse, pages=s.sel_pages, count=s.sel_count, mean=s.page_mean, std=s.page_std)
    return got


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

def _attend(q, k, v):
    """q [G, D], k / v [tokens, D] in 64 bits -> output rows and the log of the sum of the exponentials."""
    logits = q @ k.T / math.sqrt(q.shape[-1])
    lse = torch.logsumexp(logits, dim=-1)
    return torch.exp(logits - lse[:, None]) @ v, lse


def exact(case, seed):
    q, k_cache, v_cache, table, seq_lens = _inputs(case, seed)
    B, H, Hkv, D, S = (case[k] for k in ("batch", "q_heads", "kv_heads", "head_dim", "page_size"))
    dev, op, k_sel = q.device, case["op"], case["top_k"]
    lens = seq_lens.tolist()
    qd = q.double().view(B, Hkv, H // Hkv, D)
    out = torch.zeros((B, Hkv, H // Hkv, D), dtype=torch.float64, device=dev)
    lse = torch.zeros((B, Hkv, H // Hkv), dtype=torch.float64, device=dev)
    if op == "dense":
        for b, n in enumerate(lens):
            ids = table[b, :-(-n // S)].long()
            for h in range(Hkv):
                kh, vh = (c[ids, h].reshape(-1, D)[:n].double() for c in (k_cache, v_cache))
                out[b, h], lse[b, h] = _attend(qd[b, h], kh, vh)
        return {"out": out.view(B, H, D), "lse": lse.view(B, H)}

    mean = torch.zeros((k_cache.shape[0], Hkv, D), dtype=torch.float64, device=dev)
    std = torch.zeros((k_cache.shape[0], Hkv), dtype=torch.float64, device=dev)
    pages = torch.full((B, Hkv, k_sel), -1, dtype=torch.int32, device=dev)
    count = torch.zeros((B, Hkv), dtype=torch.int32, device=dev)
    scores = torch.full((B, Hkv, table.shape[1]), float("nan"), dtype=torch.float64, device=dev)
    for b, n in enumerate(lens):
        P = -(-n // S)
        first = max(0, n - case["chunk"]) // S if op == "chunk" else 0
        for p0 in range(first, P, 8192):
            p1 = min(P, p0 + 8192)
            ids = table[b, p0:p1].long()
            n_tok = (n - torch.arange(p0, p1, device=dev) * S).clamp(max=S)
            valid = (torch.arange(S, device=dev)[None, :] < n_tok[:, None])[:, None, :, None].double()
            x = k_cache[ids].double()
            m = (x * valid).sum(2) / n_tok[:, None, None]
            x = (x - m[:, :, None]) * valid
            mean[ids] = m
            std[ids] = ((x * x).sum((2, 3)) / n_tok[:, None]).sqrt()
        if op in ("build", "chunk"):
            continue
        ids = table[b, :P].long()
        m = mean[ids].to(DTYPES[case["stats"]]).double()  # scores are over the statistics as stored
        sc = torch.einsum("hgd,phd->hgp", qd[b], m)
        sc = (sc + LAMBDA * qd[b].norm(dim=-1)[:, :, None] * std[ids].T[:, None, :]).amax(1)
        scores[b, :, :P] = sc
        kb = min(k_sel, P)
        rank = sc.clone()
        if case["recent"]:
            rank[:, P - min(case["recent"], kb):] = float("inf")
        top = torch.sort(rank, dim=-1, descending=True, stable=True)[1][:, :kb].sort(-1)[0]
        pages[b, :, :kb] = top.int()
        count[b] = kb
        for h in range(Hkv):
            keep = (top[h][:, None] * S + torch.arange(S, device=dev)).reshape(-1) < n
            kh, vh = (c[ids[top[h]], h].reshape(-1, D)[keep].double() for c in (k_cache, v_cache))
            out[b, h], lse[b, h] = _attend(qd[b, h], kh, vh)
    stats = {"mean": mean, "std": std}
    if op in ("build", "chunk"):
        return stats
    got = {"out": out.view(B, H, D), "lse": lse.view(B, H), "pages": pages, "count": count, **stats}
    if op == "calls":
        got["scores"] = scores
    return got
