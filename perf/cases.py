"""The measured cases: what a serving program asks of one GPU of an elastic sequence-parallel group.

Three paths, all through the ctypes binding, with the outputs and the workspace of a call kept by the caller from step to
step (as a serving loop keeps them):

  decode   one decoding step of the requests this instance is master of: the new tokens' K/V rows are saved in the pool,
           then every request's query attends its resident rows; with peers, combined with the partial results that the
           other instances of the group returned for the same queries
  striped  one instance's share of the prefill of a batch: its query stripe against each of the group's KV shards in
           turn (fp32 partials), then the merge; with one shard it is the whole prefill on one GPU.  With `keep`, the
           rows are also kept in the token pool while they are attended (proactive scale-down)
  context  the last `new` positions of one request's `context` tokens against the `local` first of them, held as
           `shards` contiguous shards ("dense") or in the token pool ("pool": the tile transfers read the pool rows,
           "staged": through a staging copy).  Where the local rows reach to the end of the context, the new tokens'
           own rows are saved in the pool first (a follow-up turn of a chat, the next chunk of a long prompt)

Sizes: the five configurations of workloads.py, the head layouts of the tests, and request lengths of the kinds of traffic
they stand for (short chats, long documents).  Values are N(0, 1) in bf16, pool slots a random permutation.
"""
import math

import numpy as np
import torch

from paper_2404_09526_amd import binding as esp
from paper_2404_09526_amd import workloads as wl

DIM = wl.HEAD_DIM
SCALE = 1.0 / math.sqrt(DIM)


# ----------------------------------------------------------------------------------------------------------- the cases
def decode_case(requests, median, lo, hi, q_heads, kv_heads, peers, length_seed):
    return {"path": "decode", "requests": requests, "median": median, "lo": lo, "hi": hi, "q_heads": q_heads,
            "kv_heads": kv_heads, "peers": peers, "length_seed": length_seed}


def striped_case(chunks, shards, q_heads, kv_heads, keep):
    return {"path": "striped", "chunks": ",".join(str(c) for c in chunks), "shards": shards, "q_heads": q_heads,
            "kv_heads": kv_heads, "keep": keep}


def context_case(new, context, local, shards, q_heads, kv_heads, rows):
    return {"path": "context", "new": new, "context": context, "local": local, "shards": shards, "q_heads": q_heads,
            "kv_heads": kv_heads, "rows": rows}


def listed():
    return [
        # the smallest step there is (configuration 1): four short requests on four heads; launches and latency
        dict(decode_case(4, 256, 64, 512, 4, 4, 3, 0), name="decode-4-short"),
        # a chat service at low load: sixteen conversations of a few hundred tokens, grouped queries, one instance
        dict(decode_case(16, 600, 32, 4096, 32, 8, 0, 5), name="decode-16-chats-gqa"),
        # the same at medium load on the multi-head layout, decoded by a group of four
        dict(decode_case(32, 2048, 128, 16384, 32, 32, 3, 6), name="decode-32-mha"),
        # configuration 3: 64 requests, lognormal slices of 1K .. 128K tokens, multi-head
        dict(decode_case(64, 8192, 1024, 131072, 32, 32, 3, 2), name="decode-64-long-mha"),
        # configuration 5's decode on half its requests: slices of 512 .. 1M tokens, grouped queries
        dict(decode_case(128, 16384, 512, 1 << 20, 32, 8, 3, 4), name="decode-128-long-gqa"),
        # one KV head for all queries: the layout with the smallest rows
        dict(decode_case(64, 4096, 256, 65536, 32, 1, 0, 7), name="decode-64-mqa"),
        # configuration 1's prefill: 256 queries against two contiguous shards of 512 on four heads
        dict(context_case(256, 1024, 1024, 2, 4, 4, "dense"), name="prefill-256-two-shards"),
        # prompts of a chat service as one batch, prefilled on one GPU: ragged, a few hundred tokens each
        dict(striped_case([37, 129, 517, 1033, 260, 2047], 1, 32, 8, False), name="prefill-6-short-prompts"),
        # a follow-up turn: 300 new tokens against a conversation of 20K tokens that sits in the pool
        dict(context_case(300, 20300, 20300, 1, 32, 8, "pool"), name="prefill-turn-from-pool"),
        # configuration 2: the LWM-7B-shaped share, 8192 queries against four striped shards of 8192
        dict(striped_case([8192], 4, 32, 32, False), name="prefill-8192-four-shards"),
        # a var-len batch of configuration 5's kind over a group of two whose rows are kept for the scale-down
        dict(striped_case([1000, 2048, 4096, 8192], 2, 32, 8, True), name="prefill-batch-kept-gqa"),
        # configuration 4: the last 32768 positions of a 512K context against its first half
        dict(context_case(32768, 524288, 262144, 1, 32, 32, "dense"), name="prefill-256k-context"),
    ]


HEADS = ((32, 32), (32, 8), (32, 8), (64, 8), (32, 1), (32, 4), (16, 16), (8, 8), (40, 8), (12, 12), (4, 4))


def log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    while True:
        Hq, Hkv = rng.choice(HEADS)
        path = rng.choice(("decode", "decode", "striped", "context"))
        if path == "decode":
            median = log_uniform(rng, 100, 40000)
            case = decode_case(log_uniform(rng, 1, 256), median, max(1, median // 16), median * 16, Hq, Hkv, rng.choice((0, 1, 3)),
                               rng.randrange(1000))
        elif path == "striped":
            top = log_uniform(rng, 64, 16384)
            chunks = [log_uniform(rng, max(1, top // 16), top) for _ in range(rng.randint(1, 8))]
            case = striped_case(chunks, rng.choice((1, 1, 2, 4)), Hq, Hkv, rng.random() < 0.25)
        else:
            context = log_uniform(rng, 512, 262144)
            new = min(context, log_uniform(rng, 16, 16384))
            rows = rng.choice(("dense", "pool", "pool", "staged"))
            shards = rng.choice((1, 1, 2, 4)) if rows == "dense" else 1
            local = context // shards * shards
            case = context_case(new, local, local, shards, Hq, Hkv, rows)
        w = work(case)
        if w["bytes"] <= 12e9 and w["flops"] <= 2.5e13:
            return case


# ------------------------------------------------------------------------------------------------------- sizes and work
def lengths(case):
    return wl.lognormal_lengths(case["requests"], case["median"], case["lo"], case["hi"], case["length_seed"])


def chunk_list(case):
    return [int(c) for c in case["chunks"].split(",")]


def work(case):
    Hq, Hkv = case["q_heads"], case["kv_heads"]
    row, head_row = 2 * Hkv * DIM * 2, Hq * DIM * 2                   # one token's K and V; its queries or outputs
    if case["path"] == "decode":
        B, n = case["requests"], int(lengths(case).sum())
        bytes_ = n * (row + 4) + B * (2 * row + 4)                    # resident rows and their slots; the new rows, saved
        bytes_ += (B + 1) * 4 + B * (2 * head_row + Hq * 4) + case["peers"] * B * (head_row + Hq * 4)
        return {"bytes": bytes_, "flops": 4 * DIM * Hq * n}
    if case["path"] == "striped":
        chunks, S = chunk_list(case), case["shards"]
        T = sum(chunks)
        pairs = sum(c * (c + 1) // 2 + (S - 1) * (c * (c - 1) // 2) for c in chunks)
        bytes_ = T * (2 * head_row + 4 + Hq * 4) + S * T * (row + 4)
        if case["keep"]:
            bytes_ += S * T * (row + 4)
        return {"bytes": bytes_, "flops": 4 * DIM * Hq * pairs}
    new, first, local = case["new"], case["context"] - case["new"], case["local"]
    seen = np.minimum(np.arange(first, first + new, dtype=np.int64) + 1, local)
    bytes_ = new * (2 * head_row + 4 + Hq * 4) + local * (row + 4)
    if case["rows"] != "dense":
        bytes_ += local * 4 + (new * (2 * row + 4) if local == case["context"] else 0)
    return {"bytes": bytes_, "flops": 4 * DIM * Hq * int(seen.sum())}


def tolerance(case):
    # O is bf16 and the probabilities are rounded to bf16 for the second product.  Measured against attention in float64 on
    # the cases up to 1.5 TFLOP / 2 GB: O 1.7e-3 .. 2.3e-3 relative, largest single difference 4e-3 .. 4e-2 (rows that see
    # few keys); the LSE 3e-8 .. 5e-8, the pool rows exact.
    return {"rel": 1e-2, "max": 0.16}


# --------------------------------------------------------------------------------------------------------------- inputs
def normal(shape, gen):
    return torch.empty(shape, dtype=torch.bfloat16, device=gen.device).normal_(generator=gen)


def ints(values):
    return torch.as_tensor(np.asarray(values, dtype=np.int32)).cuda()


def offsets(lens):
    return ints(np.concatenate([[0], np.cumsum(lens)]))


def pool(slots, heads, gen):
    return normal((slots, heads, DIM), gen), normal((slots, heads, DIM), gen)


def slot_list(n, slots, gen):
    """n distinct slots in random order."""
    return torch.randperm(slots, generator=gen, device=gen.device)[:n].to(torch.int32)


def outputs(rows, heads, dtype=torch.bfloat16):
    return (torch.empty((rows, heads, DIM), dtype=dtype, device="cuda"), torch.empty((rows, heads), dtype=torch.float32, device="cuda"))


def bytes_of(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    return {"decode": prepare_decode, "striped": prepare_striped, "context": prepare_context}[case["path"]](case, gen)


def prepare_decode(case, gen):
    B, Hq, Hkv = case["requests"], case["q_heads"], case["kv_heads"]
    lens = lengths(case)
    total = int(lens.sum())
    slots = total + total // 8 + 64
    s = {"path": "decode", "max_len": int(lens.max()), "offsets": offsets(lens), "slot_idx": slot_list(total, slots, gen)}
    s["q"] = normal((B, Hq, DIM), gen)
    s["k_pool"], s["v_pool"] = pool(slots, Hkv, gen)
    s["new_k"], s["new_v"] = pool(B, Hkv, gen)
    s["new_slots"] = s["slot_idx"][s["offsets"][1:].long() - 1].clone()   # a request's last resident row is its new token's
    s["peer_O"] = [normal((B, Hq, DIM), gen) for _ in range(case["peers"])]
    s["peer_LSE"] = [torch.empty((B, Hq), device="cuda").normal_(math.log(case["median"]), 1.0, generator=gen) for _ in range(case["peers"])]
    s["O"], s["LSE"] = outputs(B, Hq)
    s["ws"] = bytes_of(esp.esp_decode_workspace_bytes(B, total, s["max_len"], Hq, Hkv, DIM))
    return s


def prepare_striped(case, gen):
    Hq, Hkv, S = case["q_heads"], case["kv_heads"], case["shards"]
    chunks = chunk_list(case)
    T = sum(chunks)
    local = np.concatenate([np.arange(c, dtype=np.int64) for c in chunks])
    single = len(chunks) == 1
    s = {"path": "striped", "keep": case["keep"], "q": normal((T, Hq, DIM), gen), "q_pos": ints(S * local)}
    s["cu"] = None if single else offsets(chunks)
    s["longest"] = None if single else max(chunks)
    s["k"] = [normal((T, Hkv, DIM), gen) for _ in range(S)]
    s["v"] = [normal((T, Hkv, DIM), gen) for _ in range(S)]
    s["kv_pos"] = [ints(S * local + j) for j in range(S)]
    s["parts"] = [outputs(T, Hq, torch.bfloat16 if S == 1 else torch.float32) for _ in range(S)]
    s["O"], s["LSE"] = outputs(T, Hq) if S > 1 else s["parts"][0]
    s["ws"] = bytes_of(esp.esp_prefill_workspace_bytes(T, T, len(chunks), Hq, Hkv, DIM))
    if case["keep"]:
        slots = S * T + S * T // 8
        s["k_pool"], s["v_pool"] = pool(slots, Hkv, gen)
        s["slots"] = list(slot_list(S * T, slots, gen).view(S, T).unbind(0))
    return s


def prepare_context(case, gen):
    Hq, Hkv, new, local, S = case["q_heads"], case["kv_heads"], case["new"], case["local"], case["shards"]
    first = case["context"] - new
    s = {"path": "context", "rows": case["rows"], "q": normal((new, Hq, DIM), gen), "q_pos": ints(np.arange(first, first + new))}
    s["O"], s["LSE"] = outputs(new, Hq)
    if case["rows"] == "dense":
        n = local // S
        s["k"] = [normal((n, Hkv, DIM), gen) for _ in range(S)]
        s["v"] = [normal((n, Hkv, DIM), gen) for _ in range(S)]
        s["kv_pos"] = [ints(np.arange(j * n, (j + 1) * n)) for j in range(S)]
        s["parts"] = [outputs(new, Hq, torch.float32) for _ in range(S)] if S > 1 else [(s["O"], s["LSE"])]
        s["ws"] = bytes_of(esp.esp_prefill_workspace_bytes(new, n, 1, Hq, Hkv, DIM))
        return s
    slots = local + local // 8 + 64
    s["k_pool"], s["v_pool"] = pool(slots, Hkv, gen)
    s["slots"] = slot_list(local, slots, gen)
    s["kv_pos"] = ints(np.arange(local))
    if local == case["context"]:
        s["new_k"], s["new_v"] = pool(new, Hkv, gen)
        s["new_slots"] = s["slots"][local - new:].clone()
    size = esp.esp_prefill_pool_workspace_bytes if case["rows"] == "staged" else esp.esp_prefill_workspace_bytes
    s["ws"] = bytes_of(size(new, local, 1, Hq, Hkv, DIM))
    return s


# ------------------------------------------------------------------------------------------------------------- one pass
def run(s):
    return {"decode": run_decode, "striped": run_striped, "context": run_context}[s["path"]](s)


def run_decode(s):
    esp.esp_kv_append(s["new_k"], s["new_v"], s["new_slots"], s["k_pool"], s["v_pool"])
    if s["peer_O"]:
        esp.esp_partial_attn_decode_merge(s["q"], s["k_pool"], s["v_pool"], s["slot_idx"], s["offsets"], s["max_len"], s["peer_O"],
                                          s["peer_LSE"], softmax_scale=SCALE, O=s["O"], LSE=s["LSE"], workspace=s["ws"])
    else:
        esp.esp_partial_attn_decode(s["q"], s["k_pool"], s["v_pool"], s["slot_idx"], s["offsets"], s["max_len"],
                                    softmax_scale=SCALE, O=s["O"], LSE=s["LSE"], workspace=s["ws"])
    return s["O"], s["LSE"], s["k_pool"], s["v_pool"]


def run_striped(s):
    out = (s["O"], s["LSE"])
    for j, (O, LSE) in enumerate(s["parts"]):
        if s["keep"]:
            esp.esp_partial_attn_prefill_retain(s["q"], s["k"][j], s["v"][j], s["q_pos"], s["kv_pos"][j], s["slots"][j], s["k_pool"],
                                                s["v_pool"], s["cu"], s["cu"], s["longest"], s["longest"], softmax_scale=SCALE,
                                                O=O, LSE=LSE, workspace=s["ws"])
        else:
            esp.esp_partial_attn_prefill(s["q"], s["k"][j], s["v"][j], s["q_pos"], s["kv_pos"][j], s["cu"], s["cu"], s["longest"],
                                         s["longest"], softmax_scale=SCALE, O=O, LSE=LSE, workspace=s["ws"])
    if len(s["parts"]) > 1:
        esp.esp_merge_partials([p[0] for p in s["parts"]], [p[1] for p in s["parts"]], O=out[0], LSE=out[1])
    return out + (s["k_pool"], s["v_pool"]) if s["keep"] else out


def run_context(s):
    if s["rows"] == "dense":
        for (O, LSE), k, v, kv_pos in zip(s["parts"], s["k"], s["v"], s["kv_pos"]):
            esp.esp_partial_attn_prefill(s["q"], k, v, s["q_pos"], kv_pos, softmax_scale=SCALE, O=O, LSE=LSE, workspace=s["ws"])
        if len(s["parts"]) > 1:
            esp.esp_merge_partials([p[0] for p in s["parts"]], [p[1] for p in s["parts"]], O=s["O"], LSE=s["LSE"])
        return s["O"], s["LSE"]
    if "new_k" in s:
        esp.esp_kv_append(s["new_k"], s["new_v"], s["new_slots"], s["k_pool"], s["v_pool"])
    call = esp.esp_partial_attn_prefill_pool if s["rows"] == "staged" else esp.esp_partial_attn_prefill_pool_direct
    call(s["q"], s["k_pool"], s["v_pool"], s["slots"], s["q_pos"], s["kv_pos"], softmax_scale=SCALE, O=s["O"], LSE=s["LSE"],
         workspace=s["ws"])
    return s["O"], s["LSE"], s["k_pool"], s["v_pool"]
