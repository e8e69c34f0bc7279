"""The work a prefill node has this library do, as cases that can be timed.

A case is a dict of plain values.  Four kinds, each through the public entry points of
``paper_2407_00079_amd.binding`` in the order a prefill program calls them:

  attn    one layer of chunked prefill of a batch: the chunk's new K/V rows go into their pages, then the new
          tokens attend to the reused prefix and themselves.  ``call`` is how the program drives it:
            one_shot  append and attention build and upload their own tables in every call, with a workspace that
                      has room for key slices (the README's first example)
            planned   the batch's plan was prepared once, the layer only launches (a layer loop)
            noalloc   attention without a workspace (under graph capture, or where nothing may be allocated)
  pages   layer-wise streaming inside HBM: the page order of the request once, then per layer unpack (load) and
          pack (store)
  host    layer-wise streaming against pinned host memory: per layer the reused prefix pages are loaded on one
          stream and the pages the new tokens filled are stored on another
  prefix  the scheduler's side: block keys of a batch of prompts and their longest prefix match against the
          prefill instances' caches

Lists of lengths are texts ("811,328"): one entry per request.
"""
import math

import numpy as np
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

DEV = "cuda:0"
PAGE = 16


def _ints(text):
    return [int(x) for x in text.split(",")]


def _text(values):
    return ",".join(str(int(v)) for v in values)


def _pages_of(case):
    return [-(-(p + c) // PAGE) for p, c in zip(_ints(case["prefix"]), _ints(case["new"]))]


def listed():
    mixed = W.config_shapes(4)
    return [
        # the tiny fp32 request: the smallest call, where launches and latency are everything
        dict(name="attn_tiny_f32", kind="attn", call="one_shot", dtype="f32", q_heads=4, kv_heads=1, head_dim=64,
             prefix="256", new="128", pool=64),
        # a short question behind a 128k document that is already cached: 16 new tokens, 131056 reused
        dict(name="attn_question_128k", kind="attn", call="one_shot", dtype="bf16", q_heads=64, kv_heads=8, head_dim=128,
             prefix="131056", new="16", pool=8192),
        # the paper's two printed trace samples in one batch: 6955 and 6472 tokens of which 6144 are shared
        dict(name="attn_trace_pair", kind="attn", call="one_shot", dtype="bf16", q_heads=64, kv_heads=8, head_dim=128,
             prefix="6144,6144", new="811,328", pool=1024),
        # a 16k prompt, half cached: the ordinary prefill of one layer of a 70B-class model
        dict(name="attn_half_cached_16k", kind="attn", call="planned", dtype="bf16", q_heads=64, kv_heads=8, head_dim=128,
             prefix="8192", new="8192", pool=4096),
        # the last chunk of a 128k prompt on one of eight tensor-parallel GPUs
        dict(name="attn_last_chunk_128k", kind="attn", call="planned", dtype="bf16", q_heads=8, kv_heads=1, head_dim=128,
             prefix="122880", new="8192", pool=16384),
        # sixteen requests of very different lengths in one batch: the largest call
        dict(name="attn_mixed_batch", kind="attn", call="planned", dtype="bf16", q_heads=64, kv_heads=8, head_dim=128,
             prefix=_text(mixed["prefix_lens"]), new=_text(mixed["new_lens"]), pool=mixed["num_pages"]),
        # a model with head_dim 64, lengths that are multiples of nothing
        dict(name="attn_head_dim_64", kind="attn", call="one_shot", dtype="bf16", q_heads=64, kv_heads=8, head_dim=64,
             prefix="8189", new="4099", pool=2048),
        # one pipeline stage's share (8 of 80 layers) of a 32k sequence: 2048 pages of 32 KiB each way per layer
        dict(name="pages_stage_32k", kind="pages", layers=8, n=2048, page_bytes=32768, pool=4096, ordered=True),
        # the tiny request's 24 pages for 2 layers: copies of a few microseconds each
        dict(name="pages_tiny", kind="pages", layers=2, n=24, page_bytes=4096, pool=64, ordered=False),
        # the trace sample against the host pool: 384 prefix pages in, 51 chunk pages out, for 4 layers
        dict(name="host_trace_sample", kind="host", layers=4, n_load=384, n_store=51, page_bytes=32768, pool=1024),
        # a scheduler's queue of long prompts against the caches of 16 prefill instances
        dict(name="prefix_queue", kind="prefix", tokens=_text([131072] * 64), block=512, instances=16, cached=200000),
        # one arriving request of the trace's length against 4 instances: pure latency
        dict(name="prefix_one_request", kind="prefix", tokens="6955", block=512, instances=4, cached=20000),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


#: rates (flop/s) that turn a drawn case's work into a rough time, so that none costs more than the largest listed case
_RATE = {("bf16", 128): 1.2e15, ("bf16", 64): 0.95e15, ("f32", 64): 0.12e15}


def _seconds(case):
    return work(case)["flops"] / _RATE[case["dtype"], case["head_dim"]]


def _draw_attn(rng):
    dtype, head_dim = rng.choice([("bf16", 128)] * 4 + [("bf16", 64), ("f32", 64)])
    q_heads, kv_heads = rng.choice([(64, 8), (64, 8), (8, 1), (16, 2), (8, 2), (4, 1), (12, 3), (16, 16)])
    batch = rng.choice([1, 1, 1, 2, 3, 4, 8, 16])
    prefix, new = [], []
    for _ in range(batch):
        prefix.append(0 if rng.random() < 0.15 else _log_uniform(rng, 16, 131056 // batch))
        new.append(_log_uniform(rng, 1, 8192))
    limit = _seconds(next(c for c in listed() if c["name"] == "attn_mixed_batch"))
    while True:
        case = dict(kind="attn", call=rng.choice(["one_shot", "one_shot", "planned", "planned", "noalloc"]), dtype=dtype,
                    q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim, prefix=_text(prefix), new=_text(new))
        case["pool"] = sum(_pages_of(case)) + rng.randrange(1, 512)
        if _seconds(case) <= limit:
            return case
        new = [max(1, c // 2) for c in new]


def draw(rng):
    what = rng.random()
    if what < 0.55:
        return _draw_attn(rng)
    if what < 0.75:
        n = _log_uniform(rng, 1, 2048)
        return dict(kind="pages", layers=rng.randrange(1, 9), n=n, page_bytes=rng.choice([2048, 4096, 8192, 16384, 32768, 24576]),
                    pool=n + rng.randrange(1, 2048), ordered=rng.random() < 0.5)
    if what < 0.82:
        n_load, n_store = _log_uniform(rng, 1, 512), _log_uniform(rng, 1, 128)
        return dict(kind="host", layers=rng.randrange(1, 5), n_load=n_load, n_store=n_store,
                    page_bytes=rng.choice([4096, 32768]), pool=n_load + n_store + rng.randrange(1, 512))
    batch = _log_uniform(rng, 1, 64)
    return dict(kind="prefix", tokens=_text([_log_uniform(rng, 200, 131072) for _ in range(batch)]), block=512,
                instances=rng.randrange(1, 21), cached=_log_uniform(rng, 100, 200000))


# ---------------------------------------------------------------------------------------------------------------------
# what the program has in hand before the call
# ---------------------------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _prepare_attn(case, seed):
    g = _gen(seed)
    prefix, new = _ints(case["prefix"]), _ints(case["new"])
    Hq, Hkv, D = case["q_heads"], case["kv_heads"], case["head_dim"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    pages, total = _pages_of(case), sum(new)
    s = dict(case=case, prefix=prefix, new=new)
    s["params"] = B.attn_params(Hq, Hkv, D, PAGE, case["pool"], case["dtype"])
    s["q"] = torch.randn(total, Hq, D, device=DEV, dtype=dt, generator=g)
    s["k"] = torch.randn(case["pool"], Hkv, PAGE, D, device=DEV, dtype=dt, generator=g)
    s["v"] = torch.randn(case["pool"], Hkv, PAGE, D, device=DEV, dtype=dt, generator=g)
    s["k_new"] = torch.randn(total, Hkv, D, device=DEV, dtype=dt, generator=g)
    s["v_new"] = torch.randn(total, Hkv, D, device=DEV, dtype=dt, generator=g)
    # every request's pages are scattered over the pool: slices of one permutation of its page ids
    perm = torch.randperm(case["pool"], device=DEV, generator=g).to(torch.int32)
    table = torch.zeros(len(new), max(pages), device=DEV, dtype=torch.int32)
    at = 0
    for r, n in enumerate(pages):
        table[r, :n] = perm[at:at + n]
        at += n
    s["table"] = table
    s["out"] = torch.empty(total, Hq, D, device=DEV, dtype=dt)
    s["lse"] = torch.empty(total, Hq, device=DEV, dtype=torch.float32)

    def room(n):
        return torch.empty(max(n, 16), dtype=torch.uint8, device=DEV)

    if case["call"] == "planned":
        s["ws"] = room(B.mc_prefill_attn_workspace_bytes(s["params"], len(new), total))
        s["plan"] = B.mc_prefill_attn_prepare(s["params"], prefix, new, 0, s["ws"])
    else:
        s["append_ws"] = room(B.mc_kv_append_workspace_bytes(len(new)))
        if case["call"] == "one_shot":
            s["ws"] = room(B.mc_prefill_attn_auto_workspace_bytes(s["params"], prefix, new))
    return s


def _bytes(g, *shape):
    return torch.randint(0, 256, shape, dtype=torch.uint8, device=DEV, generator=g)


def _prepare_pages(case, seed):
    g = _gen(seed)
    L, n, pb, N = case["layers"], case["n"], case["page_bytes"], case["pool"]
    return dict(case=case,
                load_ids=torch.randperm(N, device=DEV, generator=g)[:n].to(torch.int32),
                store_ids=torch.randperm(N, device=DEV, generator=g)[:n].to(torch.int32),
                order=torch.empty(n, dtype=torch.int32, device=DEV),
                # what arrives, the pools it goes into; the pools that are stored from, what leaves
                k_in=_bytes(g, L, n, pb), v_in=_bytes(g, L, n, pb), k_to=_bytes(g, L, N, pb), v_to=_bytes(g, L, N, pb),
                k_from=_bytes(g, L, N, pb), v_from=_bytes(g, L, N, pb),
                k_out=torch.empty(L, n, pb, dtype=torch.uint8, device=DEV),
                v_out=torch.empty(L, n, pb, dtype=torch.uint8, device=DEV))


def _prepare_host(case, seed):
    g = _gen(seed)
    L, nl, ns, pb, N = case["layers"], case["n_load"], case["n_store"], case["page_bytes"], case["pool"]
    ids = torch.randperm(N, device=DEV, generator=g).to(torch.int32)

    def pinned(n, fill):
        t = torch.empty(L, n, pb, dtype=torch.uint8, pin_memory=True)
        if fill:
            t.copy_(_bytes(g, L, n, pb))
        return t

    s = dict(case=case, load_ids=ids[:nl].contiguous(), store_ids=ids[nl:nl + ns].contiguous(),
             k_host_in=pinned(nl, True), v_host_in=pinned(nl, True), k_host_out=pinned(ns, False), v_host_out=pinned(ns, False),
             k_pool=_bytes(g, L, N, pb), v_pool=_bytes(g, L, N, pb), load_stream=torch.cuda.Stream(),
             store_stream=torch.cuda.Stream())
    for name, n in (("in", nl), ("out", ns)):
        for t in "kv":
            s[f"{t}_stage_{name}"] = torch.empty(L, n, pb, dtype=torch.uint8, device=DEV)
    return s


def _ascending(keys):
    """int64 bit patterns in ascending order of the uint64 values they stand for, without repeats"""
    u = torch.unique(keys)
    return torch.cat([u[u >= 0], u[u < 0]])


def _prepare_prefix(case, seed):
    g = _gen(seed)
    lens, block, NI = _ints(case["tokens"]), case["block"], case["instances"]
    off = np.concatenate([[0], np.cumsum(lens)]).tolist()
    blocks = [-(-n // block) for n in lens]
    koff = np.concatenate([[0], np.cumsum(blocks)]).tolist()
    s = dict(case=case, tok_offsets=off, key_offsets=koff)
    s["tokens"] = torch.randint(0, 128000, (off[-1],), dtype=torch.int32, device=DEV, generator=g)
    s["keys"] = torch.empty(koff[-1], dtype=torch.int64, device=DEV)
    s["hash_ws"] = torch.empty(B.mc_prefix_hash_workspace_bytes(len(lens)), dtype=torch.uint8, device=DEV)
    s["match_ws"] = torch.empty(B.mc_prefix_match_workspace_bytes(len(lens), NI), dtype=torch.uint8, device=DEV)
    B.mc_prefix_hash(s["tokens"], off, block, s["keys"], s["hash_ws"])
    # an instance's cache: keys of prompts it has seen, and of each waiting prompt a leading part that it holds
    at = torch.arange(koff[-1], device=DEV)
    first = torch.tensor(koff[:-1], device=DEV).repeat_interleave(torch.tensor(blocks, device=DEV))
    count = torch.tensor(blocks, device=DEV).repeat_interleave(torch.tensor(blocks, device=DEV))
    caches, coff = [], [0]
    for i in range(NI):
        half = torch.randint(0, 2 ** 32, (2, case["cached"]), dtype=torch.int64, device=DEV, generator=g)
        seen = half[0] << 32 | half[1]
        held = s["keys"][(at - first) * NI < count * i]
        caches.append(_ascending(torch.cat([seen, held])))
        coff.append(coff[-1] + caches[-1].numel())
    s["cache"], s["cache_offsets"] = torch.cat(caches), coff
    s["prefix_len"] = torch.empty(len(lens), NI, dtype=torch.int32, device=DEV)
    s["best_len"] = torch.empty(len(lens), dtype=torch.int32, device=DEV)
    s["best_inst"] = torch.empty(len(lens), dtype=torch.int32, device=DEV)
    return s


def prepare(case, seed):
    return {"attn": _prepare_attn, "pages": _prepare_pages, "host": _prepare_host, "prefix": _prepare_prefix}[case["kind"]](case, seed)


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------
def _run_attn(s):
    p, call = s["params"], s["case"]["call"]
    if call == "planned":
        B.mc_kv_append_run(p, s["plan"], s["k_new"], s["v_new"], s["k"], s["v"], s["table"], s["ws"])
        B.mc_prefill_attn_run(p, s["plan"], s["q"], s["k"], s["v"], s["table"], s["out"], s["lse"], s["ws"])
    else:
        B.mc_kv_append_paged(p, s["k_new"], s["v_new"], s["k"], s["v"], s["table"], s["prefix"], s["new"], s["append_ws"])
        if call == "noalloc":
            B.mc_prefill_attn_paged_noalloc(p, s["q"], s["k"], s["v"], s["table"], s["prefix"], s["new"], s["out"], s["lse"])
        else:
            B.mc_prefill_attn_paged(p, s["q"], s["k"], s["v"], s["table"], s["prefix"], s["new"], s["out"], s["lse"], s["ws"])
    return dict(out=s["out"], lse=s["lse"], k=s["k"], v=s["v"])


def _run_pages(s):
    c = s["case"]
    n, pb, N = c["n"], c["page_bytes"], c["pool"]
    if c["ordered"]:
        B.mc_kv_page_order(s["load_ids"], n, s["order"])
    for l in range(c["layers"]):
        if c["ordered"]:
            B.mc_kv_unpack_layer_ordered(s["k_in"][l], s["v_in"][l], N, pb, s["load_ids"], s["order"], n, s["k_to"][l], s["v_to"][l])
        else:
            B.mc_kv_unpack_layer(s["k_in"][l], s["v_in"][l], N, pb, s["load_ids"], n, s["k_to"][l], s["v_to"][l])
        B.mc_kv_pack_layer(s["k_from"][l], s["v_from"][l], N, pb, s["store_ids"], n, s["k_out"][l], s["v_out"][l])
    out = dict(k_to=s["k_to"], v_to=s["v_to"], k_out=s["k_out"], v_out=s["v_out"])
    return dict(out, order=s["order"]) if c["ordered"] else out


def _run_host(s):
    c = s["case"]
    pb, N = c["page_bytes"], c["pool"]
    now = torch.cuda.current_stream()
    s["load_stream"].wait_stream(now)
    s["store_stream"].wait_stream(now)
    for l in range(c["layers"]):
        B.mc_kv_load_layer(s["k_host_in"][l], s["v_host_in"][l], s["k_stage_in"][l], s["v_stage_in"][l], N, pb, s["load_ids"],
                           c["n_load"], s["k_pool"][l], s["v_pool"][l], s["load_stream"])
        B.mc_kv_store_layer(s["k_pool"][l], s["v_pool"][l], N, pb, s["store_ids"], c["n_store"], s["k_stage_out"][l],
                            s["v_stage_out"][l], s["k_host_out"][l], s["v_host_out"][l], s["store_stream"])
    now.wait_stream(s["load_stream"])
    now.wait_stream(s["store_stream"])
    return dict(k_pool=s["k_pool"], v_pool=s["v_pool"], k_host_out=s["k_host_out"], v_host_out=s["v_host_out"])


def _run_prefix(s):
    B.mc_prefix_hash(s["tokens"], s["tok_offsets"], s["case"]["block"], s["keys"], s["hash_ws"])
    B.mc_prefix_match(s["keys"], s["key_offsets"], s["cache"], s["cache_offsets"], s["prefix_len"], s["best_len"], s["best_inst"],
                      s["match_ws"])
    return dict(keys=s["keys"], prefix_len=s["prefix_len"], best_len=s["best_len"], best_inst=s["best_inst"])


def run(state):
    return {"attn": _run_attn, "pages": _run_pages, "host": _run_host, "prefix": _run_prefix}[state["case"]["kind"]](state)


# ---------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how closely two correct implementations agree
# ---------------------------------------------------------------------------------------------------------------------
def work(case):
    if case["kind"] == "attn":
        prefix, new = _ints(case["prefix"]), _ints(case["new"])
        Hq, Hkv, D = case["q_heads"], case["kv_heads"], case["head_dim"]
        size = 2 if case["dtype"] == "bf16" else 4
        keys = sum(p + c for p, c in zip(prefix, new) if c)
        pairs = sum(c * p + c * (c + 1) // 2 for p, c in zip(prefix, new))
        total = sum(new)
        # Q in, O and LSE out, the new rows in and into their pages, every visible K and V row once
        bytes_ = total * Hq * (2 * D * size + 4) + 2 * 2 * total * Hkv * D * size + 2 * keys * Hkv * D * size + 4 * sum(_pages_of(case))
        return {"bytes": bytes_, "flops": 4 * D * Hq * pairs}
    if case["kind"] == "pages":
        per_layer = 2 * 2 * 2 * case["n"] * case["page_bytes"]          # load and store, K and V, read and write
        return {"bytes": case["layers"] * per_layer + 4 * case["n"] * (3 if case["ordered"] else 2), "flops": 0}
    if case["kind"] == "host":
        # each byte is read in one memory and written in the other
        return {"bytes": case["layers"] * 2 * 2 * (case["n_load"] + case["n_store"]) * case["page_bytes"], "flops": 0}
    lens = _ints(case["tokens"])
    blocks = sum(-(-n // case["block"]) for n in lens)
    # tokens in, keys out and in again, and for every key and instance at least the entry that decides it
    return {"bytes": 4 * sum(lens) + 16 * blocks + 8 * blocks * case["instances"] + 4 * len(lens) * (case["instances"] + 2), "flops": 0}


def tolerance(case):
    if case["kind"] != "attn":
        return "exact"
    # four times what the path shows against the same attention in 64 bits (bf16: rel 2.35e-3, largest 0.03 of the root mean
    # square, from the rounding of the probabilities and of the output; f32: rel 5.8e-7, largest 4.7e-6)
    return {"rel": 9e-3, "max": 0.12} if case["dtype"] == "bf16" else {"rel": 2.5e-6, "max": 2e-5}
