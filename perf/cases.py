"""The work whose speed counts in this library: twelve listed cases and a generator of more of the same kinds.

Every case is one layer's share of what a serving loop asks of the device: the K/V scatter and the attention of one
prefill batch, one decode step, one cross-attention, or the two ends of one KV page migration, through the calls of
paper_2507_10069_amd.binding.  The head counts are those of the models whose shapes the library's named workloads use
(28 / 4 and 32 / 8 heads of 128, bf16; 4 / 1 heads of 64 for the fp32 path) and the lengths are of the size of those
workloads: images of 576 to 6516 tokens, videos of 16384, text of up to 2048.

A case is a dict of plain values:
  op         "prefill"         emm_kv_scatter + emm_prefill_attn
             "prefill_shared"  emm_kv_scatter + emm_prefill_attn_shared, with the groups its planner finds
             "cross"           emm_cross_attn
             "decode"          emm_kv_scatter + emm_decode_attn
             "decode_step"     emm_decode_step without a plan
             "decode_planned"  emm_decode_step with the units and bounds that emm_shared_prefix_plan_host finds
             "migrate"         emm_kv_pages_pack + emm_kv_pages_unpack into another pool, checksums compared
  dtype, heads, kv_heads, head_dim, page    shapes ("page": tokens per page)
  reqs       requests in the batch
  traffic    "range": cached_lo .. cached_hi cached tokens and new_lo .. new_hi new ones per request, uniform;
             "mixed": half the requests text only (log-uniform 256 .. 2048 new tokens), half with an image of 576 ..
             4096 tokens of which none, half or all is cached and 64 .. 512 new text tokens, in random order;
             "after_mixed": a decode batch whose contexts are those of such a mixed batch after its prefill
  group, shared    consecutive requests per sharing group, and the tokens whose pages they share (0: private pages)
  outliers   share of K elements that are eight times larger
  lengths    seed of the lengths (they belong to the case, the tensors' values to prepare's seed)
"""
import math
import random

import numpy as np
import torch

from paper_2507_10069_amd import binding as B

DEVICE = "cuda"
OUTLIER_FACTOR = 8.0


def _case(name, op, **kw):
    case = {"name": name, "op": op, "dtype": "bf16", "heads": 28, "kv_heads": 4, "head_dim": 128, "page": 16, "reqs": 1,
            "traffic": "range", "cached_lo": 0, "cached_hi": 0, "new_lo": 1, "new_hi": 1, "group": 1, "shared": 0,
            "outliers": 0.0, "lengths": 0}
    assert set(kw) <= set(case), kw
    case.update(kw)
    return case


def listed():
    return [
        # the fp32 path: a short prompt behind a small cached prefix, as a correctness run or a small fp32 model has it
        _case("f32_small_prompt", "prefill", dtype="f32", heads=4, kv_heads=1, head_dim=64, cached_lo=256, cached_hi=256,
              new_lo=64, new_hi=64),
        # eight questions about two images (1024 image and 32 system tokens cached, shared by four requests each)
        _case("image_prefix_batch", "prefill", reqs=8, cached_lo=1056, cached_hi=1056, new_lo=128, new_hi=512, group=4,
              shared=1056, lengths=1002),
        # two long prompts behind cached videos of 64 frames of 256 tokens: the largest prefill, with K outliers
        _case("video_prefix_batch", "prefill", reqs=2, cached_lo=16384, cached_hi=16384, new_lo=2048, new_hi=2048, outliers=0.01),
        # ordinary traffic: text-only requests beside images that are new, half cached or cached
        _case("mixed_traffic", "prefill", heads=32, kv_heads=8, reqs=32, traffic="mixed", lengths=1004),
        # encoder-decoder model: text queries over 6404 cached image tokens, two requests per image
        _case("cross_images", "cross", heads=32, kv_heads=8, reqs=16, cached_lo=6404, cached_hi=6404, new_lo=256, new_hi=1024,
              group=2, shared=6404, lengths=1005),
        # one short question about a video seen before: the time to the first token of a cache hit
        _case("video_question", "prefill", cached_lo=16384, cached_hi=16384, new_lo=36, new_hi=36),
        # many short questions about eight such videos in one batch
        _case("shared_video_questions", "prefill_shared", reqs=64, cached_lo=16384, cached_hi=16384, new_lo=4, new_hi=4, group=8,
              shared=16384),
        # the smallest call: one decode step of one chat about one image
        _case("decode_one_chat", "decode_step", cached_lo=1500, cached_hi=1500),
        # decode steps of a ragged batch, of a long uniform one, and of one whose requests share videos
        _case("decode_ragged", "decode_planned", heads=32, kv_heads=8, reqs=32, traffic="after_mixed", lengths=1004),
        _case("decode_long_batch", "decode", reqs=64, cached_lo=8191, cached_hi=8191),
        _case("decode_shared_videos", "decode_planned", reqs=32, cached_lo=18431, cached_hi=18431, group=4, shared=16384),
        # eight requests with a video each move to another instance: gather, checksum, scatter, checksum again
        _case("migrate_videos", "migrate", reqs=8, cached_lo=18432, cached_hi=18432, new_lo=0, new_hi=0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


#: the most that a drawn case may ask for: what the largest listed ones do
MOST_FLOPS, MOST_BYTES = 1.05e12, 1.2e9


def draw(rng):
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["flops"] <= (MOST_FLOPS if case["dtype"] == "bf16" else 1e9) and w["bytes"] <= MOST_BYTES:
            return case


def _draw_once(rng):
    kind = rng.choice(["f32", "prefill", "prefill", "mixed", "cross", "suffix", "prefill_shared", "decode_step", "decode_ragged",
                       "decode", "decode_shared", "migrate"])
    heads, kv_heads = rng.choice([(28, 4), (32, 8)])
    base = {"heads": heads, "kv_heads": kv_heads, "page": rng.choice([16, 16, 32, 64]), "lengths": rng.randrange(1 << 20)}
    if kind == "f32":
        cached = _log_int(rng, 16, 1024)
        new = _log_int(rng, 8, 256)
        base.update(dtype="f32", heads=rng.choice([4, 8]), kv_heads=rng.choice([1, 2]), head_dim=rng.choice([64, 128]))
        case = _case("", "prefill", reqs=rng.randint(1, 4), cached_lo=cached // 2, cached_hi=cached, new_lo=max(1, new // 2), new_hi=new, **base)
    elif kind == "prefill":
        cached = _log_int(rng, 512, 16384)
        new = _log_int(rng, 64, 2048)
        case = _case("", "prefill", reqs=rng.randint(1, 16), cached_lo=cached, cached_hi=cached, new_lo=max(1, new // 4), new_hi=new,
                     outliers=rng.choice([0.0, 0.01]), **base)
    elif kind == "mixed":
        case = _case("", "prefill", reqs=rng.randint(8, 32), traffic="mixed", **base)
    elif kind == "cross":
        image = rng.randint(576, 6516)
        case = _case("", "cross", reqs=rng.randint(1, 16), cached_lo=image, cached_hi=image, new_lo=16, new_hi=_log_int(rng, 64, 1024),
                     group=2, shared=image, **base)
    elif kind == "suffix":
        cached = _log_int(rng, 1024, 32768)
        case = _case("", "prefill", reqs=_log_int(rng, 1, 32), cached_lo=cached // 2, cached_hi=cached, new_lo=2, new_hi=rng.randint(4, 64), **base)
    elif kind == "prefill_shared":
        shared = _log_int(rng, 2048, 16384) // 64 * 64
        group = rng.randint(2, 8)
        case = _case("", "prefill_shared", reqs=group * rng.randint(1, 8), cached_lo=shared, cached_hi=shared + rng.choice([0, 600]), new_lo=2,
                     new_hi=rng.randint(4, 40), group=group, shared=shared, **base)
    elif kind == "decode_step":
        ctx = _log_int(rng, 100, 131072)
        case = _case("", "decode_step", reqs=rng.randint(1, 2), cached_lo=ctx, cached_hi=ctx, **base)
    elif kind == "decode_ragged":
        case = _case("", "decode_planned", reqs=rng.randint(4, 64), traffic="after_mixed", **base)
    elif kind == "decode":
        ctx = _log_int(rng, 512, 18431)
        case = _case("", "decode", reqs=_log_int(rng, 2, 64), cached_lo=int(ctx * rng.choice([0.25, 0.9, 1.0])), cached_hi=ctx, **base)
    elif kind == "decode_shared":
        shared = _log_int(rng, 1024, 16384) // 64 * 64
        group = rng.randint(2, 8)
        case = _case("", "decode_planned", reqs=group * rng.randint(1, 8), cached_lo=shared + 30, cached_hi=shared + rng.randint(200, 2047),
                     group=group, shared=shared, **base)
    else:
        ctx = _log_int(rng, 256, 18432)
        case = _case("", "migrate", reqs=rng.randint(1, 16), cached_lo=ctx // 2, cached_hi=ctx, new_lo=0, new_hi=0, **base)
    del case["name"]
    return case


def _lengths(case):
    """Cached and new tokens of every request."""
    rng = random.Random(case["lengths"])
    n = case["reqs"]
    if case["traffic"] == "range":
        return ([rng.randint(case["cached_lo"], case["cached_hi"]) for _ in range(n)],
                [rng.randint(case["new_lo"], case["new_hi"]) for _ in range(n)])
    pairs = []
    for i in range(n):
        if i % 2 == 0:
            pairs.append((0, _log_int(rng, 256, 2048)))
        else:
            image = rng.randint(576, 4096)
            cached = int(image * rng.choice([0.0, 0.5, 1.0]))
            pairs.append((cached, image - cached + rng.randint(64, 512)))
    rng.shuffle(pairs)
    if case["traffic"] == "after_mixed":
        pairs = [(c + m, 1) for c, m in pairs]
    return [p[0] for p in pairs], [p[1] for p in pairs]


def _causal(case):
    return case["op"] != "cross"


def _pages(case):
    """Logical pages: for every request the list of page numbers (before they are shuffled over the pool), and how many there are."""
    cached, new = _lengths(case)
    page, rows, count = case["page"], [], 0
    group_pages = {}
    for r, (c, m) in enumerate(zip(cached, new)):
        need = -(-(c + (m if _causal(case) else 0)) // page)
        row = []
        if case["shared"] and case["group"] > 1:
            # pages that receive new tokens are private; a page that is only read may be shared to its last token
            whole = min(case["shared"], c)
            n_shared = whole // page if _causal(case) else -(-whole // page)
            have = group_pages.setdefault(r // case["group"], [])
            while len(have) < n_shared:
                have.append(count)
                count += 1
            row = have[:n_shared]
        while len(row) < need:
            row = row + list(range(count, count + need - len(row)))
            count = row[-1] + 1
        rows.append(row)
    return rows, count


def work(case):
    cached, new = _lengths(case)
    rows, _ = _pages(case)
    elt = 4 if case["dtype"] == "f32" else 2
    d, heads, kv_heads, page = case["head_dim"], case["heads"], case["kv_heads"], case["page"]
    if case["op"] == "migrate":
        one = sum(len(r) for r in rows) * kv_heads * page * d * elt * 2      # K and V pages once
        return {"bytes": 4 * one, "flops": 0}                                # pack: read and write, unpack: the same
    causal = _causal(case)
    pairs = sum(m * c + (m * (m + 1) // 2 if causal else 0) for c, m in zip(cached, new))
    tokens = sum(new)
    seen = {}
    for row, c, m in zip(rows, cached, new):
        ctx = c + (m if causal else 0)
        for i in range(-(-ctx // page)):
            seen[row[i]] = max(seen.get(row[i], 0), min(page, ctx - i * page))
    slots = sum(seen.values())
    nbytes = 2 * slots * kv_heads * d * elt + 2 * tokens * heads * d * elt + 4 * tokens * heads
    if causal:
        nbytes += 4 * tokens * kv_heads * d * elt                            # new K and V read, their slots written
    return {"bytes": nbytes, "flops": 4 * d * heads * pairs}


def tolerance(case):
    """bf16: weights rounded to bf16 for the value product and a bf16 result put two implementations about 3e-3 apart (each measures
    2.0e-3 to 2.8e-3 against 64 bits); fp32: sums in another order; pools, staging and checksums are copies."""
    if case["op"] == "migrate":
        return "exact"
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.2}


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    dt = _dtype(case)
    cached, new = _lengths(case)
    rows, count = _pages(case)
    num_pages, width = count + 8, max(1, max(len(r) for r in rows))
    heads, kv_heads, d, page = case["heads"], case["kv_heads"], case["head_dim"], case["page"]

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=DEVICE, dtype=dt)

    def keys(*shape):
        x = normal(*shape)
        if case["outliers"] > 0:
            for part in x.split(max(1, x.shape[0] // 16)):
                part.mul_(1 + (OUTLIER_FACTOR - 1) * (torch.rand(part.shape, generator=gen, device=DEVICE) < case["outliers"]).to(dt))
        return x

    order = np.random.RandomState(seed % (1 << 31)).permutation(num_pages).astype(np.int32)
    table = np.full((len(rows), width), -1, dtype=np.int32)
    for r, row in enumerate(rows):
        table[r, : len(row)] = order[np.asarray(row, dtype=np.int64)] if row else []
    cu = np.zeros(len(rows) + 1, dtype=np.int32)
    cu[1:] = np.cumsum(new)
    host = {"page_table": table, "prefix_lens": np.asarray(cached, dtype=np.int32), "new_lens": np.asarray(new, dtype=np.int32), "cu_new_lens": cu}
    dev = {k: torch.from_numpy(v).to(DEVICE) for k, v in host.items()}
    s = {"op": case["op"], "host": host, "dev": dev, "k_cache": keys(num_pages, kv_heads, page, d), "v_cache": normal(num_pages, kv_heads, page, d)}
    if case["op"] == "migrate":
        ids = np.concatenate([order[np.asarray(r, dtype=np.int64)] for r in rows])
        n = len(ids)
        other = np.random.RandomState((seed + 1) % (1 << 31)).permutation(n + 8).astype(np.int32)[:n]
        s.update(n=n, num_pages=num_pages, page_bytes=kv_heads * page * d * dt.itemsize, ids=torch.from_numpy(ids).to(DEVICE),
                 other_ids=torch.from_numpy(other).to(DEVICE), staging=torch.empty((n, 2, kv_heads, page, d), device=DEVICE, dtype=dt),
                 k_other=torch.zeros((n + 8, kv_heads, page, d), device=DEVICE, dtype=dt),
                 v_other=torch.zeros((n + 8, kv_heads, page, d), device=DEVICE, dtype=dt),
                 sums=torch.zeros(n, device=DEVICE, dtype=torch.int32), sums_other=torch.zeros(n, device=DEVICE, dtype=torch.int32),
                 mismatches=torch.zeros(1, device=DEVICE, dtype=torch.int32))
        return s
    tokens = int(cu[-1])
    s["q"] = normal(tokens, heads, d)
    if _causal(case):
        s["k_new"], s["v_new"] = keys(tokens, kv_heads, d), normal(tokens, kv_heads, d)
    s["out"] = torch.empty_like(s["q"])
    s["lse"] = torch.empty((tokens, heads), device=DEVICE, dtype=torch.float32)
    batch = B.make_batch(num_reqs=len(rows), num_q_heads=heads, num_kv_heads=kv_heads, head_dim=d, page_size=page, num_pages=num_pages,
                         max_pages_per_req=width, total_new_tokens=tokens, max_new_len=max(new), dtype=case["dtype"],
                         softmax_scale=1.0 / math.sqrt(d), **dev)
    s["batch"] = batch

    def scratch(n):
        return torch.empty(n, device=DEVICE, dtype=torch.uint8) if n else None

    if case["op"] == "decode_planned":
        plan = B.emm_shared_prefix_plan_host(batch, table, host["prefix_lens"], host["new_lens"])
        arrays = {k: torch.from_numpy(np.ascontiguousarray(v if len(v) else np.zeros(1, np.int32))).to(DEVICE)
                  for k, v in plan.items() if isinstance(v, np.ndarray)}
        s["units"] = B.make_shared_prefix(plan["num_units"], planned_tiles=plan["planned_tiles"], max_own_tiles=plan["max_own_tiles"],
                                          max_unit_tiles=plan["max_unit_tiles"], **arrays)
        s["workspace"] = scratch(B.emm_decode_attn_shared_workspace_size(batch, s["units"]))
    elif case["op"] == "decode_step":
        s["units"] = None
        s["workspace"] = scratch(B.emm_decode_attn_shared_workspace_size(batch, B.make_shared_prefix(0)))
    elif case["op"] == "prefill_shared":
        plan = B.emm_prefill_shared_plan_host(batch, table, host["prefix_lens"], host["new_lens"], cu)
        s["groups"] = None
        if plan["num_groups"] > 0:
            arrays = {k: torch.from_numpy(np.ascontiguousarray(v)).to(DEVICE) for k, v in plan.items() if isinstance(v, np.ndarray)}
            groups, own = plan["groups"], plan["own"]
            groups.page_table, groups.prefix_lens = arrays["group_page_table"].data_ptr(), arrays["group_prefix_lens"].data_ptr()
            groups.new_lens, groups.cu_new_lens = arrays["group_new_lens"].data_ptr(), arrays["group_cu_new_lens"].data_ptr()
            own.page_table, own.prefix_lens = arrays["own_page_table"].data_ptr(), arrays["own_prefix_lens"].data_ptr()
            own.new_lens, own.cu_new_lens = dev["new_lens"].data_ptr(), dev["cu_new_lens"].data_ptr()
            s.update(groups=groups, own=own, plan_arrays=arrays)
            s["workspace"] = scratch(B.emm_prefill_attn_shared_workspace_size(groups, own))
        else:                                                                # the planner found nothing to gain: the plain call
            s["workspace"] = scratch(B.emm_prefill_attn_workspace_size(batch))
    else:
        s["workspace"] = scratch(B.emm_prefill_attn_workspace_size(batch))
    return s


def run(s):
    op = s["op"]
    if op == "migrate":
        B.emm_kv_pages_pack(s["k_cache"], s["v_cache"], s["num_pages"], s["page_bytes"], s["ids"], s["n"], s["staging"], s["sums"])
        B.emm_kv_pages_unpack(s["staging"], s["other_ids"], s["n"], s["k_other"], s["v_other"], s["n"] + 8, s["page_bytes"], s["sums_other"],
                              s["sums"], s["mismatches"])
        return {"staging": s["staging"], "k": s["k_other"], "v": s["v_other"], "sums": s["sums"], "sums_other": s["sums_other"],
                "mismatches": s["mismatches"]}
    b, q, kc, vc, out, lse, ws = s["batch"], s["q"], s["k_cache"], s["v_cache"], s["out"], s["lse"], s["workspace"]
    if op == "cross":
        B.emm_cross_attn(b, q, kc, vc, out, lse, ws)
        return {"out": out, "lse": lse}
    if op in ("decode_step", "decode_planned"):
        B.emm_decode_step(b, s["units"], q, s["k_new"], s["v_new"], kc, vc, out, lse, ws)
    else:
        B.emm_kv_scatter(b, s["k_new"], s["v_new"], kc, vc)
        if op == "decode":
            B.emm_decode_attn(b, q, kc, vc, out, lse, ws)
        elif op == "prefill_shared" and s["groups"] is not None:
            B.emm_prefill_attn_shared(s["groups"], s["own"], s["plan_arrays"]["req_shared_len"], q, kc, vc, out, lse, ws)
        else:
            B.emm_prefill_attn(b, q, kc, vc, out, lse, ws)
    return {"out": out, "lse": lse, "k_cache": kc, "v_cache": vc}


def exact(case, seed):
    s = prepare(case, seed)
    if case["op"] == "migrate":
        k, v = s["k_cache"][s["ids"].long()], s["v_cache"][s["ids"].long()]
        k_other, v_other = s["k_other"], s["v_other"]
        k_other[s["other_ids"].long()] = k
        v_other[s["other_ids"].long()] = v
        return {"staging": torch.stack([k, v], dim=1), "k": k_other, "v": v_other, "sums": None, "sums_other": None, "mismatches": 0}
    cached, new = _lengths(case)
    causal, page, heads, kv_heads, d = _causal(case), case["page"], case["heads"], case["kv_heads"], case["head_dim"]
    g = heads // kv_heads
    kc, vc = s["k_cache"], s["v_cache"]
    table = torch.from_numpy(s["host"]["page_table"]).to(DEVICE).long()
    if causal:
        at = 0
        for r, (c, m) in enumerate(zip(cached, new)):
            slot = torch.arange(c, c + m, device=DEVICE)
            pages, offs = table[r, slot // page], slot % page
            kc[pages, :, offs] = s["k_new"][at : at + m]
            vc[pages, :, offs] = s["v_new"][at : at + m]
            at += m
    tokens = int(s["host"]["cu_new_lens"][-1])
    out = torch.zeros((tokens, heads, d), device=DEVICE, dtype=torch.float64)
    lse = torch.full((tokens, heads), -math.inf, device=DEVICE, dtype=torch.float64)
    at = 0
    for r, (c, m) in enumerate(zip(cached, new)):
        ctx = c + (m if causal else 0)
        pages = table[r, : -(-ctx // page)]
        for h in range(kv_heads if ctx else 0):
            k = kc[pages, h].reshape(-1, d)[:ctx].double()
            v = vc[pages, h].reshape(-1, d)[:ctx].double()
            step = max(1, (1 << 27) // (ctx * g))                            # at most a gigabyte of scores at a time
            for t0 in range(0, m, step):
                t1 = min(m, t0 + step)
                q = s["q"][at + t0 : at + t1, h * g : (h + 1) * g].double().reshape(-1, d)
                sc = (q @ k.t().contiguous()) / math.sqrt(d)
                if causal:
                    last = (c + torch.arange(t0, t1, device=DEVICE)).repeat_interleave(g)
                    sc.masked_fill_(torch.arange(ctx, device=DEVICE)[None, :] > last[:, None], -math.inf)
                top = torch.logsumexp(sc, dim=1)
                lse[at + t0 : at + t1, h * g : (h + 1) * g] = top.reshape(-1, g)
                out[at + t0 : at + t1, h * g : (h + 1) * g] = (torch.exp(sc - top[:, None]) @ v).reshape(-1, g, d)
        at += m
    return {"out": out, "lse": lse, "k_cache": kc, "v_cache": vc} if causal else {"out": out, "lse": lse}
