"""The calls whose speed is kept: what a trainer and its rollout workers do
with this library at every policy step, from one matrix to a whole model.

A trainer compares the weights before and after the step (extract, to
indices or straight to coded indices, or chunk by chunk into host memory)
and packs the versioned artifact; a worker verifies and activates an
artifact, applies an index stream, or catches up over several missed steps
(in one pass, or by composing the chain for a relay).

Weight lists are the Qwen3 shapes of ``synth``, or lists of odd-sized
tensors packed back to back (``ragged``, a flat parameter shard) or at
256-byte boundaries.  Densities lie between 0.1% and 10% of the words, about
1% in a real step, spread evenly or with 80% of the changes in 5% of the
4096-word rows (``clustered``).

Every output is a position, a count, a byte or a 16-bit word that is moved
and never computed with, so outputs are compared exactly; bf16 words are
returned as their bit patterns.
"""
import math
import random

import torch

import paper_2602_11456_amd as ad
from paper_2602_11456_amd import synth

ROW = 4096                   # words of a row of the clustered change pattern
HOT, HOT_SHARE = 0.05, 0.8   # share of the rows that are hot, share of the changes there
CHUNK = 1 << 28              # words generated at a time


def listed():
    return [
        # one projection matrix, the smallest call: launches and latency
        dict(name="extract_matrix", op="extract_one", words=2048 * 2048, density=0.01,
             index="int32"),
        # a rank's flat shard of odd-sized tensors, extracted every step
        dict(name="extract_shard", op="extract", words=103_456_789, tensors=37, layout=5,
             ragged=True, density=0.01),
        # the whole model at the density a reinforcement learning step has
        dict(name="extract_8b", op="extract", model="qwen3-8b", density=0.01),
        # a large step: every output word counts
        dict(name="extract_4b_dense", op="extract", model="qwen3-4b", density=0.1),
        # the sender's one call: coded indices and words
        dict(name="extract_coded_4b", op="extract_coded", model="qwen3-4b", density=0.01),
        # the same streamed into pinned host memory, 256 MB chunks
        dict(name="pipeline_4b", op="pipeline", model="qwen3-4b", density=0.01, coded=True,
             chunk=1 << 27),
        # the versioned, hashed artifact from an extract's output
        dict(name="pack_4b", op="pack", model="qwen3-4b", density=0.01, clustered=True,
             coding="leb128"),
        # a worker: verify the artifact and apply it
        dict(name="activate_4b", op="activate", model="qwen3-4b", density=0.01,
             coding="leb128"),
        # a worker on the same node: the index stream itself
        dict(name="apply_8b", op="apply", model="qwen3-8b", density=0.01, sorted=False),
        # a dense delta, known to be sorted
        dict(name="apply_4b_dense", op="apply", model="qwen3-4b", density=0.1, sorted=True),
        # a worker four steps behind
        dict(name="catch_up_4b", op="catch_up", model="qwen3-4b", density=0.01, chain=4),
        # a relay that forwards one delta for four steps
        dict(name="compose_4b", op="compose", model="qwen3-4b", density=0.01, chain=4),
    ]


def draw(rng):
    op = rng.choice(["extract_one", "extract", "extract_coded", "pipeline", "pack", "activate",
                     "apply", "catch_up", "compose"])
    most = {"extract_one": 1 << 27, "pipeline": 1 << 30}.get(op, 4_000_000_000)
    words = int(math.exp(rng.uniform(math.log(1 << 17), math.log(most))))
    density = round(math.exp(rng.uniform(math.log(0.001), math.log(0.1))), 5)
    c = dict(op=op, words=words, density=density)
    if op == "extract_one":
        c["index"] = rng.choice(["int32", "int64"])
        return c
    c.update(tensors=rng.randint(1, 64), layout=rng.randrange(1 << 20),
             ragged=rng.random() < 0.5, clustered=rng.random() < 0.3)
    if op == "pipeline":
        c.update(coded=rng.random() < 0.5, chunk=1 << rng.randint(25, 27),
                 density=min(density, 0.02))
    elif op in ("pack", "activate"):
        c["coding"] = rng.choice(["int64", "leb128"])
    elif op == "apply":
        c["sorted"] = rng.random() < 0.5
    elif op in ("catch_up", "compose"):
        c["chain"] = rng.randint(2, 12)
    # no more entries in a call than the largest of the whole-model calls has
    entries = {"catch_up": 160e6, "compose": 160e6}.get(op, 400e6)
    c["density"] = round(min(c["density"], entries / c.get("chain", 1) / words), 6)
    return c


# ------------------------------------------------------------------ inputs

def sizes(case):
    """Words of every tensor of the list."""
    if "model" in case:
        return [synth.numel(s) for _, s in synth.qwen3_tensor_table(case["model"])]
    if case["op"] == "extract_one":
        return [case["words"]]
    rng = random.Random(case["layout"])
    cuts = sorted(rng.randrange(case["words"] + 1) for _ in range(case["tensors"] - 1))
    edges = [0] + cuts + [case["words"]]
    return [b - a for a, b in zip(edges, edges[1:])]


def starts(case, nums):
    """First word of every tensor in its flat buffer, and the buffer's size."""
    step = 1 if case.get("ragged") else 128
    at, out = 0, []
    for n in nums:
        out.append(at)
        at += -(-n // step) * step
    return out, at


def views(flat, nums, at):
    return [flat[a:a + n] for n, a in zip(nums, at)]


def chances(case, lo, n, g):
    """Probability of a change of each of the words [lo, lo + n): one number,
    or, clustered, one per row (whole rows: lo is a multiple of ROW)."""
    d = case["density"]
    if not case.get("clustered"):
        return d
    rows = -(-n // ROW)
    hot = torch.rand(rows, generator=g, device="cuda") < HOT
    return torch.where(hot, min(0.9, d * HOT_SHARE / HOT), d * (1 - HOT_SHARE) / (1 - HOT))


def changed(case, n, g, lo):
    p = chances(case, lo, n, g)
    r = torch.rand(n, generator=g, device="cuda")
    if not torch.is_tensor(p):
        return r < p
    return r < p.repeat_interleave(ROW)[:n]


def step_pair(case, total, seed, new=True):
    """Flat words before a step, and after it (a changed word is the bf16 of
    the old one plus N(0, 1e-3), or its neighbour where that is the same)."""
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 17)
    prev = torch.empty(total, dtype=torch.bfloat16, device="cuda")
    nxt = torch.empty_like(prev) if new else None
    for lo in range(0, total, CHUNK):
        n = min(CHUNK, total - lo)
        x = torch.randn(n, generator=g, device="cuda").mul_(0.02)
        old = x.to(torch.bfloat16)
        prev[lo:lo + n] = old
        if not new:
            continue
        x.add_(torch.randn(n, generator=g, device="cuda"), alpha=1e-3)
        bits, ob = x.to(torch.bfloat16).view(torch.int16), old.view(torch.int16)
        bits = torch.where(bits == ob, ob ^ 1, bits)
        nxt[lo:lo + n] = torch.where(changed(case, n, g, lo), bits, ob).view(torch.bfloat16)
    return prev, nxt


def delta_of(case, nums, seed, density):
    """One step's delta over the tensor list: sorted global indices and new
    words.  The gaps between a tensor's entries are drawn for the case and put
    in another order by the seed (64 neighbours at a time, which keeps rows of
    many changes together), so that every seed's delta has the same number of
    entries and of code bytes.  No tensor's word 0 changes."""
    fixed = torch.Generator(device="cuda").manual_seed(len(nums) + 101 * int(1e6 * density))
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 29)
    total = sum(nums)
    base = torch.tensor([0] + nums, device="cuda").cumsum(0)
    idx = []
    for lo in range(0, total, CHUNK):
        n = min(CHUNK, total - lo)
        idx.append(changed(dict(case, density=density), n, fixed, lo).nonzero().view(-1).add_(lo))
    idx = torch.cat(idx)
    t = torch.searchsorted(base, idx, right=True) - 1    # tensor of every entry
    idx, t = idx[idx != base[t]], t[idx != base[t]]
    if idx.numel() == 0:
        return idx, torch.empty(0, dtype=torch.bfloat16, device="cuda")
    gap = idx.diff(prepend=idx[:1])
    first = t.diff(prepend=t[:1] - 1) != 0
    gap = torch.where(first, idx - base[t], gap)
    block = torch.arange(idx.numel(), device="cuda") // 64 + t
    key = torch.rand(int(block[-1]) + 1, generator=g, device="cuda", dtype=torch.float64)
    gap = gap[torch.sort(key[block] + t, stable=True).indices]
    run = gap.cumsum(0)
    before = (run - gap)[first]                          # of each nonempty tensor's first entry
    idx = run - before[first.cumsum(0) - 1] + base[t]
    val = torch.randn(idx.numel(), generator=g, device="cuda").mul_(0.02)
    return idx, val.to(torch.bfloat16)


def chain_of(case, nums, seed):
    """The deltas of `chain` consecutive steps, each of the case's density, as
    parts of the delta that holds every index of them: an entry is in step j
    first, and in every later step with the density's probability."""
    d, k = case["density"], case["chain"]
    idx, _ = delta_of(case, nums, seed, 1 - (1 - d) ** k)
    fixed = torch.Generator(device="cuda").manual_seed(k)
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 43)
    u = torch.rand(idx.numel(), generator=fixed, device="cuda", dtype=torch.float64)
    first = (torch.log1p(-u * (1 - (1 - d) ** k)) / math.log1p(-d)).long().clamp_(0, k - 1)
    shift = random.Random(seed).randrange(idx.numel() + 1)
    out = []
    for j in range(k):
        again = torch.rand(idx.numel(), generator=fixed, device="cuda") < d
        sel = idx[torch.roll((first == j) | ((first < j) & again), shift)]
        val = torch.randn(sel.numel(), generator=g, device="cuda").mul_(0.02)
        out.append((sel, val.to(torch.bfloat16)))
    return out


def offsets_of(idx, nums):
    """First entry of every tensor in the delta, and the total."""
    ends = torch.tensor([0] + nums, device="cuda").cumsum(0)
    return torch.searchsorted(idx, ends)


def room(case, total):
    """Capacity of preallocated outputs: the expected entries and a margin."""
    return min(total, int(total * case["density"] * 1.25) + 8192)


_streams = []


def streams():
    """The program's pipeline streams, made once."""
    while len(_streams) < 4:
        _streams.append(torch.cuda.Stream())
    return list(_streams)


def prepare(case, seed):
    op, nums = case["op"], sizes(case)
    total = sum(nums)
    at, flat = starts(case, nums)
    zeros = lambda n, t=torch.int64: torch.zeros(n, dtype=t, device="cuda")  # noqa: E731
    s = dict(op=op, case=case, nums=nums)
    if op in ("extract_one", "extract", "extract_coded", "pipeline"):
        prev, new = step_pair(case, flat, seed)
        cap = room(case, total)
        if op == "extract_one":
            s.update(prev=prev, new=new, idx=zeros(cap, getattr(torch, case["index"])),
                     val=zeros(cap, torch.int16), count=zeros(1),
                     ws=zeros(ad.delta_extract_workspace_bytes(total), torch.uint8))
            return s
        plan = ad.MultiPlan(views(prev, nums, at), views(new, nums, at)).prepare()
        s["plan"] = plan
        if op == "pipeline":
            need = (ad.delta_pipeline_leb128_staging_bytes if case["coded"]
                    else ad.delta_pipeline_staging_bytes)(nums, case["chunk"], 4)
            s.update(staging=zeros(need, torch.uint8), streams=streams(),
                     h_val=torch.zeros(cap, dtype=torch.int16, pin_memory=True))
            if case["coded"]:
                s["h_code"] = torch.zeros(3 * cap, dtype=torch.uint8, pin_memory=True)
            else:
                s["h_idx"] = torch.zeros(cap, dtype=torch.int64, pin_memory=True)
            return s
        s.update(val=zeros(cap, torch.int16), count=zeros(1), offs=zeros(len(nums) + 1))
        if op == "extract":
            s.update(idx=zeros(cap), ws=zeros(plan.workspace_bytes, torch.uint8))
        else:
            s.update(code=zeros(3 * cap, torch.uint8), nbytes=zeros(1),
                     byte_offs=zeros(len(nums) + 1),
                     ws=zeros(ad.delta_extract_multi_leb128_workspace_bytes(nums), torch.uint8))
        return s
    if op in ("compose", "catch_up"):
        s["deltas"] = chain_of(case, nums, seed)
    else:
        s["idx"], s["val"] = delta_of(case, nums, seed, case["density"])
    if op in ("apply", "activate", "catch_up"):
        s["flat"], _ = step_pair(case, flat, seed, new=False)
        s["weights"] = views(s["flat"], nums, at)
    if op == "apply":
        need = (ad.delta_apply_multi_sorted_workspace_bytes if case["sorted"]
                else ad.delta_apply_multi_workspace_bytes)(len(nums))
        s.update(flag=zeros(1, torch.int32), ws=zeros(max(need, 1), torch.uint8))
    if op in ("pack", "activate"):
        s["offs"] = offsets_of(s["idx"], nums)
    if op == "activate":
        s["art"], _ = ad.pack_artifact(s.pop("idx"), s.pop("val"), s["offs"], nums, 8, 7,
                                       coding=case["coding"])
    return s


# -------------------------------------------------------------------- call

def run(s):
    op = s["op"]
    if op == "extract_one":
        ad.delta_extract_into(s["prev"], s["new"], s["idx"], s["val"], s["count"], s["ws"])
        return [s["idx"], s["val"], s["count"]]
    if op == "extract":
        ad.delta_extract_multi_into(s["plan"], s["idx"], s["val"], s["count"], s["ws"], s["offs"])
        return [s["idx"], s["val"], s["count"], s["offs"]]
    if op == "extract_coded":
        ad.delta_extract_multi_leb128_into(s["plan"], s["code"], s["val"], s["count"],
                                           s["nbytes"], s["ws"], s["offs"], s["byte_offs"])
        return [s["code"], s["val"], s["count"], s["nbytes"], s["offs"], s["byte_offs"]]
    if op == "pipeline" and s["case"]["coded"]:
        code, val, counts, chunk = ad.delta_extract_pipelined_leb128_plan(
            s["plan"], s["case"]["chunk"], 4, s["h_code"], s["h_val"], s["staging"], s["streams"])
        return [s["h_code"], s["h_val"], torch.tensor(counts), code.numel(), val.numel(), chunk]
    if op == "pipeline":
        idx, val = ad.delta_extract_pipelined_plan(
            s["plan"], s["case"]["chunk"], 4, s["h_idx"], s["h_val"], s["staging"], s["streams"])
        return [s["h_idx"], s["h_val"], idx.numel(), val.numel()]
    if op == "pack":
        art, _ = ad.pack_artifact(s["idx"], s["val"], s["offs"], s["nums"], 8, 7,
                                  coding=s["case"]["coding"])
        return art
    if op == "activate":
        version = ad.activate_artifact(s["art"], s["weights"], 7)
        return [s["flat"].view(torch.int16), version]
    if op == "apply":
        ad.delta_apply_multi(s["weights"], s["idx"], s["val"], error_flag=s["flag"],
                             workspace=s["ws"], sorted_indices=s["case"]["sorted"])
        return [s["flat"].view(torch.int16), s["flag"]]
    if op == "catch_up":
        ad.delta_catch_up(s["weights"], s["deltas"])
        return s["flat"].view(torch.int16)
    idx, val = ad.delta_compose(s["deltas"])
    return [idx, val.view(torch.int16)]


def work(case):
    n = sum(sizes(case))
    d = case["density"]
    k = n * d
    # bytes of an even delta's gap code: a gap g has probability d (1 - d)^(g - 1)
    code = k * (1 + (1 - d) ** 127 + (1 - d) ** 16383)
    op = case["op"]
    if op == "extract_one":
        b = 4 * n + k * ((4 if case["index"] == "int32" else 8) + 2)
    elif op == "extract" or (op == "pipeline" and not case["coded"]):
        b = 4 * n + 10 * k
    elif op in ("extract_coded", "pipeline"):
        b = 4 * n + code + 2 * k
    elif op == "pack":
        b = 10 * k + (code if case["coding"] == "leb128" else 8 * k) + 2 * k
    elif op == "activate":
        b = (code if case["coding"] == "leb128" else 8 * k) + 4 * k
    elif op == "apply":
        b = 12 * k
    else:   # a chain: every entry read, every distinct index written once
        distinct = n * (1 - (1 - d) ** case["chain"])
        b = 10 * k * case["chain"] + (2 if op == "catch_up" else 10) * distinct
    return {"bytes": float(b), "flops": 0.0}


def tolerance(case):
    return "exact"
