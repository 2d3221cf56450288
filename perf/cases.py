"""The work this library is measured on: decode attention over a paged, prefix-aliased KV cache, and what goes with it.

A case is one call - or the calls of one decode step - that a serving program makes through the public entry points,
with everything such a program already holds (caches, tables, lengths, workspace, plan) prepared before.  Lengths and
the sharing structure follow from the case alone; tokens, q, K, V and the scatter of the blocks over the pool follow
from the seed.  Host bookkeeping (block tables, scheduler) runs once per request of thousands of decode steps and is
not timed here.
"""
import math
import random

import numpy as np
import torch

import paper_2605_06046_amd as fea

BLOCK = 16


def _attention(name, dtype, heads, head_dim, groups, per_group, prefix, suffix, system=0, worn=False, peak=1.0,
               layers=1, plan="new", lens=1):
    """groups x per_group requests in arrival order; all share `system` leading tokens, a group shares `prefix` more,
    a request adds suffix[0]..suffix[1] of its own.  worn: blocks scattered over a pool 1.5 times as large (a pool that
    has been in use), else handed out in order.  peak: gain on q (how concentrated the softmax is).  layers: layers of
    the step that append their new rows and attend; plan: made at the first layer ("new") or an earlier step's plan
    stretched ("refresh"); the other layers use it again."""
    c = dict(kind="attention", dtype=dtype, q_heads=heads[0], kv_heads=heads[1], head_dim=head_dim, groups=groups,
             per_group=per_group, system=system, prefix=prefix, suffix_lo=suffix[0], suffix_hi=suffix[1], worn=worn,
             peak=peak, layers=layers, plan=plan, lens=lens)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a handful of short float32 requests (the parity shape); launches and latency count.
        _attention("f32_tiny", "f32", (8, 2), 64, 1, 4, 256, (64, 64)),
        # A few short chats with nothing in common, seven query heads to a KV head, ragged lengths.
        _attention("short_chats", "bf16", (28, 4), 128, 8, 1, 0, (90, 700), worn=True, peak=2.0),
        # One homogeneous batch on a Llama-3-8B-shaped layer: the shape the benchmark quotes.
        _attention("homogeneous", "bf16", (32, 8), 128, 1, 64, 4096, (128, 1024)),
        # Eight prefix groups mixed into one batch in arrival order.
        _attention("mixed_groups", "bf16", (32, 8), 128, 8, 32, 4096, (128, 1024)),
        # Questions about one long document, blocks scattered over a pool that has been in use.
        _attention("long_document", "bf16", (32, 8), 128, 1, 32, 32768, (512, 512), worn=True),
        # The largest: first come first served, nothing shared, eight query heads to a KV head.
        _attention("unshared", "bf16", (64, 8), 128, 512, 1, 0, (512, 4096)),
        # float32 caches beyond the toy size (numerical work on a real layer's shape).
        _attention("f32_layer", "f32", (32, 8), 128, 1, 16, 1024, (128, 1024), peak=2.0),
        # Head dim 64, prefix groups mixed.
        _attention("head64_groups", "bf16", (32, 8), 64, 8, 16, 2040, (64, 777), worn=True, peak=2.0),
        # Head dim 256, one homogeneous batch.
        _attention("head256_prefix", "bf16", (16, 4), 256, 1, 48, 3000, (100, 900), peak=2.0),
        # Four layers of one decode step: append, attend, one plan made for the step; conversations on a common
        # system prompt (nested prefixes), five query heads to a KV head.
        _attention("step_nested", "bf16", (40, 8), 128, 6, 8, 1000, (33, 500), system=1024, worn=True, peak=2.0, layers=4),
        # The same between plans: the plan of some steps ago stretched to the lengths of now.
        _attention("step_refreshed", "bf16", (32, 8), 128, 4, 8, 2048, (60, 900), worn=True, peak=2.0, layers=4, plan="refresh"),
        # Prefix hashes of an arriving batch on the device.
        dict(name="hash_arrivals", kind="hash", requests=64, tokens_lo=4224, tokens_hi=5120, lens=1),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.1:
        hi = _loguniform(rng, 16, 8000)
        n = _loguniform(rng, 1, 512)
        return dict(kind="hash", requests=n, tokens_lo=rng.randint(1, hi), tokens_hi=hi, lens=rng.randrange(1 << 30))
    while True:
        dtype = "bf16" if rng.random() < 0.8 else "f32"
        heads = rng.choice([(32, 8), (32, 8), (28, 4), (40, 8), (64, 8), (8, 2), (8, 8), (16, 4), (12, 4), (32, 2)])
        d = rng.choice([128, 128, 64, 256])
        B = _loguniform(rng, 1, 512)
        shape = rng.random()
        if shape < 0.3:                       # nothing shared
            groups, per, prefix, system = B, 1, 0, 0
        else:
            groups = min(B, _loguniform(rng, 1, 16))
            per = max(1, B // groups)
            prefix = _loguniform(rng, 32, 16384)
            system = _loguniform(rng, 32, 2048) if shape > 0.8 else 0
        lo = _loguniform(rng, 20, 1000)
        hi = lo + _loguniform(rng, 1, 4000)
        layers = rng.choice([1, 1, 1, 2, 3, 4])
        c = _attention(None, dtype, heads, d, groups, per, prefix, (lo, hi), system=system, worn=rng.random() < 0.6,
                       peak=rng.choice([1.0, 2.0, 3.0]), layers=layers,
                       plan="refresh" if layers > 1 and rng.random() < 0.5 else "new", lens=rng.randrange(1 << 30))
        w = work(c)
        _, _, unique, logical = _structure(c)
        # no dearer than the largest listed case: its bytes and operations, and a vector unit's time for float32
        vector_us = logical * heads[0] * (d / 64.0) ** 1.6 * 3e-5 * layers if dtype == "f32" else 0.0
        if w["bytes"] < 3.5e9 and w["flops"] < 3.5e10 and vector_us < 500:
            return c


def _structure(c):
    """Request lengths, each request's group (in arrival order), tokens stored once, tokens attended to."""
    rng = random.Random(c["lens"])
    B = c["groups"] * c["per_group"]
    group = [g for g in range(c["groups"]) for _ in range(c["per_group"])]
    if c["groups"] > 1:
        rng.shuffle(group)
    own = [rng.randint(c["suffix_lo"], c["suffix_hi"]) for _ in range(B)]
    shared = c["system"] + c["prefix"] if c["per_group"] > 1 or c["system"] else c["prefix"]
    lens = [shared + s for s in own]
    sys_t, grp_t = _shared_blocks(c)
    sys_t, grp_t = sys_t * BLOCK, grp_t * BLOCK
    unique = sys_t + c["groups"] * grp_t + sum(L - sys_t - grp_t for L in lens)
    return lens, group, unique, sum(lens)


def _shared_blocks(c):
    """Full blocks everybody shares, and full blocks a group shares after those."""
    sysb = c["system"] // BLOCK
    return sysb, (c["system"] + c["prefix"]) // BLOCK - sysb


def _tables(c, np_rng):
    """Block tables as the pool hands them out: requests in order, columns left to right, shared blocks once."""
    lens, group, _, _ = _structure(c)
    sysb, grpb = _shared_blocks(c)
    total = sysb + c["groups"] * grpb + sum(-(-L // BLOCK) - sysb - grpb for L in lens)
    nblocks = total * 3 // 2 if c["worn"] else total
    ids = (np_rng.permutation(nblocks) if c["worn"] else np.arange(nblocks)).astype(np.int32)
    width = max(-(-L // BLOCK) for L in lens) + 4          # room for the next steps
    bt = np.full((len(lens), width), -1, dtype=np.int32)
    at, common, of_group = 0, None, {}

    def take(n):
        nonlocal at
        at += n
        return ids[at - n:at]

    for i, (L, g) in enumerate(zip(lens, group)):
        if common is None:
            common = take(sysb)
        if g not in of_group:
            of_group[g] = take(grpb)
        nb = -(-L // BLOCK)
        bt[i, :sysb] = common
        bt[i, sysb:sysb + grpb] = of_group[g]
        bt[i, sysb + grpb:nb] = take(nb - sysb - grpb)
    return bt, np.array(lens, dtype=np.int32), nblocks


def _hash_lens(c):
    rng = random.Random(c["lens"])
    return [rng.randint(c["tokens_lo"], c["tokens_hi"]) for _ in range(c["requests"])]


AGE = 16   # steps since the plan that a "refresh" step stretches was made


def prepare(case, seed):
    np_rng = np.random.default_rng([seed & 0x7FFFFFFF, 7])
    if case["kind"] == "hash":
        lens = np.array(_hash_lens(case), dtype=np.int64)
        tok_off = np.concatenate([[0], np.cumsum(lens)])
        hash_off = np.concatenate([[0], np.cumsum(-(-lens // BLOCK))])
        tokens = np_rng.integers(0, 32000, size=int(tok_off[-1]), dtype=np.int32)
        return dict(case=case, tokens=torch.from_numpy(tokens).cuda(), tok_off=torch.from_numpy(tok_off).cuda(),
                    hash_off=torch.from_numpy(hash_off).cuda(),
                    hashes=torch.zeros(int(hash_off[-1]), dtype=torch.int64, device="cuda"))
    bt, lens, nblocks = _tables(case, np_rng)
    B, layers = len(lens), case["layers"]
    Hq, Hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=dt)

    s = dict(case=case, bt=torch.from_numpy(bt).cuda(), lens=torch.from_numpy(lens).cuda(),
             q=[normal(B, Hq, d) * case["peak"] for _ in range(layers)],
             k=[normal(nblocks, Hkv, BLOCK, d) for _ in range(layers)],
             v=[normal(nblocks, Hkv, BLOCK, d) for _ in range(layers)],
             out=[torch.empty(B, Hq, d, device="cuda", dtype=dt) for _ in range(layers)])
    if layers > 1:
        s["k_new"] = [normal(B, Hkv, d) for _ in range(layers)]
        s["v_new"] = [normal(B, Hkv, d) for _ in range(layers)]
    code = fea.FEA_DTYPE_F32 if case["dtype"] == "f32" else fea.FEA_DTYPE_BF16
    s["first"] = fea.AttnParams(Hq, Hkv, d, code, flags=fea.FEA_FLAG_REFRESH_PLAN if case["plan"] == "refresh" else 0)
    s["other"] = fea.AttnParams(Hq, Hkv, d, code, flags=fea.FEA_FLAG_REUSE_PLAN)
    s["ws"] = torch.empty(fea.fea_decode_workspace_bytes(s["first"], B, bt.shape[1]), dtype=torch.uint8, device="cuda")
    if case["plan"] == "refresh":          # what an earlier step left in the workspace
        made = fea.AttnParams(Hq, Hkv, d, code, flags=fea.FEA_FLAG_PLAN_ONLY)
        fea.fea_decode_attention(made, s["q"][0], s["k"][0], s["v"][0], s["bt"], s["lens"] - AGE, s["out"][0], s["ws"])
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "hash":
        fea.fea_chunk_hashes_device(state["tokens"], state["tok_off"], state["hash_off"], state["hashes"])
        return state["hashes"]
    bt, lens, ws = state["bt"], state["lens"], state["ws"]
    if case["layers"] == 1:
        fea.fea_decode_attention(state["first"], state["q"][0], state["k"][0], state["v"][0], bt, lens, state["out"][0], ws)
        return state["out"][0]
    for x in range(case["layers"]):
        fea.fea_kv_append(state["first"], state["k_new"][x], state["v_new"][x], state["k"][x], state["v"][x], bt, lens)
        fea.fea_decode_attention(state["first"] if x == 0 else state["other"], state["q"][x], state["k"][x], state["v"][x],
                                 bt, lens, state["out"][x], ws)
    return dict(out=state["out"], k=state["k"], v=state["v"])


def work(case):
    if case["kind"] == "hash":
        lens = _hash_lens(case)
        # every token is read once, every 16th position's hash written; integer work: about 8 operations per token
        return {"bytes": 4 * sum(lens) + 8 * sum(-(-n // BLOCK) for n in lens), "flops": 0}
    lens, _, unique, logical = _structure(case)
    es = 4 if case["dtype"] == "f32" else 2
    B, Hq, Hkv, d = len(lens), case["q_heads"], case["kv_heads"], case["head_dim"]
    per_layer = unique * 2 * Hkv * d * es + 2 * B * Hq * d * es
    if case["layers"] > 1:
        per_layer += 2 * 2 * B * Hkv * d * es       # the new rows: read, and written into the caches
    tables = 4 * sum(-(-L // BLOCK) for L in lens) + 4 * B
    return {"bytes": case["layers"] * per_layer + tables, "flops": case["layers"] * 4 * Hq * d * logical}


def tolerance(case):
    if case["kind"] == "hash":
        return "exact"
    # float32: sums of products of up to some thousand terms in another order.  bfloat16: one rounding of the result
    # (2^-9), and the softmax weights rounded to 16 bits for the second product.
    return {"rel": 2e-6, "max": 4e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.1}


def exact(case, seed):
    """The definition in float64 (hashes: in 64-bit integers), request by request."""
    s = prepare(case, seed)
    if case["kind"] == "hash":
        return torch.from_numpy(_hashes(s["tokens"].cpu().numpy(), np.array(_hash_lens(case))))
    bt, lens = s["bt"].long(), s["lens"].tolist()
    Hq, Hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    outs = []
    for x in range(case["layers"]):
        k, v = s["k"][x], s["v"][x]
        if case["layers"] > 1:
            pos = s["lens"].long() - 1
            blk = bt.gather(1, (pos // BLOCK)[:, None])[:, 0]
            k[blk, :, pos % BLOCK] = s["k_new"][x]
            v[blk, :, pos % BLOCK] = s["v_new"][x]
        out = torch.empty(len(lens), Hq, d, device=k.device, dtype=torch.float64)
        for i, L in enumerate(lens):
            rows = bt[i, :-(-L // BLOCK)]
            ki = k[rows].transpose(0, 1).reshape(Hkv, -1, d)[:, :L].double()
            vi = v[rows].transpose(0, 1).reshape(Hkv, -1, d)[:, :L].double()
            qi = s["q"][x][i].double().view(Hkv, Hq // Hkv, d)
            p = torch.softmax(qi @ ki.transpose(1, 2).contiguous() / math.sqrt(d), dim=-1)
            out[i] = (p @ vi).view(Hq, d)
        outs.append(out)
    if case["layers"] == 1:
        return outs[0]
    return dict(out=outs, k=[t.double() for t in s["k"]], v=[t.double() for t in s["v"]])


def _mix(x):
    x = x ^ (x >> np.uint64(30))
    x = x * np.uint64(0xBF58476D1CE4E5B9)
    x = x ^ (x >> np.uint64(27))
    x = x * np.uint64(0x94D049BB133111EB)
    return x ^ (x >> np.uint64(31))


def _hashes(tokens, lens):
    """The documented chunk-parallel prefix hash: leaves of 16 tokens, chained."""
    gamma = np.uint64(0x9E3779B97F4A7C15)
    n, first = len(lens), np.concatenate([[0], np.cumsum(lens)])[:-1]
    chunks = -(-lens // BLOCK)
    out_at = np.concatenate([[0], np.cumsum(chunks)])
    out = np.zeros(int(out_at[-1]), dtype=np.uint64)
    h = np.full(n, 0x243F6A8885A308D3, dtype=np.uint64)
    tok = tokens.astype(np.uint32).astype(np.uint64)
    for c in range(int(chunks.max())):
        on = np.nonzero(chunks > c)[0]
        size = np.minimum(lens[on] - c * BLOCK, BLOCK)
        a = _mix(gamma ^ size.astype(np.uint64))
        for j in range(BLOCK):
            has = size > j
            a[has] = _mix(a[has] ^ tok[first[on][has] + c * BLOCK + j])
        h[on] = _mix(_mix(h[on] + gamma) ^ a)
        out[out_at[:-1][on] + c] = h[on]
    return out.view(np.int64)
