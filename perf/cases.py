"""The work whose time matters to a user of librollattn, as callable cases.

Every case is one engine step (or the part of one) of a multi-turn rollout over a paged KV cache, taken through
the public entry points of `paper_2512_22560_amd.binding` with the buffers an engine keeps (pools, tables, output,
workspace) made beforehand.  Lengths belong to the case (drawn from its `lengths` seed with the recipe of
`workloads.py`), values and the physical placement of the pages to the seed that `prepare` is given.  Head shapes,
length distributions and batch sizes are those of the workloads the repository states, and smaller ones of the
same kind: a rollout starts with hundreds of trajectories in step and ends with a handful of long ones, and
environments answer one by one.

Kinds of case:
  decode    attn_decode: one token per trajectory over its whole context
  token     kv_write of one token per trajectory, then attn_decode: what an engine does per generated token
  append    attn_append: a chunk per trajectory behind its cached prefix (prefix 0: recomputation)
  turn      kv_write of the chunks, then attn_append: an observation arrives
  step      attn_step: a mixed batch, `chunks` of its trajectories with a chunk and the others with one token
  shared    attn_decode_shared: groups that share their prompt's pages
  kv_write  kv_write alone: the chunks of a step go into the cache
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_2512_22560_amd import binding as B
from paper_2512_22560_amd import workloads as W

PAGE = W.PAGE_SIZE
ITEM = {"f32": 4, "bf16": 2, "fp8_e4m3": 1}
GROUP = W.SHARED_PROMPT_GROUP


def _case(kind, batch, heads, q, kv, ctx, new=(1, 1), chunks=0, prompt=0, lengths=0, name=None):
    """ctx: (kind, *numbers) as in workloads.Workload; new: least and most new tokens of a chunk."""
    c = {"kind": kind, "batch": batch, "q_heads": heads[0], "kv_heads": heads[1], "head_dim": heads[2], "q": q, "kv": kv,
         "ctx": ctx[0], "new_lo": new[0], "new_hi": new[1], "chunks": chunks, "prompt": prompt, "lengths": lengths}
    c.update({"ctx%d" % i: v for i, v in enumerate(ctx[1:])})
    return c if name is None else dict(c, name=name)


def listed():
    c1, c2, c3, c4, c5 = (W.CONFIGS[i] for i in range(1, 6))
    rc, sp = W.RECOMPUTE, W.SHARED_PROMPT

    def heads(w):
        return w.num_q_heads, w.num_kv_heads, w.head_dim

    return [
        # the smallest call: four short float32 contexts, nothing but launches and latency
        _case("decode", c1.batch, heads(c1), "f32", "f32", c1.ctx, lengths=c1.seed, name="decode_f32_tiny"),
        # the tail of a rollout: the last few long trajectories still generate, one token at a time
        _case("token", 5, heads(c2), "bf16", "bf16", ("loguniform", 2048, 32768), lengths=11, name="token_bf16_few"),
        # an ordinary decode step
        _case("decode", c2.batch, heads(c2), "bf16", "bf16", c2.ctx, lengths=c2.seed, name="decode_bf16_b64"),
        # a large decode step with long-tailed histories
        _case("decode", c3.batch, heads(c3), "bf16", "bf16", c3.ctx, lengths=c3.seed, name="decode_bf16_b256_longtail"),
        # the same over an FP8 cache: the generating part of the mixed batch
        _case("decode", 384, heads(c5), "bf16", "fp8_e4m3", c5.ctx, lengths=12, name="decode_fp8_b384"),
        # environments answer one by one: three observations at a time, written and prefilled
        _case("turn", 3, heads(c4), "bf16", "bf16", c4.ctx, new=(16, 512), lengths=13, name="turn_bf16_few"),
        # terse observations of a medium batch over an FP8 cache
        _case("turn", 33, heads(c5), "bf16", "fp8_e4m3", c5.ctx, new=(3, 96), lengths=14, name="turn_fp8_short"),
        # observations of a whole batch behind long prefixes
        _case("append", c4.batch, heads(c4), "bf16", "bf16", c4.ctx, new=c4.qlen[1:], lengths=c4.seed, name="append_bf16_b64"),
        # after a weight update every history is prefilled again
        _case("append", rc.batch, heads(rc), "bf16", "bf16", ("const", 0), new=rc.qlen[1:], lengths=rc.seed, name="recompute_bf16_b64"),
        # one engine step of a full batch, a quarter of it with observations, FP8 cache: the largest
        _case("step", c5.batch, heads(c5), "bf16", "fp8_e4m3", c5.ctx, new=c5.qlen[1:], chunks=c5.append_rows, lengths=c5.seed,
              name="step_fp8_b512"),
        # early turns of grouped rollouts: eight trajectories per prompt
        _case("shared", sp.batch, heads(sp), "bf16", "fp8_e4m3", sp.ctx, prompt=W.SHARED_PROMPT_TOKENS, lengths=sp.seed,
              name="shared_fp8_b512"),
        # the new rows of a step's observations are quantised into the cache
        _case("kv_write", 128, heads(c5), "bf16", "fp8_e4m3", c5.ctx, new=c5.qlen[1:], lengths=15, name="kv_write_fp8_b128"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges; none has more bytes or operations than the largest listed one."""
    most = {"bytes": 8.5e9, "flops": 1.43e13}
    while True:
        kind = rng.choice(["decode", "token", "append", "turn", "step", "shared", "kv_write"])
        if kind == "decode" and rng.random() < 0.25:
            lo = _log_int(rng, 1, 128)
            c = _case("decode", _log_int(rng, 1, 16), (8, 2, 64), "f32", "f32", ("uniform", lo, 2 * lo + rng.randrange(256)))
        else:
            heads = rng.choice([(32, 8, 128), (64, 8, 128), (64, 4, 128)])
            kv = rng.choice(["bf16", "fp8_e4m3"])
            batch = _log_int(rng, 1, 512)
            lo = _log_int(rng, 256, 8192)
            hi = _log_int(rng, lo, 65536)
            ctx = rng.choice([("loguniform", lo, hi), ("uniform", lo, hi), ("lognormal", (lo + hi) // 2, 0.8, lo, hi)])
            new, chunks, prompt = (1, 1), 0, 0
            if kind in ("append", "turn", "step", "kv_write"):
                a, b = sorted((_log_int(rng, 2, 1024), _log_int(rng, 2, 1024)))
                new = (a, b)
                if kind == "append" and rng.random() < 0.25:      # recomputation
                    ctx, new = ("const", 0), (a, 8 * b)
                if kind == "step":
                    batch = max(2, batch)
                    chunks = max(1, int(batch * rng.uniform(0.1, 0.6)))
            if kind == "shared":
                batch = GROUP * max(1, batch // GROUP)
                prompt = PAGE * _log_int(rng, 32, 1024)
                ctx = ("uniform", prompt + 1 + rng.randrange(64), prompt + 64 + _log_int(rng, 16, 2048))
            c = _case(kind, batch, heads, "bf16", kv, ctx, new, chunks, prompt)
        c["lengths"] = rng.randrange(1 << 30)
        w = work(c)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]:
            return c


def _lengths(c):
    """The workload of a case, its context lengths (new tokens included) and new tokens per trajectory."""
    chunky = c["kind"] in ("append", "turn", "step", "kv_write")
    params = [c["ctx%d" % i] for i in range(4) if "ctx%d" % i in c]
    w = W.Workload(c.get("name", c["kind"]), c["batch"], c["q_heads"], c["kv_heads"], c["head_dim"], c["q"], c["kv"],
                   (c["ctx"], *params), qlen=("loguniform" if c["ctx"] == "const" else "uniform", c["new_lo"], c["new_hi"]) if chunky else ("const", 1),
                   append_rows=c["chunks"] or None, ctx_is_prefix=chunky, seed=c["lengths"])
    ctx, new, _, _ = W.draw_structure(w)
    return w, ctx, new


def _page_table(c, ctx):
    """Logical page numbers of every trajectory (groups share their prompt's), -1 where unused, and how many there are."""
    pages = (ctx + PAGE - 1) // PAGE
    table = np.full((len(ctx), max(1, int(pages.max()))), -1, dtype=np.int64)
    head, used = c["prompt"] // PAGE, 0
    for b, n in enumerate(pages.tolist()):
        first = 0
        if head and b % GROUP:
            first = head
            table[b, :head] = table[b - b % GROUP, :head]
        table[b, first:n] = np.arange(used, used + n - first)
        used += n - first
    return table, used


def _fp8_pool(shape, gen, dev):
    """N(0,1) values as E4M3 codes with the scale absmax / 448 of their page."""
    codes = torch.empty(shape, dtype=torch.uint8, device=dev)
    scale = torch.empty(shape[0], dtype=torch.float32, device=dev)
    slab = 32768
    for p in range(0, shape[0], slab):
        x = torch.randn((min(slab, shape[0] - p), *shape[1:]), generator=gen, device=dev)
        s = x.abs().amax(dim=(1, 2, 3)) / 448.0
        scale[p:p + slab] = s
        codes[p:p + slab] = x.div_(s.view(-1, 1, 1, 1)).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes, scale


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    w, ctx, new = _lengths(case)
    table, used = _page_table(case, ctx)
    place = torch.randperm(used, generator=gen, device=dev).to(torch.int32)
    logical = torch.from_numpy(table).to(dev)
    s = {"kind": case["kind"], "max_q": int(new.max()), "scale": w.sm_scale, "k_scale": None, "v_scale": None,
         "table": torch.where(logical >= 0, place[logical.clamp_min(0)], -1).to(torch.int32).contiguous()}

    def ints(x):
        return torch.from_numpy(np.asarray(x).astype(np.int32)).to(dev)

    total = int(new.sum())
    s["ctx"], s["new"], s["off"] = ints(ctx), ints(new), ints(np.concatenate([[0], np.cumsum(new)]))
    dtype = torch.float32 if case["q"] == "f32" else torch.bfloat16

    def rows(n, heads):
        return torch.randn((n, heads, case["head_dim"]), generator=gen, device=dev, dtype=dtype)

    shape = (used, case["kv_heads"], PAGE, case["head_dim"])
    if case["kv"] == "fp8_e4m3":
        s["k"], s["k_scale"] = _fp8_pool(shape, gen, dev)
        s["v"], s["v_scale"] = _fp8_pool(shape, gen, dev)
    else:
        s["k"], s["v"] = (torch.randn(shape, generator=gen, device=dev, dtype=dtype) for _ in range(2))
    if case["kind"] in ("token", "turn", "kv_write"):
        s["k_new"], s["v_new"] = rows(total, case["kv_heads"]), rows(total, case["kv_heads"])
    if case["kind"] == "kv_write":
        return s
    s["q"] = rows(total, case["q_heads"])
    s["out"] = torch.empty_like(s["q"])
    desc = B.make_desc(s["q"], s["k"], s["table"], sm_scale=s["scale"], k_scale=s["k_scale"], v_scale=s["v_scale"])
    if case["kind"] == "shared":
        s["shared"] = torch.full((case["batch"] // GROUP,), case["prompt"], dtype=torch.int32, device=dev)
        n = B.lib().rollattn_shared_workspace_bytes(ctypes.byref(desc), GROUP)
    elif case["kind"] == "step":
        n = B.lib().rollattn_step_workspace_bytes(ctypes.byref(desc), total)
    else:
        n = B.workspace_bytes(desc, total)
    s["ws"] = torch.empty(int(n), dtype=torch.uint8, device=dev)
    return s


def run(s):
    kind = s["kind"]
    pools, where, scales = (s["k"], s["v"]), (s["table"], s["ctx"]), {"k_scale": s["k_scale"], "v_scale": s["v_scale"]}
    if kind in ("token", "turn", "kv_write"):
        B.kv_write(s["k_new"], s["v_new"], s["new"], s["off"], *pools, *where, max_q_len=s["max_q"], **scales)
        if kind == "kv_write":
            return {"k": s["k"], "v": s["v"], **scales}
    kept = {"sm_scale": s["scale"], "out": s["out"], "workspace": s["ws"], **scales}
    if kind in ("decode", "token"):
        out = B.attn_decode(s["q"], *pools, *where, **kept)
    elif kind == "shared":
        out = B.attn_decode_shared(s["q"], *pools, *where, group_size=GROUP, shared_lens=s["shared"], **kept)
    else:
        call = B.attn_step if kind == "step" else B.attn_append
        out = call(s["q"], s["new"], s["off"], *pools, *where, max_q_len=s["max_q"], **kept)
    return {"out": out, "k": s["k"], "v": s["v"], **scales} if kind in ("token", "turn") else out


def work(case):
    w, ctx, new = _lengths(case)
    total, pages = int(new.sum()), int(((ctx + PAGE - 1) // PAGE).sum())
    first = ctx - new
    touched = int(((ctx + PAGE - 1) // PAGE - first // PAGE).sum())
    rows = total * case["kv_heads"] * case["head_dim"]
    fp8 = case["kv"] == "fp8_e4m3"
    # new K and V rows: read once, written once; a table entry and, over FP8, two scales read and written per page
    write = 2 * rows * (ITEM[case["q"]] + ITEM[case["kv"]]) + touched * (4 + (16 if fp8 else 0))
    if case["kind"] == "kv_write":
        return {"bytes": write, "flops": 0}
    a = W.algorithmic_work(w, ctx, new)
    n = a["bytes"]
    if case["kind"] == "shared":          # the prompt's pages once per group
        again = case["batch"] - case["batch"] // GROUP
        n -= again * case["prompt"] * 2 * case["kv_heads"] * case["head_dim"] * ITEM[case["kv"]]
        n -= again * (case["prompt"] // PAGE) * (12 if fp8 else 4)
    if case["kind"] in ("token", "turn"):
        n += write
    return {"bytes": n, "flops": a["flops"]}


def tolerance(case):
    # About four times what sampled rows of these cases differ by from attention in 64 bits on the same stored inputs:
    # 1.6e-7 (largest 5.4e-7) in float32; 2.1e-3 .. 2.9e-3 (largest 7e-3 .. 1.3e-2) in bf16, where the rounding of the
    # output to bf16 alone is 1.7e-3.  In a recomputation the first rows of a history dominate the norm: 2e-4.
    if case["kind"] == "kv_write":
        return "exact"
    if case["q"] == "f32":
        return {"rel": 1e-6, "max": 3e-6}
    return {"rel": 1e-3 if case["ctx"] == "const" else 1e-2, "max": 0.05}
