"""Decode rows taken whole by a wave each: on both sides of the rule that chooses it (word 6 of the plan), against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import attention as O
from paper_2512_22560_amd import binding as B
from paper_2512_22560_amd import workloads as W
from tests.gpu_common import check, oracle_append
from tests.helpers import oracle_args

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
WORKERS = 2048


def _whole(lens, heads, kvd):
    """The rule, as plan_whole states it, for the trajectories that take part.  No case here is a near tie."""
    group, tiles = heads[0] // heads[1], -(-(heads[0] // heads[1]) // 16)
    rows_per_b = heads[1] * tiles
    blocks = -(-np.asarray(lens) // 32)
    if len(blocks) <= 64 or not blocks.any():
        return False
    busy = (900 if kvd == "fp8_e4m3" else 450) * tiles
    longest, rows, total = int(blocks.max()), int((blocks > 0).sum()) * rows_per_b, int(blocks.sum()) * rows_per_b
    step = -(-longest // 32)
    levels = np.arange(0, longest, step)
    n = (blocks[None, :] > (levels + (step - 1) // 2)[:, None]).sum(1) * rows_per_b * min(1.0, WORKERS / rows)
    late = (np.minimum(step, longest - levels) * np.maximum(0.0, 1 - n / busy)).sum()
    per = max(1, -(-total // WORKERS))
    used = -(-total // per)
    late -= per * max(0.0, 1 - used / busy)
    gain = 1.2 + (used - 1) * (1 - rows / total) * group * heads[2] / (tiles * 16 * 128) / 130 + (4 if rows > WORKERS else 0)
    assert abs(late - gain) > 0.01
    return late <= gain


def _batch(name, batch, heads, kvd, lens, seed):
    b = W.build(W.Workload(name, batch, *heads, "bf16", kvd, ("const", int(max(1, lens.max()))), seed=W.BASE_SEED + seed), DEV)
    b.ctx_lens_host[:] = lens
    b.ctx_lens.copy_(torch.from_numpy(lens.astype(np.int32)))
    return b


# rows per KV head: one, and two of 20 query heads; rows fewer than waves and more of them, none for some; contexts of one token, of whole
# blocks and none; short ones alone, and the same with one long one among them, which would go on by itself for most of the call
WHOLE, DEALT = True, False


@pytest.mark.parametrize("kvd", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("batch,heads,lens,longest,expect", [
    (64, (64, 4, 128), (33, 64), 64, DEALT), (65, (64, 4, 128), (33, 64), 64, WHOLE), (65, (64, 4, 128), (33, 64), 544, DEALT),
    (65, (32, 8, 128), (32, 32), 544, DEALT), (400, (40, 2, 64), (200, 260), 260, WHOLE), (400, (40, 2, 64), (200, 260), 800, DEALT),
    (1300, (32, 2, 128), (1, 70), 96, WHOLE), (1300, (32, 2, 128), (1, 70), 900, DEALT), (1300, (8, 2, 64), (1, 33), 64, WHOLE),
    (300, (16, 8, 128), (1, 100), 128, WHOLE), (300, (16, 8, 128), (1, 100), 700, DEALT),
])
def test_rows_whole_and_dealt(batch, heads, lens, longest, expect, kvd):
    lens = np.random.default_rng(batch).integers(lens[0], lens[1] + 1, batch)
    lens[3::41] = 0
    lens[1::13] = 32
    lens[batch // 2] = longest
    assert _whole(lens, heads, kvd) == expect
    b = _batch("whole", batch, heads, kvd, lens, 210)
    w = b.workload
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=w.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale)
    ws = B.alloc_workspace(desc, batch, DEV)
    out, lse = B.attn_decode_lse(b.q, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, sm_scale=w.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale, workspace=ws)
    ref = O.attn_decode(W.raw_numpy(b.q), **dict(oracle_args(b), ctx_lens=lens))
    check(out, ref, "bf16", "whole rows")
    if batch > 64:
        assert ws.view(torch.int32)[6].item() == expect
    # the same rows dealt to one worker less: the same attention and denominators, but for the order of the sums
    before = B.set_decode_workers(WORKERS - 1)
    try:
        dealt, lse_dealt = B.attn_decode_lse(b.q, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, sm_scale=w.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale)
    finally:
        B.set_decode_workers(before)
    check(dealt, ref, "bf16", "dealt rows")
    live = torch.from_numpy(lens > 0).to(DEV)
    assert torch.equal(torch.isinf(lse), torch.isinf(lse_dealt)) and bool(torch.isinf(lse[~live]).all())
    # float sums of up to 2^11 weights in two orders: 2^11 roundings of 2^-24 at most, in log2 units, and as much for the references
    assert (lse[live] - lse_dealt[live]).abs().max().item() <= 1e-3


def test_more_rows_than_a_launch_has_waves():
    # a million rows over few pages: each wave takes hundreds, some trajectories have none
    n, heads = 131080, (8, 8, 64)
    gen, rng = torch.Generator(device=DEV).manual_seed(5), np.random.default_rng(5)
    lens = rng.integers(0, 17, n).astype(np.int32)
    table = rng.integers(0, 64, (n, 1)).astype(np.int32)
    q = torch.randn((n, heads[0], heads[2]), generator=gen, device=DEV, dtype=torch.bfloat16)
    k, v = (torch.randn((64, heads[1], 16, heads[2]), generator=gen, device=DEV, dtype=torch.bfloat16) for _ in range(2))
    args = (q, k, v, torch.from_numpy(table).to(DEV), torch.from_numpy(lens).to(DEV))
    ws = B.alloc_workspace(B.make_desc(q, k, args[3], sm_scale=0.125), n, DEV)
    out = torch.full_like(q, float("nan"))
    B.attn_decode(*args, sm_scale=0.125, out=out, workspace=ws)
    assert ws.view(torch.int32)[6].item() == 1
    before = B.set_decode_workers(WORKERS - 1)
    try:
        dealt = B.attn_decode(*args, sm_scale=0.125)       # rows of one block are never cut
    finally:
        B.set_decode_workers(before)
    assert torch.equal(out, dealt)
    some = np.concatenate([np.arange(40), rng.integers(0, n, 60), [n - 1]])
    at = torch.from_numpy(some).to(DEV)
    check(out[at], O.attn_decode(W.raw_numpy(q[at]), W.raw_numpy(k), W.raw_numpy(v), table[some], lens[some], sm_scale=0.125, q_dtype="bf16", kv_dtype="bf16"),
          "bf16", "many rows")


@pytest.mark.parametrize("heads,kvd", [((64, 4, 128), "fp8_e4m3"), ((40, 2, 64), "bf16"), ((32, 8, 128), "bf16")])
@pytest.mark.parametrize("groups,prompt,own", [(9, 320, (1, 90)), (9, 0, (1, 300)), (40, 96, (1, 64)), (40, 96, (300, 700))])
def test_whole_private_parts_take_the_shared_half(groups, prompt, own, heads, kvd):
    b = W.build(W.Workload("own", 8 * groups, *heads, "bf16", kvd, ("uniform", prompt + own[0], prompt + own[1]), seed=W.BASE_SEED + 211), DEV)
    if prompt:
        b = W.alias_shared_prefix(b, 8, np.full(groups, prompt))
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=b.workload.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale)
    ws = torch.full((B.lib().rollattn_shared_workspace_bytes(ctypes.byref(desc), 8),), 255, dtype=torch.uint8, device=DEV)
    out = B.attn_decode_shared(b.q, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, group_size=8, sm_scale=b.workload.sm_scale, workspace=ws,
                               shared_lens=torch.full((groups,), prompt, dtype=torch.int32, device=DEV), k_scale=b.k_scale, v_scale=b.v_scale)
    shared = np.minimum(prompt, b.ctx_lens_host.reshape(groups, 8).min(1) - 1) // 32 * 32
    assert ws.view(torch.int32)[6].item() == _whole(b.ctx_lens_host - np.repeat(shared, 8), heads, kvd)
    check(out, O.attn_decode(W.raw_numpy(b.q), **oracle_args(b)), "bf16", "shared")


@pytest.mark.parametrize("decode_rows,ctx,whole", [(64, (33, 64), DEALT), (65, (33, 64), WHOLE), (200, (33, 150), WHOLE), (200, (33, 3000), DEALT)])
def test_a_step_takes_its_rows_as_a_call_of_their_own_would(decode_rows, ctx, whole):
    # (with 64 the call of their own plans in its waves, and the step must not take them whole either)
    heads = (64, 4, 128)
    b = W.build(W.Workload("step", decode_rows + 30, *heads, "bf16", "bf16", ("uniform", *ctx), qlen=("uniform", 2, 40), append_rows=30,
                           ctx_is_prefix=True, seed=W.BASE_SEED + 212), DEV)
    sel = np.flatnonzero(b.q_lens_host == 1)
    assert len(sel) == decode_rows and _whole(b.ctx_lens_host[sel], heads, "bf16") == whole
    w = b.workload
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=w.sm_scale)
    ws = torch.empty(B.lib().rollattn_step_workspace_bytes(ctypes.byref(desc), int(b.q_lens_host.sum())), dtype=torch.uint8, device=DEV)
    out = B.attn_step(b.q, b.q_lens, b.q_offsets, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, sm_scale=w.sm_scale, max_q_len=40, workspace=ws)
    assert ws.view(torch.int32)[6].item() == whole
    check(out, oracle_append(b), "bf16", "step")
    at = torch.from_numpy(np.concatenate([[0], np.cumsum(b.q_lens_host)])[sel]).to(DEV)
    rows = torch.from_numpy(sel).to(DEV)
    q, table, ctx_lens = b.q[at].contiguous(), b.page_table[rows].contiguous(), b.ctx_lens[rows].contiguous()
    own_ws = B.alloc_workspace(B.make_desc(q, b.k_pages, table, sm_scale=w.sm_scale), decode_rows, DEV)
    own = B.attn_decode(q, b.k_pages, b.v_pages, table, ctx_lens, sm_scale=w.sm_scale, workspace=own_ws)
    assert decode_rows == 64 or own_ws.view(torch.int32)[6].item() == whole
    assert torch.equal(out[at], own)


# Page scales are worked out for 64 pages at a time: contexts that end at, before and behind such windows (1024 tokens), in steps
# of 64 tokens and of 128 (short chunks), with scales that differ from page to page; tiles that walk five windows, and the same cut
# into pieces, which start again at the first.
@pytest.mark.parametrize("cut", [False, True])
@pytest.mark.parametrize("new", [3, 40])
@pytest.mark.parametrize("hkv,d", [(1, 128), (2, 64)])
def test_append_over_fp8_pages_of_several_scale_windows(new, hkv, d, cut):
    lens = np.array([1008, 1023, 1024, 1025, 1040, 1088, 2047, 2049, 2112, 3071, 3073, 4100])
    b = W.build(W.Workload("windows", len(lens), 8 * hkv, hkv, d, "bf16", "fp8_e4m3", ("const", 4100), qlen=("const", new), seed=W.BASE_SEED + 213), DEV)
    factor = torch.exp2(torch.from_numpy(np.random.default_rng(3).integers(-2, 2, b.k_scale.numel()).astype(np.float32)).to(DEV))
    b.k_scale.mul_(factor)
    b.v_scale.mul_(torch.flip(factor, [0]) * 0.5)          # (values of unit scale or less, where the bar is stated)
    b.ctx_lens_host[:] = lens
    b.ctx_lens.copy_(torch.from_numpy(lens.astype(np.int32)))
    w = b.workload
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=w.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale)
    least = 256 + -(-32 * B.lib().rollattn_append_plan_capacity(ctypes.byref(desc), b.total_q) // 256) * 256   # room for the list, none for partials
    ws = torch.empty(B.workspace_bytes(desc, b.total_q) if cut else least, dtype=torch.uint8, device=DEV)
    out = B.attn_append(b.q, b.q_lens, b.q_offsets, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, sm_scale=w.sm_scale, max_q_len=new,
                        k_scale=b.k_scale, v_scale=b.v_scale, workspace=ws)
    tiles, merges = ws.view(torch.int32)[4:6].tolist()
    longest = max(ws[256:].view(torch.int32)[:8 * tiles].view(-1, 8)[:, 6].tolist())
    assert (merges > 0) == cut and (longest < 32 if cut else longest == -(-4100 // 64))
    args = dict(oracle_args(b), ctx_lens=lens)
    ref = O.attn_append(W.raw_numpy(b.q), b.q_lens_host, **args)
    check(out, ref, "bf16", "windows")
    # (the bar tells scales of two windows before from the right ones)
    table, stale = args["page_table"], {}
    for name in ("k_scale", "v_scale"):
        stale[name] = args[name].copy()
        for i, n in enumerate(-(-lens // 16)):
            stale[name][table[i, 128:n]] = args[name][table[i, :max(0, n - 128)]]
    wrong = O.attn_append(W.raw_numpy(b.q), b.q_lens_host, **dict(args, **stale))
    with pytest.raises(AssertionError):
        check(torch.from_numpy(wrong), ref, "bf16", "stale windows")
