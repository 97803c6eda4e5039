"""The merge of split rows at every count of pieces where it changes its way of folding them."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import attention as O
from paper_2512_22560_amd import binding as B
from paper_2512_22560_amd import workloads as W
from tests.gpu_common import check, oracle_decode
from tests.helpers import oracle_args

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PIECES = [0, 1, 2, 3, 4, 5, 6, 8, 9, 15, 16, 17, 18, 64, 65, 131]


# group 5 and 3: the last chunk of a row is not full; 20: a second head tile; 16 over 8 KV heads: a workgroup takes several chunks
@pytest.mark.parametrize("qd,hkv,group,d,copies", [("f32", 1, 5, 64, 1), ("f32", 1, 4, 128, 1), ("bf16", 2, 5, 128, 1), ("bf16", 1, 20, 64, 1),
                                                   ("bf16", 1, 3, 64, 1), ("bf16", 8, 16, 128, 3)])
def test_rows_of_every_number_of_pieces(qd, hkv, group, d, copies):
    # with fewer blocks than workers every block of 32 tokens is a piece (with three copies over eight heads: every few)
    lens = np.array([max(0, 32 * p - (p % 3)) for p in PIECES] * copies)
    b = W.build(W.Workload("pieces", len(lens), hkv * group, hkv, d, qd, qd, ("const", 1), seed=W.BASE_SEED + 95), DEV)
    w, dt = b.workload, torch.float32 if qd == "f32" else torch.bfloat16
    gen = torch.Generator(device=DEV).manual_seed(96)
    pages = (lens + 15) // 16
    table = np.full((len(lens), int(pages.max())), -1, dtype=np.int32)
    ids = np.random.default_rng(97).permutation(int(pages.sum())).astype(np.int32)
    for i, end in enumerate(np.cumsum(pages)):
        table[i, :pages[i]] = ids[end - pages[i]:end]
    k, v = (torch.randn((int(pages.sum()), hkv, 16, d), generator=gen, device=DEV).to(dt) for _ in range(2))
    pt, cl = torch.from_numpy(table).to(DEV), torch.from_numpy(lens.astype(np.int32)).to(DEV)
    out, lse = B.attn_decode_lse(b.q, k, v, pt, cl, sm_scale=w.sm_scale)
    args = dict(k_pages=W.raw_numpy(k), v_pages=W.raw_numpy(v), page_table=table, ctx_lens=lens, sm_scale=w.sm_scale, q_dtype=qd, kv_dtype=qd)
    check(out, O.attn_decode(W.raw_numpy(b.q), **args), qd, "pieces")
    assert torch.isneginf(lse[cl == 0]).all() and torch.isfinite(lse[cl > 0]).all() and not out[cl == 0].any()
    again, lse2 = B.attn_decode_lse(b.q, k, v, pt, cl, sm_scale=w.sm_scale)
    assert torch.equal(out, again) and torch.equal(lse, lse2)


# more groups than the plan keeps in LDS; odd groups with a long private part (many pieces per row), one without shared
# tokens and one whose member is shorter than the prompt; one long prompt and private parts of one token (one piece per row)
@pytest.mark.parametrize("group_size,groups,ctx,shared", [(1, 4097, (1, 70), 32), (3, 3, (3000, 9000), 2500), (3, 4, (64, 700), 640), (8, 2, (1025, 1025), 1024)])
def test_shared_half_folds_into_rows_of_every_kind(group_size, groups, ctx, shared):
    b = W.build(W.Workload("fold", group_size * groups, 16, 4, 128, "bf16", "bf16", ("uniform", *ctx), seed=W.BASE_SEED + 98), DEV)
    used = np.full(groups, shared)
    used[-1] = 0 if groups == 3 else shared
    b = W.alias_shared_prefix(b, group_size, np.minimum(used, b.ctx_lens_host.reshape(groups, group_size).min(1)))
    out = B.attn_decode_shared(b.q, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, group_size=group_size,
                               shared_lens=torch.from_numpy(used.astype(np.int32)).to(DEV), sm_scale=b.workload.sm_scale)
    check(out, oracle_decode(b), "bf16", "shared")


# one row, a last token that is alone in its step, more rows than lanes in a wave, the longest table that is not cut and the shortest that is
@pytest.mark.parametrize("batch,hq,hkv,d,ctx", [(1, 4, 1, 64, (1, 1)), (4, 8, 2, 64, (32, 256)), (5, 5, 1, 128, (63, 130)), (70, 12, 2, 64, (0, 200)), (64, 8, 1, 128, (0, 512)),
                                                (3, 8, 2, 64, (500, 512)), (3, 8, 2, 128, (257, 512)), (3, 8, 2, 64, (513, 520))])
def test_short_float32_contexts(batch, hq, hkv, d, ctx):
    b = W.build(W.Workload("short", batch, hq, hkv, d, "f32", "f32", ("uniform", *ctx), seed=W.BASE_SEED + 99), DEV)
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=b.workload.sm_scale)
    ws = B.alloc_workspace(desc, batch, DEV)
    out, lse = B.attn_decode_lse(b.q, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, sm_scale=b.workload.sm_scale, workspace=ws)
    check(out, oracle_decode(b), "f32", "short")
    assert torch.equal(torch.isneginf(lse), (b.ctx_lens == 0)[:, None].expand_as(lse))
    per, total, starts = B.read_plan(desc, ws)
    o_per, o_total, o_starts, _ = O.split_plan(b.ctx_lens_host, hkv * -(-hq // hkv // 4), B.plan_workers(desc))
    assert (per, total) == (o_per, o_total) and np.array_equal(starts, o_starts)


# up to 64 trajectories every wave plans for itself; empty ones in front, between and behind
@pytest.mark.parametrize("batch,lens", [(1, [1]), (1, [40000]), (3, [0, 33, 0]), (2, [0, 0]), (64, None), (65, None)])
def test_small_batches_are_planned_by_the_decode_waves(batch, lens):
    lens = np.array(lens if lens else np.random.default_rng(batch).integers(0, 900, batch) * np.random.default_rng(9).integers(0, 2, batch))
    b = W.build(W.Workload("waves", batch, 20, 2, 128, "bf16", "fp8_e4m3", ("const", max(1, int(lens.max()))), seed=W.BASE_SEED + 100), DEV)
    cl = torch.from_numpy(lens.astype(np.int32)).to(DEV)
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=b.workload.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale)
    ws = B.alloc_workspace(desc, batch, DEV)
    out = B.attn_decode(b.q, b.k_pages, b.v_pages, b.page_table, cl, sm_scale=b.workload.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale, workspace=ws)
    args = dict(oracle_args(b), ctx_lens=lens)
    check(out, O.attn_decode(W.raw_numpy(b.q), **args), "bf16", "waves")
    per, total, starts = B.read_plan(desc, ws)
    o_per, o_total, o_starts, _ = O.split_plan(lens, 2, B.plan_workers(desc))
    assert (per, total) == (o_per, o_total) and np.array_equal(starts, o_starts)


# Word 32 of the plan says whether pages are read by several workers (plain loads).  Up to 64 trajectories every wave decides for
# its own run (the word is the first one's), for more the plan launch does (8200: more than it looks through).
# Members of a group need not be neighbours; an empty trajectory's table is not looked at; one shared page is not worth plain loads.
@pytest.mark.parametrize("kvd", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("groups,each", [(3, 8), (12, 8), (2050, 4)])
def test_pages_read_with_and_without_the_streaming_hint(groups, each, kvd):
    batch, pages = groups * each, 3 if groups > 100 else 20
    lens = np.random.default_rng(groups).integers(17, 16 * pages + 1, batch)
    lens[5::7] = 0
    b = W.build(W.Workload("hint", batch, 8, 2, 128, "bf16", kvd, ("const", 1), seed=W.BASE_SEED + 101), DEV)
    own = np.arange(batch * pages, dtype=np.int32).reshape(batch, pages)
    own = np.random.default_rng(1).permutation(own.size).astype(np.int32)[own]
    grouped = own.copy()
    leader = np.arange(batch) % groups                    # member m of group g stands at m * groups + g
    grouped[:, :2] = own[leader, :2]
    first = own.copy()
    first[:, 0] = own[0, 0]
    stale = own.copy()
    stale[lens == 0] = own[(np.flatnonzero(lens == 0) + 1) % batch]
    gen = torch.Generator(device=DEV).manual_seed(102)
    k, v = (torch.randn((own.size, 2, 16, 128), generator=gen, device=DEV) for _ in range(2))
    ks = vs = None
    if kvd != "bf16":
        ks, vs = (x.abs().amax(dim=(1, 2, 3)) / 448.0 for x in (k, v))
        k, v = ((x / s.view(-1, 1, 1, 1)).to(torch.float8_e4m3fn).view(torch.uint8) for x, s in ((k, ks), (v, vs)))
    else:
        k, v = k.bfloat16(), v.bfloat16()
    cl = torch.from_numpy(lens.astype(np.int32)).to(DEV)
    members = np.bincount(leader[lens > 16], minlength=groups)
    for table, expect in ((own, lens < 0), (grouped, (lens > 16) & (members[leader] > 1)), (first, lens < 0), (stale, lens < 0)):
        pt = torch.from_numpy(table).to(DEV)
        desc = B.make_desc(b.q, k, pt, sm_scale=b.workload.sm_scale, k_scale=ks, v_scale=vs)
        ws = B.alloc_workspace(desc, batch, DEV)
        out = B.attn_decode(b.q, k, v, pt, cl, sm_scale=b.workload.sm_scale, k_scale=ks, v_scale=vs, workspace=ws)
        check(out, O.attn_decode(W.raw_numpy(b.q), k_pages=W.raw_numpy(k), v_pages=W.raw_numpy(v), page_table=table, ctx_lens=lens, sm_scale=b.workload.sm_scale,
                                 q_dtype="bf16", kv_dtype=kvd, k_scale=W.raw_numpy(ks), v_scale=W.raw_numpy(vs)), "bf16", "hint")
        per, total, starts = B.read_plan(desc, ws)
        blocks = -(-lens // 32)
        if batch > 64:                                   # a quarter of all blocks
            again = batch > 8192 or 4 * blocks[expect].sum() >= blocks.sum()
        else:
            again = expect[:int(np.searchsorted(np.cumsum(2 * blocks), starts[0, 3])) + 1].any()
        assert ws.view(torch.int32)[32].item() == again


def test_rows_of_one_kv_head_read_its_pages_again():
    # 20 query heads per KV head are two rows; a pool smaller than the contexts must be shared whatever the second pages say
    for batch, hq, pool, again in ((4, 20, 200, True), (4, 10, 200, False), (4, 10, 100, True), (70, 20, 4000, True), (70, 10, 4000, False), (70, 10, 1700, True)):
        b = W.build(W.Workload("tiles", batch, hq, 1, 128, "bf16", "bf16", ("const", 768), seed=W.BASE_SEED + 103), DEV)
        table = torch.from_numpy((np.arange(batch * 48).reshape(batch, 48) % pool).astype(np.int32)).to(DEV)
        k, v = (torch.randn((pool, 1, 16, 128), device=DEV, dtype=torch.bfloat16) for _ in range(2))
        desc = B.make_desc(b.q, k, table, sm_scale=b.workload.sm_scale)
        ws = B.alloc_workspace(desc, batch, DEV)
        out = B.attn_decode(b.q, k, v, table, b.ctx_lens, sm_scale=b.workload.sm_scale, workspace=ws)
        args = dict(oracle_args(b), k_pages=W.raw_numpy(k), v_pages=W.raw_numpy(v), page_table=W.raw_numpy(table))
        check(out, O.attn_decode(W.raw_numpy(b.q), **args), "bf16", "tiles")
        assert ws.view(torch.int32)[32].item() == again


def test_a_row_of_many_pieces_folds_alike_alone_and_among_many_rows():
    # three long contexts in a step of 150 trajectories (a chunk of the merge per wave) and by themselves (a workgroup per chunk)
    batch, long_ = 150, 3
    lens = np.full(batch, 40)
    lens[::50] = 20000
    b = W.build(W.Workload("fold", batch, 32, 8, 128, "bf16", "bf16", ("const", 1), seed=W.BASE_SEED + 104), DEV)
    rows, sel = np.where(lens > 40, 1, 2), np.flatnonzero(lens > 40)
    pages = (lens + 15) // 16
    table = np.full((batch, int(pages.max())), -1, dtype=np.int32)
    for i, end in enumerate(np.cumsum(pages)):
        table[i, :pages[i]] = np.arange(end - pages[i], end)
    gen = torch.Generator(device=DEV).manual_seed(105)
    k, v = (torch.randn((int(pages.sum()), 8, 16, 128), generator=gen, device=DEV).bfloat16() for _ in range(2))
    q = torch.randn((int(rows.sum()), 32, 128), generator=gen, device=DEV).bfloat16()
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x).astype(np.int32)).to(DEV)
    off = np.concatenate([[0], np.cumsum(rows)])
    kw = dict(sm_scale=b.workload.sm_scale)
    step = B.attn_step(q, to(rows), to(off), k, v, to(table), to(lens), max_q_len=2, **kw)
    alone = B.attn_decode(q[off[sel]].contiguous(), k, v, to(table[sel]), to(lens[sel]), **kw)
    assert len(sel) == long_ and torch.equal(step[off[sel]], alone)


def test_more_rows_than_a_launch_has_workgroups():
    # 64 rows of one head per trajectory, 2^24 of them and some: a workgroup per row would be more threads than a launch may have
    batch = (1 << 18) + 60
    q = torch.ones((batch, 64, 64), dtype=torch.bfloat16, device=DEV)
    k, v = (torch.randn((1, 64, 16, 64), device=DEV).bfloat16() for _ in range(2))
    table = torch.zeros((batch, 1), dtype=torch.int32, device=DEV)
    lens = torch.ones(batch, dtype=torch.int32, device=DEV)
    lens[::1000] = 0
    out = B.attn_decode(q, k, v, table, lens, sm_scale=0.125)
    assert torch.equal(out[1], v[0, :, 0]) and not out[::1000].any()
    out[::1000] = v[0, :, 0]
    assert bool((out == v[0, :, 0]).all())


# pages left in common by the private parts: none; a short member leaves the prompt to the others; the caller says nothing
@pytest.mark.parametrize("groups", [4, 40])
@pytest.mark.parametrize("said,short,again", [(640, False, False), (656, False, False), (640, True, True), (0, False, True)])
def test_private_parts_that_share_pages_read_them_plainly(groups, said, short, again):
    b = W.build(W.Workload("own", 8 * groups, 16, 4, 128, "bf16", "bf16", ("uniform", 700, 900), seed=W.BASE_SEED + 106), DEV)
    b = W.alias_shared_prefix(b, 8, np.full(groups, max(said, 640)))
    lens = b.ctx_lens_host.copy()
    if short:
        lens[3::8] = 40
    cl = torch.from_numpy(lens.astype(np.int32)).to(DEV)
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=b.workload.sm_scale)
    ws = torch.empty(B.lib().rollattn_shared_workspace_bytes(ctypes.byref(desc), 8), dtype=torch.uint8, device=DEV)
    out = B.attn_decode_shared(b.q, b.k_pages, b.v_pages, b.page_table, cl, group_size=8, shared_lens=torch.full((groups,), said, dtype=torch.int32, device=DEV),
                               sm_scale=b.workload.sm_scale, workspace=ws)
    assert ws.view(torch.int32)[32].item() == again
    check(out, O.attn_decode(W.raw_numpy(b.q), **dict(oracle_args(b), ctx_lens=lens)), "bf16", "own")
