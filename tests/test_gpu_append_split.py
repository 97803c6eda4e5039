"""Append calls with few tiles: their tiles are cut into pieces of the context whose partial results a merge folds."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import attention as O
from paper_2512_22560_amd import binding as B
from paper_2512_22560_amd import workloads as W
from tests.gpu_common import check, gpu_append, oracle_append
from tests.helpers import oracle_args

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _append(b):
    w = b.workload
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=w.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale)
    ws = B.alloc_workspace(desc, b.total_q, DEV)
    out, lse = B.attn_append_lse(b.q, b.q_lens, b.q_offsets, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, sm_scale=w.sm_scale,
                                 max_q_len=int(b.q_lens_host.max()), k_scale=b.k_scale, v_scale=b.v_scale, workspace=ws)
    pieces, merges = ws.view(torch.int32)[4:6].tolist()
    return out, lse, pieces, merges, B.read_append_plan(desc, ws, b.total_q)


# (name, batch, Hq, Hkv, D, prefix, new tokens, cut): contexts too short to be cut, on and just past a block edge; one tile and several; half tiles; chunks longer than a piece, whose first
# rows do not see its later pieces; half tiles of one to five blocks; groups that leave a tile ragged; one KV head and more than eight
CASES = [
    ("below", 1, 8, 8, 128, (900, 900), (40, 40), False), ("block_edge", 1, 8, 8, 128, (1495, 1495), (41, 41), True),
    ("past_edge", 1, 8, 8, 128, (1496, 1496), (41, 41), True), ("long", 2, 32, 8, 128, (6000, 9000), (3, 3), True),
    ("half", 5, 64, 4, 128, (100, 9000), (1, 8), True), ("causal", 1, 16, 4, 128, (0, 0), (3001, 3001), True),
    ("g3_d64", 3, 6, 2, 64, (2000, 5000), (100, 300), True), ("one_head", 2, 40, 1, 128, (3000, 8000), (5, 70), True),
    ("sixteen", 2, 16, 16, 64, (2500, 2600), (257, 300), True), ("skewed", 30, 16, 4, 128, (10, 14000), (1, 200), True),
    # the cheapest cut would need more slots than there are, another one fits
    ("crowded", 13, 32, 8, 64, (12000, 12000), (64, 64), True),
    # few tokens per chunk over bf16 pools: the chip already reads as fast as it can
    ("at_memory_rate", 40, 64, 4, 128, (6000, 6000), (2, 2), None),
    ("steps", 40, 64, 4, 128, (0, 260), (1, 8), False), ("steps_d64", 40, 4, 2, 64, (0, 260), (1, 30), False),
]


@pytest.mark.parametrize("kvd", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("name,batch,hq,hkv,d,prefix,new,cut", CASES, ids=[c[0] for c in CASES])
def test_pieces_and_merge_against_the_oracle(name, batch, hq, hkv, d, prefix, new, cut, kvd):
    b = W.build(W.Workload(name, batch, hq, hkv, d, "bf16", kvd, ("loguniform" if name == "skewed" else "uniform", *prefix),
                           qlen=("uniform", *new), ctx_is_prefix=True, seed=W.BASE_SEED + 91), DEV)
    out, lse, pieces, merges, tiles = _append(b)
    if cut is None:                                   # whole over bf16 pools, cut over the half as wide FP8 ones
        cut = kvd != "bf16"
    assert (merges > 0) == cut and (pieces > len(tiles)) == cut
    half = int(b.q_lens_host.max()) * (hq // hkv) <= 128
    assert np.array_equal(tiles, O.append_tile_plan(b.q_lens_host, b.ctx_lens_host, max(1, (128 if half else 256) // (hq // hkv)))[:, :2])
    check(out, oracle_append(b), "bf16", name)
    if b.total_q * hq <= 5000:                        # (the oracle's denominators go row by row)
        ref = O.attn_lse(W.raw_numpy(b.q), b.q_lens_host, **{k: v for k, v in oracle_args(b).items() if k not in ("v_pages", "v_scale")})
        # log2 of the denominators: as tests/test_gpu_lse_merge.py states for append over bf16 pools (the scaled query is rounded)
        assert np.abs(lse.double().cpu().numpy() - ref).max() <= 1e-2
    again = _append(b)
    assert torch.equal(out, again[0]) and torch.equal(lse, again[1])


# over FP8 pools the pieces of the 63-block prompt have odd numbers of blocks too, and end inside a step of two
@pytest.mark.parametrize("kvd", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("prompt", [4000, 6976])
def test_shared_prompts_of_few_groups_are_cut_too(prompt, kvd):
    shared = np.array([prompt, 0])                    # one long prompt, one group that shares nothing
    b = W.build(W.Workload("sp", 16, 32, 8, 128, "bf16", kvd, ("uniform", prompt + 100, prompt + 400), seed=W.BASE_SEED + 92), DEV)
    b = W.alias_shared_prefix(b, 8, shared)
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=b.workload.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale)
    ws = torch.empty(B.lib().rollattn_shared_workspace_bytes(ctypes.byref(desc), 8), dtype=torch.uint8, device=DEV)
    out = B.attn_decode_shared(b.q, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, group_size=8, shared_lens=torch.from_numpy(shared.astype(np.int32)).to(DEV),
                               sm_scale=b.workload.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale, workspace=ws)
    # (the shared half's plan lies behind the private half's workspace, as in a mixed step)
    app = ws[B.lib().rollattn_step_append_offset(ctypes.byref(desc)):]
    tiles, merges = app.view(torch.int32)[4:6].tolist()
    blocks = app[256:].view(torch.int32)[:8 * tiles].view(-1, 8)[:, 6].tolist()
    assert merges == 1 and tiles > 3 and sum(blocks) == -(-prompt // 64)
    assert any(n % 2 for n in blocks if n)
    check(out, O.attn_decode(W.raw_numpy(b.q), **oracle_args(b)), "bf16", "shared")


@pytest.mark.parametrize("kvd", ["bf16", "fp8_e4m3"])
def test_a_workspace_without_room_for_pieces_leaves_the_tiles_whole(kvd):
    # sized for the records alone, all that a call needs; one for a decode step of the same descriptor is enough to cut, if
    # into fewer pieces than the size the call is told to bring
    b = W.build(W.Workload("room", 18, 32, 8, 64, "bf16", kvd, ("loguniform", 3000, 12000), qlen=("uniform", 40, 70), ctx_is_prefix=True,
                           seed=W.BASE_SEED + 93), DEV)
    w = b.workload
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=w.sm_scale, k_scale=b.k_scale, v_scale=b.v_scale)
    least = 256 + -(-32 * B.lib().rollattn_append_plan_capacity(ctypes.byref(desc), b.total_q) // 256) * 256
    got, pieces, ref = [], [], oracle_append(b)
    for n in (least, B.workspace_bytes(desc, w.batch), B.workspace_bytes(desc, b.total_q)):
        ws = torch.empty(n, dtype=torch.uint8, device=DEV)
        got.append(gpu_append(b, workspace=ws))
        pieces.append(ws.view(torch.int32)[4].item() if ws.view(torch.int32)[5].item() else 0)
        check(got[-1], ref, "bf16", "room")
    assert 0 == pieces[0] < pieces[1] <= pieces[2] and (pieces[1] < pieces[2] or kvd == "bf16")
    with pytest.raises(B.RollattnError):
        gpu_append(b, workspace=torch.empty(least - 256, dtype=torch.uint8, device=DEV))
    # a mixed step of the chunks alone cuts them alike, where it has to in the room of the decode rows' partials
    more = B.lib().rollattn_step_workspace_bytes(ctypes.byref(desc), b.total_q)
    less = B.lib().rollattn_step_append_offset(ctypes.byref(desc)) + 256 + 32 * 8 * (96 + 32)
    for n, same in ((more, got[2]), (less, got[1])):
        step = B.attn_step(b.q, b.q_lens, b.q_offsets, b.k_pages, b.v_pages, b.page_table, b.ctx_lens, sm_scale=w.sm_scale, k_scale=b.k_scale,
                           v_scale=b.v_scale, max_q_len=int(b.q_lens_host.max()), workspace=torch.empty(n, dtype=torch.uint8, device=DEV))
        assert torch.equal(step, same)


@pytest.mark.parametrize("lend", [False, True])
def test_a_mixed_step_with_cut_chunks_and_split_rows(lend):
    # two chunks behind long prefixes, cut; the decode rows, split over many workers, take the same room for their partials afterwards
    b = W.build(W.Workload("both", 6, 32, 8, 128, "bf16", "bf16", ("uniform", 6000, 9000), qlen=("uniform", 20, 90), ctx_is_prefix=True,
                           append_rows=2, seed=W.BASE_SEED + 94), DEV)
    w = b.workload
    desc = B.make_desc(b.q, b.k_pages, b.page_table, sm_scale=w.sm_scale)
    n = B.lib().rollattn_step_append_offset(ctypes.byref(desc)) + 256 + 32 * 8 * (96 + 32) if lend else B.lib().rollattn_step_workspace_bytes(ctypes.byref(desc), b.total_q)
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    args = (b.q, b.q_lens, b.q_offsets, b.k_pages, b.v_pages, b.page_table, b.ctx_lens)
    kw = dict(sm_scale=w.sm_scale, max_q_len=int(b.q_lens_host.max()), workspace=ws)
    out = B.attn_step(*args, **kw).clone()
    assert ws[B.lib().rollattn_step_append_offset(ctypes.byref(desc)):].view(torch.int32)[5].item() > 0
    check(out, oracle_append(b), "bf16", "both")
    assert all(torch.equal(out, B.attn_step(*args, **kw)) for _ in range(3))


# half tiles over FP8 pools: steps of one block and of two, chosen by each tile's blocks; below 20 blocks of 64 tokens and from there on
@pytest.mark.parametrize("hq,hkv,d", [(64, 4, 128), (4, 2, 64)])
@pytest.mark.parametrize("ctx", [(1, 70), (1000, 1208), (1209, 1290)])
def test_steps_of_one_block_and_of_two(hq, hkv, d, ctx):
    b = W.build(W.Workload("steps", 140, hq, hkv, d, "bf16", "fp8_e4m3", ("uniform", *ctx), qlen=("uniform", 1, 8), ctx_is_prefix=True,
                           seed=W.BASE_SEED + 96), DEV)
    out = gpu_append(b)
    check(out, oracle_append(b), "bf16", "steps")
    wide = torch.full((b.page_table.shape[0], 200), -1, dtype=torch.int32, device=DEV)
    wide[:, :b.page_table.shape[1]] = b.page_table
    b.page_table = wide
    assert torch.equal(out, gpu_append(b))               # a wider table, the same tiles
