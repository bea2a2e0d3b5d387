"""GPU parity of the group kernel (up to 128 query rows per work item, chosen by the planner where
shared rows meet many query rows) against the CPU oracle: every split of the rows over its waves,
ragged steps around its tiles of 32 and 64 rows, small and whole-workgroup items of few rows, both
head sizes and pool formats, growth between decode steps, graph capture."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_13575_amd as ets
from workload import (Tree, TreeConfig, make_values_fp8_host, make_values_host, with_growth_room)

from _gpu_util import compare, make_ctx, oracle_rows, pool_to_device, pool_to_host, to_device

pytestmark = pytest.mark.gpu

KS, VS = 0.0123, 0.0217
LENGTHS = [1, 15, 16, 17, 31, 32, 33, 47, 48, 63, 64, 65, 96, 127, 130, 200]


def edge_tree(root, sizes, seed):
    """A root, under it branches of `sizes` leaf queries (a shared node each, and one more that all
    but the first of them share), lengths around the kernel's tiles, some leaf nodes empty or long."""
    r = np.random.default_rng(seed)
    parent, n_tok, leaves = [-1], [root], []
    for c in sizes:
        parent.append(0)
        n_tok.append(int(r.choice(LENGTHS)))
        top = len(parent) - 1
        parent.append(top)
        n_tok.append(int(r.choice(LENGTHS)))
        for j in range(c):
            parent.append(top if j == 0 else top + 1)
            n_tok.append(int(r.choice(LENGTHS + [0, 700])))
            leaves.append(len(parent) - 1)
    parent, n_tok = np.array(parent, np.int32), np.array(n_tok, np.int32)
    off = np.cumsum(n_tok.astype(np.int64)) - n_tok
    return Tree(parent, off, n_tok, np.array(leaves, np.int32), int(n_tok.sum()), np.zeros(parent.size, np.int32))


def sizes_for(rows, group, seed):
    """Branch sizes whose leaf queries have `rows` query rows together."""
    r = np.random.default_rng(seed)
    n, out = rows // group, []
    while n > 0:
        out.append(min(n, int(r.choice([1, 2, 3, 4, 5, 7, 8, 9, 12, 16, 17, 31]))))
        n -= out[-1]
    return out


def attend(ctx, st, tree, kd, vd, qd):
    out = torch.full((tree.n_leaves, ctx.shape.n_q_heads, ctx.shape.head_dim), float("nan"), device="cuda:0")
    lse = torch.full((tree.n_leaves, ctx.shape.n_q_heads), float("nan"), device="cuda:0")
    ws = torch.empty(max(st.workspace_bytes, 16), dtype=torch.uint8, device="cuda:0")
    ctx.decode(kd, vd, kd.shape[1], qd, out, lse, ws, ws.numel())
    return out, lse, ws


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("hq,d,rows,root", [
    # several groups (with one or two heads to a kv head more rows of leaf nodes stand beside the root: it has
    # to be long enough for the planner to choose this kernel)
    (64, 128, 512, 4160), (32, 128, 516, 4170), (16, 128, 520, 8320), (8, 128, 510, 16321),
    (64, 128, 192, 11000), (64, 128, 104, 33000), (32, 128, 232, 8300),  # fewer than two
    (64, 64, 560, 4160), (32, 64, 600, 4175), (8, 64, 515, 12320)])
def test_parity_over_row_counts_formats_and_head_sizes(hq, d, rows, root, fp8):
    cfg = TreeConfig("group", 8, hq, d, "bf16", 0, 0, 0, 0, 0, None, seed=71 + rows)
    group = hq // 8
    tree = edge_tree(root, sizes_for(rows, group, rows + hq), rows + d)
    print("case group", hq, d, rows, root, fp8, flush=True)
    k, v, q = make_values_fp8_host(cfg, tree, KS, VS) if fp8 else make_values_host(cfg, tree)
    r = np.random.default_rng(5)
    pick = (np.concatenate([np.arange(min(tree.n_leaves, 12)), r.integers(0, tree.n_leaves, 180)]),
            r.integers(0, hq, min(tree.n_leaves, 12) + 180))
    with make_ctx(cfg) as ctx:
        if fp8:
            ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, KS, VS)
        st = ctx.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node)
        assert ctx.item_rows() == 128
        assert ctx.check().violations == 0
        kd, vd, qd = pool_to_device(k), pool_to_device(v), to_device(q)
        out, lse, _ = attend(ctx, st, tree, kd, vd, qd)
        again, lse2, _ = attend(ctx, st, tree, kd, vd, qd)
        torch.cuda.synchronize()
    assert torch.equal(out, again) and torch.equal(lse, lse2)
    if fp8:
        oo, ol = oracle.tree_decode_attn_fp8kv(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node,
                                               k, v, KS, VS, q, 8, hq, d, rows=pick)
    else:
        oo, ol = oracle_rows(cfg, tree, k, v, q, *pick)
    compare(out.cpu().numpy()[pick], lse.cpu().numpy()[pick], oo, ol, "bf16", "group")


@pytest.mark.parametrize("hq,d", [(64, 128), (32, 64)])
def test_growth_between_decode_steps(hq, d):
    """The step lists of joined segments follow the advances: 36 of them, past the room the lists keep
    for growth, against a fresh plan of the grown tree and the oracle."""
    cfg = TreeConfig("group", 8, hq, d, "bf16", 0, 0, 0, 0, 0, None, seed=73)
    tree = edge_tree(4160, sizes_for(576, hq // 8, 9), 10)
    grows = np.unique(tree.leaf_node)
    tree = with_growth_room(tree, 40)
    k, v, q = make_values_host(cfg, tree)
    kd, vd, qd = pool_to_device(k), pool_to_device(v), to_device(q)
    print("case group growth", hq, d, flush=True)
    with make_ctx(cfg) as ctx, make_ctx(cfg) as fresh:
        ctx.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node)
        assert ctx.item_rows() == 128
        n_tokens = tree.n_tokens.copy()
        for step in range(36):
            ctx.plan_advance()
            n_tokens[grows] += 1
            if step not in (0, 4, 30, 35):
                continue
            grown = Tree(tree.parent, tree.tok_offset, n_tokens, tree.leaf_node, tree.pool_tokens, tree.leaf_node)
            out, lse, _ = attend(ctx, ctx.stats(), tree, kd, vd, qd)
            st = fresh.plan(tree.parent, tree.tok_offset, n_tokens, tree.leaf_node)
            want, want_lse, _ = attend(fresh, st, tree, kd, vd, qd)
            torch.cuda.synchronize()
            compare(out.cpu().numpy().reshape(-1, d), lse.cpu().numpy().reshape(-1),
                    want.cpu().numpy().reshape(-1, d), want_lse.cpu().numpy().reshape(-1), "bf16", "grown %d" % step)
            pick = (np.arange(0, tree.n_leaves, 3), np.arange(0, tree.n_leaves, 3) % hq)
            oo, ol = oracle_rows(cfg, grown, k, v, q, *pick)
            compare(out.cpu().numpy()[pick], lse.cpu().numpy()[pick], oo, ol, "bf16", "grown %d" % step)


def test_replayed_from_a_graph():
    cfg = TreeConfig("group", 8, 64, 128, "bf16", 0, 0, 0, 0, 0, None, seed=77)
    tree = edge_tree(4160, sizes_for(520, 8, 3), 4)
    k, v, q = make_values_host(cfg, tree)
    kd, vd, qd = pool_to_device(k), pool_to_device(v), to_device(q)
    with make_ctx(cfg) as ctx:
        st = ctx.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node)
        assert ctx.item_rows() == 128
        want, want_lse, ws = attend(ctx, st, tree, kd, vd, qd)
        out, lse = torch.empty_like(want), torch.empty_like(want_lse)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ctx.decode(kd, vd, kd.shape[1], qd, out, lse, ws, ws.numel(), s.cuda_stream)
        for _ in range(3):
            out.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want) and torch.equal(lse, want_lse)
            attend(ctx, st, tree, kd, vd, qd)


@pytest.mark.parametrize("hq,d,rows,root", [
    (64, 128, 144, 12500), (64, 128, 208, 11000),  # one list per segment: 144 = 128 + 16, 208 = 3 x 64 + 16
    (64, 128, 520, 4160), (32, 128, 516, 4170), (16, 128, 520, 8320), (8, 128, 520, 16321), (64, 64, 584, 4160)])
def test_v_past_fp16_is_cut_off_for_no_more_rows_than_in_items_of_64(hq, d, rows, root):
    """Items of more than 16 query rows hold V in fp16, others as it is: with V = 99 840 and equal
    weights the output is the mean of 65 504 and 99 840 over the rows read in the one and in the other kind,
    exactly up to fp32 sums of at most 40 000 equal terms in steps of 32 (1 300 roundings at 2^-24)."""
    cfg = TreeConfig("group", 8, hq, d, "bf16", 0, 0, 0, 0, 0, None, seed=79)
    tree = edge_tree(root, sizes_for(rows, hq // 8, rows + hq), rows + d)
    k = torch.randn(8, tree.pool_tokens, d, device="cuda:0").to(torch.bfloat16)
    v = torch.full((8, tree.pool_tokens, d), 99840.0, dtype=torch.bfloat16, device="cuda:0")
    q = torch.zeros(tree.n_leaves, hq, d, dtype=torch.bfloat16, device="cuda:0")
    print("case group large v", hq, d, rows, root, flush=True)
    with make_ctx(cfg) as ctx, make_ctx(cfg, {"cascade_rows": 64}) as by64:
        st = ctx.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node)
        assert ctx.item_rows() == 128 and ctx.check().violations == 0
        out, lse, _ = attend(ctx, st, tree, k, v, q)
        st = by64.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node)
        want, want_lse, _ = attend(by64, st, tree, k, v, q)
        torch.cuda.synchronize()
    tol = 1300 * 2.0 ** -24
    assert bool((want < 99840 * (1 - tol)).any()) and bool((out <= 99840 * (1 + tol)).all())
    assert bool((out >= want * (1 - 2 * tol)).all())
    assert torch.allclose(lse, want_lse, atol=2 * tol, rtol=0)


def long_list_tree():
    """Step lists at the kernel's limit of 256: a root of 256 steps under 21 leaf queries, below it nodes of
    255 steps under 4 of them, of 258 (two lists) under 6 and of 256 with a short last one under 11; one
    leaf query of the first two ends a path of 100 and of 300 nodes of 1 to 3 rows that do not touch."""
    parent, n_tok, leaves = [-1], [8192], []
    for length, count, chain in ((8160, 4, 100), (8225, 6, 300), (8191, 11, 0)):
        parent.append(0)
        n_tok.append(length)
        top = len(parent) - 1
        for j in range(count):
            parent.append(top)
            n_tok.append(5 + 7 * j)
            for i in range(chain if j == 1 else 0):
                parent.append(len(parent) - 1)
                n_tok.append(1 + i % 3)
            leaves.append(len(parent) - 1)
    parent, n_tok = np.array(parent, np.int32), np.array(n_tok, np.int32)
    off = np.cumsum(n_tok.astype(np.int64) + 1) - n_tok - 1  # a free row behind every node
    return Tree(parent, off, n_tok, np.array(leaves, np.int32), int(n_tok.sum()) + n_tok.size,
                np.zeros(parent.size, np.int32))


@pytest.mark.parametrize("wave_items", [100000, 0])  # the paths' items: one wave's, a workgroup's
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("d", [128, 64])
def test_step_lists_of_up_to_256_steps(d, fp8, wave_items):
    cfg = TreeConfig("group", 8, 64, d, "bf16", 0, 0, 0, 0, 0, None, seed=83)
    tree = long_list_tree()
    print("case group long lists", d, fp8, wave_items, flush=True)
    k, v, q = make_values_fp8_host(cfg, tree, KS, VS) if fp8 else make_values_host(cfg, tree)
    with make_ctx(cfg, {"cascade_chunk": 100000, "stream_chunk": 100000, "wave_items": wave_items}) as ctx:
        if fp8:
            ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, KS, VS)
        st = ctx.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node)
        assert ctx.item_rows() == 128 and ctx.check().violations == 0
        # partials of a leaf query: the root's list, its node's one or two, its own one, the longer path's two
        assert st.n_partials == 4 * 3 + 6 * 4 + 1 + 11 * 3
        assert st.n_cascade_items == 2 + 1 + 2 + 1 + 22
        kd, vd, qd = pool_to_device(k), pool_to_device(v), to_device(q)
        out, lse, _ = attend(ctx, st, tree, kd, vd, qd)
        torch.cuda.synchronize()
    pick = (np.repeat(np.arange(21), 8), np.tile(np.arange(0, 64, 8), 21) + np.repeat(np.arange(21), 8) % 8)
    if fp8:
        oo, ol = oracle.tree_decode_attn_fp8kv(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node,
                                               k, v, KS, VS, q, 8, 64, d, rows=pick)
    else:
        oo, ol = oracle_rows(cfg, tree, k, v, q, *pick)
    compare(out.cpu().numpy()[pick], lse.cpu().numpy()[pick], oo, ol, "bf16", "long lists")
