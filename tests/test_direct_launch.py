"""Small calls over fp32 pools in one launch (every path cut into at most sixteen items, merged in the
workgroup): the edges of its items and of the rule, empty paths, growth past the plan, bf16 results."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_13575_amd as ets
from workload import Tree, TreeConfig, make_values_host

from _gpu_util import compare, gpu_attn, make_ctx, oracle_full, pool_to_device, to_device


def _tree(root, lengths, room=0):
    """A root and one leaf step of each of `lengths` rows below it, one unused row between nodes."""
    n_tok = np.array([root] + list(lengths), np.int32)
    gaps = np.array([1] + [1 + room] * len(lengths))
    off = (np.cumsum(n_tok + gaps) - n_tok - gaps).astype(np.int64)
    return Tree(np.array([-1] + [0] * len(lengths), np.int32), off, n_tok,
                np.arange(1, len(lengths) + 1, dtype=np.int32), int((n_tok + gaps).sum()))


# root, leaf steps, partial results of the leaf query with the longest path
CASES = [(0, (1, 0, 16), 1), (0, (17, 3), 2), (200, (56, 0, 1), 16), (255, (1, 2, 17), 9),
         (480, (32, 31, 1), 16), (300, (7,) * 40, 10), (481, (32,), None)]


@pytest.mark.parametrize("root,lengths,most", CASES)
def test_items(root, lengths, most):
    t = _tree(root, lengths)
    with ets.Context(2, 4, 64, ets.ETS_F32, -1) as ctx:
        ctx.plan(t.parent, t.tok_offset, t.n_tokens, t.leaf_node)
        assert ctx.check().violations == 0
        counts = []
        for l in range(t.n_leaves):
            rows, n = ctx.leaf_cover(l)
            assert np.array_equal(rows, np.concatenate(
                [np.arange(t.tok_offset[x], t.tok_offset[x] + t.n_tokens[x]) for x in (0, l + 1)]))
            counts.append(n)
        # beyond 512 rows: items of 64 rows and a second launch
        assert max(counts) == (most if most is not None else -(-(root + max(lengths)) // 64))


# heads, head_dim, longest path in one launch; with paths of 40 rows the most leaf queries with items of 16 rows
# (three each) and of 32 (two each) in one launch
RULE = [((4, 4, 64), 512, 833, 1875), ((4, 8, 128), 512, 416, 937), ((2, 8, 64), 416, 416, 937),
        ((2, 8, 128), 416, 416, 937), ((1, 8, 64), 320, 833, 937), ((1, 8, 128), 400, 833, 937)]


def _items(tree, hkv, hq, d):
    with ets.Context(hkv, hq, d, ets.ETS_F32, -1) as ctx:
        st = ctx.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node)
        assert ctx.check().violations == 0 and st.workspace_bytes <= ets.ETS_STATIC_SCRATCH_BYTES
        return ctx.leaf_cover(tree.n_leaves - 1)[1]


@pytest.mark.parametrize("heads,longest,leaves16,leaves32", RULE)
def test_where_the_rule_ends(heads, longest, leaves16, leaves32):
    for rows, items in ((256, 16), (257, 9), (longest, -(-longest // 32)), (longest + 1, -(-(longest + 1) // 64))):
        assert _items(_tree(rows - 30, (30,)), *heads) == items, rows
    for leaves, items in ((leaves16, 3), (leaves16 + 1, 2), (leaves32, 2), (leaves32 + 1, 1)):
        assert _items(_tree(30, (10,) * leaves), *heads) == items, leaves


@pytest.mark.gpu
@pytest.mark.parametrize("hkv,hq,d,leaves", [(1, 8, 128, 833), (1, 8, 128, 937), (2, 8, 64, 417), (4, 4, 64, 1875)])
def test_many_leaves_against_the_oracle(hkv, hq, d, leaves):
    """Calls at the upper end: several workgroups of two or three waves to a compute unit."""
    tree = _tree(30, (10,) * leaves)
    cfg = TreeConfig("direct", hkv, hq, d, "f32", 0, 0, 0, 0, 0, None, seed=leaves + hq)
    print("case direct leaves", hkv, hq, d, leaves, flush=True)
    k, v, q = make_values_host(cfg, tree)
    with make_ctx(cfg) as ctx:
        out, lse, _ = gpu_attn(ctx, tree, pool_to_device(k), pool_to_device(v), to_device(q))
    oo, ol = oracle_full(cfg, tree, k, v, q)
    compare(out.cpu().numpy().reshape(-1, d), lse.cpu().numpy().reshape(-1), oo.reshape(-1, d), ol.reshape(-1),
            "f32", "direct leaves")


@pytest.mark.gpu
@pytest.mark.parametrize("hkv,hq,d", [(1, 1, 64), (2, 4, 64), (1, 4, 128), (3, 24, 128), (2, 16, 64)])
@pytest.mark.parametrize("root,lengths", [c[:2] for c in CASES])
def test_direct_against_the_oracle(root, lengths, hkv, hq, d):
    tree = _tree(root, lengths, room=40)
    cfg = TreeConfig("direct", hkv, hq, d, "f32", 0, 0, 0, 0, 0, None, seed=root + hq)
    print("case direct", root, lengths[:4], hkv, hq, d, flush=True)
    k, v, q = make_values_host(cfg, tree)
    kd, vd, qd = pool_to_device(k), pool_to_device(v), to_device(q)
    n_tokens = tree.n_tokens.copy()
    with make_ctx(cfg) as ctx:
        st = ctx.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node)
        ws = torch.empty(max(st.workspace_bytes, 16) + 4096, dtype=torch.uint8, device="cuda:0")
        out = torch.full((tree.n_leaves, hq, d), float("nan"), device="cuda:0")
        lse = torch.full((tree.n_leaves, hq), float("nan"), device="cuda:0")
        half = torch.empty_like(out, dtype=torch.bfloat16)
        for step in range(0, 36, 7):
            ctx.decode(kd, vd, kd.shape[1], qd, out, lse, ws, ws.numel())
            torch.cuda.synchronize()
            grown = Tree(tree.parent, tree.tok_offset, n_tokens, tree.leaf_node, tree.pool_tokens)
            oo, ol = oracle_full(cfg, grown, k, v, q)
            compare(out.cpu().numpy().reshape(-1, d), lse.cpu().numpy().reshape(-1), oo.reshape(-1, d),
                    ol.reshape(-1), "f32", "direct %d" % step)
            if step == 0:
                ctx.set_option("out_bf16", 1)
                ctx.decode(kd, vd, kd.shape[1], qd, half, lse, ws, ws.numel())
                torch.cuda.synchronize()
                assert torch.equal(half, out.to(torch.bfloat16))
                ctx.set_option("out_bf16", 0)
            if min(lengths) == 0:
                break  # a growing node without a row has the tree planned again
            for _ in range(7):
                ctx.plan_advance()
                n_tokens[np.unique(tree.leaf_node)] += 1
