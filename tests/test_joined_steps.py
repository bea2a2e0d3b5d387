"""Steps of 32 rows in which the rest of one piece of a run list is joined with the start of the next:
pieces behind and in front of one another in the pool, steps that stay short, pieces too short or too
far apart to be joined.  On the host the step counts and the rows seen; on the GPU every result
against the oracle, with pools whose rows outside the tree hold NaN (a row past the end of a joined
step has to read as zero, not as its neighbour)."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2502_13575_amd as ets
from workload import Tree, TreeConfig, make_prefill_queries_host, make_values_fp8_host, make_values_host

from _gpu_util import (compare, gpu_attn, gpu_prefill, make_ctx, oracle_full, oracle_prefill, pool_to_device,
                       to_device)

KS, VS = 0.0123, 0.0217
OWN = 40
ROOT = 192  # six steps, which step prefill requests ahead of its walk and keeps apart
FAR = 1 << 23


def _tree(lengths, order, leaves=1, room=0):
    """A chain of a node of ROOT rows and nodes of these lengths, with `leaves` steps of OWN rows below it and
    three unused rows between any two nodes (and `room` behind a leaf step); `order`: where a node lies behind the one above it in the pool."""
    lengths = (ROOT,) + tuple(lengths)
    n = len(lengths)
    n_tok = np.array(list(lengths) + [OWN] * leaves, np.int32)
    parent = np.array([-1] + list(range(n - 1)) + [n - 1] * leaves, np.int32)
    place = {"behind": np.arange(n), "front": np.arange(n)[::-1],
             "mixed": np.random.default_rng(n).permutation(n)}[order]
    off = np.zeros(n + leaves, np.int64)
    at = 0
    for i in list(np.argsort(place)) + list(range(n, n + leaves)):
        off[i] = at
        at += n_tok[i] + 3 + (room if i >= n else 0)
    return Tree(parent, off, n_tok, np.arange(n, n + leaves, dtype=np.int32), int(at))


# lengths of the ancestors below the root, order in the pool, steps they take
CASES = [
    ((45, 45, 45), "behind", 5), ((45, 45, 45), "front", 5),    # 32, 13 + 19, 26 + 6, 32, 7
    ((20, 9, 40), "behind", 3),                                  # 20 + 9 (short), 32, 8
    ((20, 9, 40), "front", 3),                                   # 20, 9 + 23, 17
    ((10, 10), "behind", 1), ((10, 10), "front", 2),             # a short step is joined forwards only
    ((7, 7, 7), "behind", 2), ((7, 25, 7), "front", 2),          # two pieces to a step
    ((3, 4, 1, 6), "behind", 4), ((4, 4, 7), "behind", 2),       # fewer than eight rows stay apart
    ((1, 31, 1, 31), "front", 2), ((31, 1, 31, 1), "front", 2),  # joins at the edges of a step
    ((16, 16, 16, 48), "front", 3), ((33, 15, 47, 1), "mixed", None),
    (tuple(range(1, 60)), "mixed", None), (tuple(range(60, 0, -1)), "behind", None),
    ((100,) * 120, "mixed", 375),                                # the descriptor ring is refilled
]


@pytest.mark.parametrize("lengths,order,steps", CASES)
def test_prefill_steps_and_rows(lengths, order, steps):
    t = _tree(lengths, order)
    with ets.Context(1, 4, 128, ets.ETS_BF16, -1) as ctx:
        st = ctx.plan_prefill(t.parent, t.tok_offset, t.n_tokens, t.leaf_node)
        if steps is not None:
            assert st.n_runs == ROOT // 32 + steps + -(-OWN // 32)
        for tok in (0, 31, OWN - 1):
            want = oracle.visible_rows(t.parent, t.tok_offset, t.n_tokens, int(t.leaf_node[0]), tok + 1)
            assert np.array_equal(ctx.prefill_cover(0, tok), want)
        assert ctx.check().violations == 0


LIMIT = 1 << 22  # rows between the pieces, at most


@pytest.mark.parametrize("back", [False, True])
@pytest.mark.parametrize("beyond", [0, 1])
def test_the_largest_gap(back, beyond):
    """205 rows (the seventh step has 13), then 45: joined 13 + 19 up to the limit, both ways, not beyond."""
    t = _far_tree(back, beyond)
    with ets.Context(1, 4, 128, ets.ETS_BF16, -1) as ctx:
        st = ctx.plan_prefill(t.parent, t.tok_offset, t.n_tokens, t.leaf_node)
        assert st.n_runs == 10 + beyond
        ctx.plan(t.parent, t.tok_offset, t.n_tokens, t.leaf_node, ets.ETS_PLAN_FLAT)
        assert ctx.check().violations == 0
        want = oracle.visible_rows(t.parent, t.tok_offset, t.n_tokens, 2, OWN)
        assert np.array_equal(ctx.prefill_cover(0, OWN - 1), want) and np.array_equal(ctx.leaf_cover(0)[0], want)


def _far_tree(back, beyond=0):
    first = (LIMIT + beyond - 205) if back else 0
    second = 0 if back else 205 + LIMIT + beyond
    return Tree(np.array([-1, 0, 1], np.int32), np.array([first, second, LIMIT + 400], np.int64),
                np.array([205, 45, OWN], np.int32), np.array([2], np.int32), LIMIT + 400 + OWN)


def test_pieces_too_far_apart_are_not_joined():
    n = ROOT + 45
    for gap, runs in ((FAR // 4, 3), (FAR, 4)):  # 45 + 45 rows: 32, 13 + 19, 26, or 32, 13, 32, 13
        for off in ([0, n + gap, 4 * FAR], [n + gap, 0, 4 * FAR]):
            with ets.Context(1, 4, 128, ets.ETS_BF16, -1) as ctx:
                st = ctx.plan_prefill(np.array([-1, 0, 1], np.int32), np.array(off, np.int64),
                                      np.array([n, 45, 8], np.int32), np.array([2], np.int32))
                assert st.n_runs == ROOT // 32 + runs + 1 and ctx.check().violations == 0


PLAN_MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "prefill_plan.h"
// A chain of nodes of these many rows with five unused rows between any two, and one leaf step of 40 rows
// below it; prints whether the plan's runs may be joined, how many are, and how many runs there are.
int main(int argc, char** argv) {
    std::vector<int32_t> parent, rows;
    std::vector<int64_t> off;
    int64_t at = 0;
    for (int i = 1; i <= argc; ++i) {
        parent.push_back(i - 2);
        rows.push_back(i < argc ? std::atoi(argv[i]) : 40);
        off.push_back(at);
        at += rows.back() + 5;
    }
    const int32_t leaf = argc - 1;
    const ets_shape shape{1, 4, 128, ETS_BF16, 0.f};
    const ets_tree tree{argc, parent.data(), off.data(), rows.data(), 1, &leaf};
    ets::PrefillPlan p;
    if (ets::build_prefill_plan(shape, tree, p, 2) != ETS_OK) return 1;
    int joined = 0;
    for (const ets::Run& r : p.runs) joined += r.join != 0;
    std::printf("%d %d %d\n", (int)p.joins, joined, (int)p.runs.size());
    return 0;
}
"""


def test_prefill_joins_are_kept_where_they_save_runs(tmp_path):
    """The kernel's loop that takes joined runs is the longer one: a plan in which no run is saved, or too few,
    has no joined run and goes to the other loop."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    csrc = os.path.join(root, "paper_2502_13575_amd", "csrc")
    main, exe = tmp_path / "main.cpp", str(tmp_path / "plan")
    main.write_text(PLAN_MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + csrc, "-I" + os.path.join(root, "include"), str(main),
                    os.path.join(csrc, "prefill_plan.cpp"), os.path.join(csrc, "plan.cpp"), "-o", exe], check=True)
    for rows, want in [([192, 40, 63], "0 0 12"),           # joined 32, 8 + 24, 32, 7: four runs either way
                       ([192, 20, 20], "0 0 10"),           # joined 20 + 12, 8: two either way
                       ([192, 45, 45, 45], "1 2 13"),       # 32, 13 + 19, 26 + 6, 32, 7 instead of six
                       ([192] + [60] * 32, "0 0 72"),       # every second run 28 + 4: none saved in 64
                       ([192] + [48] * 8, "1 4 20")]:       # 32, 16 + 16, 32: 12 instead of 16
        out = subprocess.run([exe] + [str(x) for x in rows], check=True, capture_output=True, text=True).stdout
        assert out.strip() == want, rows


def _poisoned(x, tree):
    """The same pool with NaN in every row that no node holds."""
    used = np.zeros(x.shape[0], bool)
    for o, n in zip(tree.tok_offset, tree.n_tokens):
        used[o:o + n] = True
    x = x.copy()
    x[~used] = 0x7F if x.dtype == np.uint8 else 0x7FC0
    return x


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "e4m3"])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("lengths,order", [c[:2] for c in CASES])
def test_prefill_over_joined_steps(lengths, order, rows, kv):
    tree = _tree(lengths, order)
    cfg = TreeConfig("joined", 2, 8, 128, "bf16", 0, 0, 0, 0, 0, None, seed=len(lengths) + rows)
    k, v = (make_values_host(cfg, tree) if kv == "bf16" else make_values_fp8_host(cfg, tree, KS, VS))[:2]
    k, v = _poisoned(k, tree), _poisoned(v, tree)
    q = make_prefill_queries_host(cfg, tree)
    n = q.shape[0]
    with make_ctx(cfg) as ctx:
        if kv == "e4m3":
            ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, KS, VS)
        for copies in range(1, 400):  # the planner picks the item size by the number of items
            st = ctx.plan_prefill(tree.parent, tree.tok_offset, tree.n_tokens, np.tile(tree.leaf_node, copies))
            if st.rows_per_item == rows:
                break
        assert st.rows_per_item == rows and ctx.check().violations == 0
        print("case joined prefill", lengths[:4], order, rows, kv, flush=True)
        kd, vd = pool_to_device(k), pool_to_device(v)
        out = torch.full((n * copies, 8, 128), float("nan"), device="cuda:0")
        lse = torch.full((n * copies, 8), float("nan"), device="cuda:0")
        ctx.prefill(kd, vd, kd.shape[1], to_device(q).repeat(copies, 1, 1), out, lse)
        torch.cuda.synchronize()
    if kv == "bf16":
        oo, ol = oracle_prefill(cfg, tree, k, v, q)
    else:
        oo, ol = oracle.tree_prefill_attn_fp8kv(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node,
                                                k, v, KS, VS, q, 2, 8, 128)
    compare(out[-n:].cpu().numpy().reshape(-1, 128), lse[-n:].cpu().numpy().reshape(-1),
            oo.reshape(-1, 128), ol.reshape(-1), "bf16", "joined prefill %s" % kv)


@pytest.mark.parametrize("leaves,options", [(1, {}), (9, {}), (9, {"cascade_chunk": 64}), (9, {"stream_chunk": 64}),
                                            (9, {"cascade_min_leaves": 0}), (9, {"wide_rows": 16})])
@pytest.mark.parametrize("lengths,order", [c[:2] for c in CASES])
def test_decode_rows_and_growth(lengths, order, leaves, options):
    """Whatever kernel reads the lists, and after 36 tokens, past the room they keep for growth."""
    t = _tree(lengths, order, leaves, room=40)
    n_tokens = t.n_tokens.copy()
    with ets.Context(2, 8, 128, ets.ETS_BF16, -1) as ctx:
        for k, x in options.items():
            ctx.set_option(k, x)
        ctx.plan(t.parent, t.tok_offset, n_tokens, t.leaf_node)
        for step in range(37):
            if step in (0, 1, 9, 36):
                assert ctx.check().violations == 0
                for l in {0, leaves - 1}:
                    want = oracle.visible_rows(t.parent, t.tok_offset, n_tokens, int(t.leaf_node[l]),
                                               int(n_tokens[t.leaf_node[l]]))
                    assert np.array_equal(ctx.leaf_cover(l)[0], want)
            ctx.plan_advance()
            n_tokens[t.leaf_node] += 1


def _decode(cfg, tree, kv, options, mode):
    """One decode call on poisoned pools against the oracle."""
    hkv, hq, d = cfg.n_kv_heads, cfg.n_q_heads, cfg.head_dim
    k, v, q = make_values_host(cfg, tree) if kv == "bf16" else make_values_fp8_host(cfg, tree, KS, VS)
    k, v = _poisoned(k, tree), _poisoned(v, tree)
    with make_ctx(cfg, options) as ctx:
        if kv == "e4m3":
            ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, KS, VS)
        st = ctx.plan(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node, mode)
        assert ctx.check().violations == 0
        kd, vd = pool_to_device(k), pool_to_device(v)
        out = torch.full((tree.n_leaves, hq, d), float("nan"), device="cuda:0")
        lse = torch.full((tree.n_leaves, hq), float("nan"), device="cuda:0")
        ws = torch.empty(max(st.workspace_bytes, 16), dtype=torch.uint8, device="cuda:0")
        ctx.decode(kd, vd, kd.shape[1], to_device(q), out, lse, ws, ws.numel())
        torch.cuda.synchronize()
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    args = (tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node, k, v)
    if kv == "bf16":
        oo, ol = oracle.tree_decode_attn(*args, q, hkv, hq, d)
    else:
        oo, ol = oracle.tree_decode_attn_fp8kv(*args, KS, VS, q, hkv, hq, d)
    compare(out.reshape(-1, d), lse.reshape(-1), oo.reshape(-1, d), ol.reshape(-1), "bf16", "joined decode")


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "e4m3"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("leaves,mode,options", [
    (1, "tree", {}),                       # one leaf query (small items, one wave each: test_growth_of_joined_tails)
    (3, "flat", {"wave_items": 0}),        # at most 16 query rows, four waves
    (9, "tree", {}), (40, "tree", {"cascade_chunk": 96}),  # row-parallel
    (9, "tree", {"fuse_merge": 1})])
@pytest.mark.parametrize("lengths,order", [c[:2] for c in CASES if len(c[0]) < 100])
def test_decode_over_joined_steps(lengths, order, leaves, mode, options, d, kv):
    tree = _tree(lengths, order, leaves)
    cfg = TreeConfig("joined", 2, 8, d, "bf16", 0, 0, 0, 0, 0, None, seed=len(lengths) + leaves)
    print("case joined decode", lengths[:4], order, leaves, mode, options, d, kv, flush=True)
    _decode(cfg, tree, kv, options, ets.ETS_PLAN_TREE if mode == "tree" else ets.ETS_PLAN_FLAT)


@pytest.mark.gpu
@pytest.mark.parametrize("back", [False, True])
def test_the_largest_gap_on_the_device(back):
    """Decode and step prefill with pieces a GiB apart in the pool; whatever no node holds is NaN."""
    far = _far_tree(back)
    n_tok = far.n_tokens
    near = Tree(far.parent, np.array([0, 205, 250], np.int64), n_tok, far.leaf_node, 250 + OWN)  # the same rows
    cfg = TreeConfig("far", 1, 4, 128, "bf16", 0, 0, 0, 0, 0, None, seed=4)
    k, v, q = make_values_host(cfg, near)
    qs = make_prefill_queries_host(cfg, near)
    print("case largest gap", back, flush=True)
    pools = []
    for x in (k, v):
        pool = torch.full((1, far.pool_tokens, 128), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        rows = pool_to_device(x)
        for node in range(3):
            at, a, n = int(far.tok_offset[node]), int(near.tok_offset[node]), int(n_tok[node])
            pool[:, at:at + n] = rows[:, a:a + n]
        pools.append(pool)
    with make_ctx(cfg) as ctx:
        out, lse, _ = gpu_attn(ctx, far, *pools, to_device(q), ets.ETS_PLAN_FLAT)
        pout, plse, st = gpu_prefill(ctx, far, *pools, to_device(qs))
        assert st.n_runs == 10 and ctx.check().violations == 0
    for got, got_lse, want in ((out, lse, oracle_full(cfg, near, k, v, q)),
                               (pout, plse, oracle_prefill(cfg, near, k, v, qs))):
        compare(got.cpu().numpy().reshape(-1, 128), got_lse.cpu().numpy().reshape(-1), want[0].reshape(-1, 128),
                want[1].reshape(-1), "bf16", "largest gap")


GROWING = [(205, 10, False), (205, 19, False), (237, 10, False), (205, 19, True)]  # rows above, own, own in front


@pytest.mark.gpu
@pytest.mark.parametrize("d,kv", [(64, "bf16"), (128, "bf16"), (128, "e4m3")])
@pytest.mark.parametrize("leaves,mode,options,small", [
    (3, "flat", {}, False), (3, "flat", {"stream_chunk": 64}, False),  # four waves to an item
    (9, "tree", {}, False), (9, "tree", {"cascade_chunk": 64, "fuse_merge": 1}, False),  # row-parallel
    (5, "flat", {}, True), (5, "flat", {"stream_chunk": 64}, True)])   # one wave to an item
def test_growth_of_joined_tails(leaves, mode, options, small, d, kv):
    """Leaf queries on a node whose last step is joined with the rows above it: 13 + 10 rows fill up to 32 and
    go on in the spare step, 13 + 19 are full from the start; with chunks of 64 rows that step is the first of
    its item (205 rows above) or the second (237), of which the start table holds copies.  After 33 tokens the
    tree is planned again.  Items of one wave need a call whose bytes take long: another search in the same
    forest, of as many rows as the planner asks for."""
    hkv, hq = 2, 8
    cfg = TreeConfig("growth", hkv, hq, d, "bf16", 0, 0, 0, 0, 0, None, seed=leaves + d)
    for above, own, front in GROWING:
        print("case growth", above, own, front, leaves, mode, options, small, d, kv, flush=True)
        room = own + 40
        off = np.array([room + 3, 0] if front else [0, above + 3], np.int64)
        near = Tree(np.array([-1, 0], np.int32), off, np.array([above, own], np.int32), np.ones(leaves, np.int32),
                    above + 3 + room)
        k, v, q = make_values_host(cfg, near) if kv == "bf16" else make_values_fp8_host(cfg, near, KS, VS)
        k, v = _poisoned(k, near), _poisoned(v, near)
        kd, vd = pool_to_device(k), pool_to_device(v)
        parent, n_tok, leaf_node = near.parent, near.n_tokens, near.leaf_node
        qd = to_device(q)
        if small:
            other = 550000 * 128 // d * 2
            parent, n_tok = np.append(parent, np.int32(-1)), np.append(n_tok, np.int32(other))
            off, leaf_node = np.append(off, near.pool_tokens), np.append(leaf_node, np.int32(2))
            qd = torch.cat([qd, qd[:1]])

            def wider(x):
                y = torch.empty((hkv, near.pool_tokens + other + 40, d), dtype=x.dtype, device="cuda:0")
                y.normal_() if kv == "bf16" else y.random_(0, 120)
                y[:, :near.pool_tokens] = x
                return y
            kd, vd = wider(kd), wider(vd)
        with make_ctx(cfg, options) as ctx:
            if kv == "e4m3":
                ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, KS, VS)
            st = ctx.plan(parent, off, n_tok, leaf_node, ets.ETS_PLAN_TREE if mode == "tree" else ets.ETS_PLAN_FLAT)
            if small:  # the longest item that one wave takes
                ns = st.unique_kv_bytes * (2 if kv == "e4m3" else 1) // 5500
                assert ns // 4 // 2500 * 16 >= above + own + 40
            grown, replans = near.n_tokens, 0
            for step in range(37):
                if step > 0:
                    fresh = Tree(near.parent, near.tok_offset, near.n_tokens, leaf_node, leaf_node.size)
                    kn, vn = (make_values_host(cfg, fresh, step) if kv == "bf16" else
                              make_values_fp8_host(cfg, fresh, KS, VS, step))[:2]
                    replans += bool(ctx.plan_advance())
                    ctx.kv_append(kd, vd, kd.shape[1], to_device(kn), to_device(vn))
                    grown = oracle.append_kv(near.tok_offset, grown, near.leaf_node, k, v, kn[:leaves], vn[:leaves])
                if step not in (0, 1, 2, 8, 9, 10, 22, 23, 32, 33, 36):
                    continue
                assert ctx.check().violations == 0
                L = leaf_node.size
                out = torch.full((L, hq, d), float("nan"), device="cuda:0")
                lse = torch.full((L, hq), float("nan"), device="cuda:0")
                ws = torch.empty(ctx.stats().workspace_bytes, dtype=torch.uint8, device="cuda:0")
                ctx.decode(kd, vd, kd.shape[1], qd, out, lse, ws, ws.numel())
                torch.cuda.synchronize()
                args = (near.parent, near.tok_offset, grown, near.leaf_node, k, v)
                if kv == "bf16":
                    oo, ol = oracle.tree_decode_attn(*args, q, hkv, hq, d)
                else:
                    oo, ol = oracle.tree_decode_attn_fp8kv(*args, KS, VS, q, hkv, hq, d)
                compare(out[:leaves].cpu().numpy().reshape(-1, d), lse[:leaves].cpu().numpy().reshape(-1),
                        oo.reshape(-1, d), ol.reshape(-1), "bf16", "growth %d" % step)
            assert replans == 1
