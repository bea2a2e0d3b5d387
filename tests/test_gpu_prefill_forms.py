"""Step prefill with work items of 128 and of 256 query rows (and, among the latter, last blocks
of at most 128 rows, which are walked like the former): the same trees through both, over bf16
pools and pools of E4M3 codes, every row of the first copy of the leaf queries against the oracle.
The planner picks the size by the number of items, so the leaf queries are repeated until it
picks the one asked for; the copies have to give the same bits."""
import numpy as np
import pytest
import torch

import paper_2502_13575_amd as ets
import oracle
from workload import (Tree, TreeConfig, make_prefill_queries_host, make_values_fp8_host,
                      make_values_host, random_tree)

from _gpu_util import compare, make_ctx, oracle_prefill, pool_to_device, to_device

pytestmark = pytest.mark.gpu

KS, VS = 0.0123, 0.0217


def _edge(n):
    # a root of 45 rows (ragged second run), a child of n rows; queries on both
    return Tree(np.array([-1, 0], np.int32), np.array([n, 0], np.int64),
                np.array([45, n], np.int32), np.array([1, 0], np.int32), n + 45)


def _scattered():
    # 700 one-token ancestors that do not merge: the descriptor ring is refilled
    n = 700
    n_tok = np.ones(n, np.int32)
    n_tok[-1] = 37
    off = (np.arange(n, dtype=np.int64) * 7919) % n * 40
    return Tree(np.arange(-1, n - 1, dtype=np.int32), off, n_tok, np.array([n - 1, 350], np.int32),
                int(off.max()) + 40)


def _long():
    return Tree(np.array([-1, 0], np.int32), np.array([0, 9000], np.int64),
                np.array([9000, 40], np.int32), np.array([1], np.int32), 9040)


CASES = {
    "fuzz0": (2, 8, lambda: random_tree(40, n_nodes=30, n_leaves=7, max_tokens=70, p_empty=0.15)),
    "fuzz1": (2, 16, lambda: random_tree(41, n_nodes=30, n_leaves=7, max_tokens=150, p_empty=0.15)),
    "fuzz2": (3, 12, lambda: random_tree(42, n_nodes=30, n_leaves=9, max_tokens=150, p_empty=0.15)),
    "fuzz3": (1, 2, lambda: random_tree(43, n_nodes=20, n_leaves=6, max_tokens=300)),
    "fuzz4": (1, 1, lambda: random_tree(44, n_nodes=20, n_leaves=6, max_tokens=500)),
    "fuzz5": (8, 32, lambda: random_tree(45, n_nodes=30, n_leaves=5, max_tokens=90, p_empty=0.15)),
    "scattered": (1, 4, _scattered), "long": (1, 4, _long),
}
# lengths around the edges of waves, blocks and runs of both item sizes (4 query heads per kv head)
for _n in (1, 8, 9, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 95, 96, 97, 127, 128, 129):
    CASES["edge%d" % _n] = (2, 8, lambda n=_n: _edge(n))


@pytest.mark.parametrize("kv", ["bf16", "e4m3"])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("name", sorted(CASES))
def test_prefill_both_item_sizes(name, rows, kv):
    hkv, hq, make = CASES[name]
    tree = make()
    cfg = TreeConfig("forms", hkv, hq, 128, "bf16", 0, 0, 0, 0, 0, None, seed=1000 + len(name))
    if kv == "bf16":
        k, v, _ = make_values_host(cfg, tree)
    else:
        k, v, _ = make_values_fp8_host(cfg, tree, KS, VS)
    q = make_prefill_queries_host(cfg, tree)
    n = q.shape[0]
    with make_ctx(cfg) as ctx:
        if kv == "e4m3":
            ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, KS, VS)
        for copies in range(1, 400):
            st = ctx.plan_prefill(tree.parent, tree.tok_offset, tree.n_tokens,
                                  np.tile(tree.leaf_node, copies))
            if st.rows_per_item == rows:
                break
        assert st.rows_per_item == rows and st.n_q_rows == n * copies
        print("case forms", name, kv, "items", st.n_items, "of", rows, "copies", copies, flush=True)
        kd, vd = pool_to_device(k), pool_to_device(v)
        qd = to_device(q).repeat(copies, 1, 1)
        out = torch.full((n * copies, hq, 128), float("nan"), device="cuda:0")
        lse = torch.full((n * copies, hq), float("nan"), device="cuda:0")
        ctx.prefill(kd, vd, kd.shape[1], qd, out, lse)
        torch.cuda.synchronize()
    out, lse = out.view(copies, n, hq, 128), lse.view(copies, n, hq)
    assert torch.equal(out, out[:1].expand_as(out)) and torch.equal(lse, lse[:1].expand_as(lse))
    if kv == "bf16":
        oo, ol = oracle_prefill(cfg, tree, k, v, q)
    else:
        oo, ol = oracle.tree_prefill_attn_fp8kv(tree.parent, tree.tok_offset, tree.n_tokens,
                                                tree.leaf_node, k, v, KS, VS, q, hkv, hq, 128)
    compare(out[0].cpu().numpy().reshape(-1, 128), lse[0].cpu().numpy().reshape(-1),
            oo.reshape(-1, 128), ol.reshape(-1), "bf16", "forms %s %s %d" % (name, kv, rows))
