"""More kv heads than a context holds factors for (64): every kernel that scales by a head's factor, against
the oracle with one scale for all heads.  Results of all heads are compared."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_13575_amd as ets
from workload import (Tree, TreeConfig, make_prefill_queries_host, make_values_fp8_host,
                      make_values_host)

from _gpu_util import compare, gpu_attn, gpu_prefill, make_ctx, oracle_full, oracle_prefill, pool_to_device, to_device

pytestmark = pytest.mark.gpu

KS, VS = 0.0123, 0.0217


def _tree(root, leaves, own):
    return Tree(np.array([-1] + [0] * leaves, np.int32),
                np.concatenate([[0], root + own * np.arange(leaves)]).astype(np.int64),
                np.array([root] + [own] * leaves, np.int32), np.arange(1, leaves + 1, dtype=np.int32),
                root + own * leaves)


# heads, head_dim, pools, options, (root, leaf steps, their rows), query rows per item of the shared-node kernel
CASES = [
    (65, 64, "f32", {}, (60, 3, 20), 0),                       # one launch
    (70, 128, "f32", {"stream_chunk": 64}, (60, 3, 20), 0),    # per-leaf kernel and merge
    (65, 128, "bf16", {}, (300, 3, 40), 64), (66, 64, "bf16", {"fuse_merge": 1}, (300, 3, 40), 64),
    (65, 128, "bf16", {"mfma": 0}, (300, 3, 40), 0),
    (65, 128, "e4m3", {}, (300, 3, 40), 64), (65, 64, "e4m3", {"fuse_merge": 1}, (300, 3, 40), 64),
    (65, 128, "e4m3", {"wide_rows": 1}, (300, 40, 8), 64),
    (80, 64, "e4m3", {}, (1700, 128, 4), 128),                 # the group kernel
]


@pytest.mark.parametrize("heads,d,kv,options,shape,rows", CASES)
def test_decode(heads, d, kv, options, shape, rows):
    tree = _tree(*shape)
    cfg = TreeConfig("heads", heads, heads, d, "f32" if kv == "f32" else "bf16", 0, 0, 0, 0, 0, None, seed=heads + d)
    k, v, q = make_values_fp8_host(cfg, tree, KS, VS) if kv == "e4m3" else make_values_host(cfg, tree)
    print("case many heads", heads, d, kv, options, shape, flush=True)
    with make_ctx(cfg, options) as ctx:
        if kv == "e4m3":
            ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, KS, VS)
        out, lse, st = gpu_attn(ctx, tree, pool_to_device(k), pool_to_device(v), to_device(q))
        assert ctx.item_rows() == rows and st.merge_fused == options.get("fuse_merge", 0)
        assert (st.n_wide_items > 0) == ("wide_rows" in options)
    if kv == "e4m3":
        oo, ol = oracle.tree_decode_attn_fp8kv(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node, k, v,
                                               KS, VS, q, heads, heads, d)
    else:
        oo, ol = oracle_full(cfg, tree, k, v, q)
    compare(out.cpu().numpy().reshape(-1, d), lse.cpu().numpy().reshape(-1), oo.reshape(-1, d), ol.reshape(-1),
            cfg.dtype, "many heads %s" % kv)


@pytest.mark.parametrize("kv", ["bf16", "e4m3"])
def test_prefill(kv):
    tree = _tree(300, 2, 40)
    cfg = TreeConfig("heads", 65, 65, 128, "bf16", 0, 0, 0, 0, 0, None, seed=7)
    k, v = (make_values_fp8_host(cfg, tree, KS, VS) if kv == "e4m3" else make_values_host(cfg, tree))[:2]
    q = make_prefill_queries_host(cfg, tree)
    print("case many heads prefill", kv, flush=True)
    with make_ctx(cfg) as ctx:
        if kv == "e4m3":
            ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, KS, VS)
        out, lse, _ = gpu_prefill(ctx, tree, pool_to_device(k), pool_to_device(v), to_device(q))
    if kv == "e4m3":
        oo, ol = oracle.tree_prefill_attn_fp8kv(tree.parent, tree.tok_offset, tree.n_tokens, tree.leaf_node, k, v,
                                                KS, VS, q, 65, 65, 128)
    else:
        oo, ol = oracle_prefill(cfg, tree, k, v, q)
    compare(out.cpu().numpy().reshape(-1, 128), lse.cpu().numpy().reshape(-1), oo.reshape(-1, 128), ol.reshape(-1),
            "bf16", "many heads prefill %s" % kv)
