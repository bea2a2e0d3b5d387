"""Plans of the group kernel (many query rows per shared row) on the host: leaf queries cut into
groups, segments of a group joined into one list.  Indexing against the oracle's walk, the replay of
the kernel's table reads, and both after decode-step advances, over random forests whose 64 kv heads
bring them over the planner's line."""
import numpy as np
import pytest

import oracle
import paper_2502_13575_amd as ets
from workload import random_tree, with_growth_room

SHAPES = [(64, 512, 128), (64, 256, 64), (64, 128, 128), (64, 64, 64)]


def _plan(ctx, t):
    return ctx.plan(t.parent, t.tok_offset, t.n_tokens, t.leaf_node)


def _covers(ctx, t, n_tokens):
    optr, onodes = oracle.paths(t.parent, t.leaf_node)
    total = 0
    for l in range(t.n_leaves):
        rows, n = ctx.leaf_cover(l)
        nodes = onodes[optr[l]:optr[l + 1]]
        want = np.concatenate([np.zeros(0, np.int64)] +
                              [np.arange(t.tok_offset[x], t.tok_offset[x] + n_tokens[x]) for x in nodes])
        assert np.array_equal(np.sort(rows), np.sort(want)), l
        total += n
    assert total == ctx.stats().n_partials


@pytest.mark.parametrize("block", range(8))
def test_group_plans_of_random_forests(block):
    joined = apart = 0
    for seed in range(31000 + 30 * block, 31030 + 30 * block):
        r = np.random.default_rng(seed)
        t = random_tree(seed, n_nodes=int(r.integers(20, 160)), n_leaves=int(r.integers(40, 300)),
                        max_tokens=int(r.choice([200, 1000, 3000])), p_root=float(r.choice([0.01, 0.05])),
                        p_empty=float(r.choice([0.0, 0.15, 0.4])))
        t = with_growth_room(t, 40)
        hk, hq, d = SHAPES[seed % len(SHAPES)]
        with ets.Context(hk, hq, d, ets.ETS_BF16, -1) as ctx, ets.Context(hk, hq, d, ets.ETS_BF16, -1) as by64:
            ctx.set_option("stream_chunk", int(r.choice([0, 0, 64])))
            ctx.set_option("cascade_chunk", int(r.choice([0, 0, 96])))
            ctx.set_option("wave_items", int(r.choice([512, 0, 100000])))
            ctx.set_option("interleave", int(r.choice([1, 1, 0])))
            st = _plan(ctx, t)
            by64.set_option("cascade_rows", 64)
            _plan(by64, t)
            assert st.unique_tokens == by64.stats().unique_tokens
            # a segment whose leaf queries are all in different groups is read by each of them (two at least)
            by_all = by64.stats()
            assert st.cascade_tokens <= by_all.cascade_tokens
            assert st.stream_tokens - by_all.stream_tokens >= 2 * (by_all.cascade_tokens - st.cascade_tokens)
            if ctx.item_rows() == 64:
                assert st.stream_tokens == by_all.stream_tokens
            apart += st.cascade_tokens < by_all.cascade_tokens
            assert by64.item_rows() == 64
            joined += ctx.item_rows() == 128
            rep = ctx.check()
            assert rep.violations == 0 and rep.max_entry_overreach <= 15, (seed, rep.as_dict())
            _covers(ctx, t, t.n_tokens)
            n_tokens = t.n_tokens.copy()
            for step in range(int(r.choice([1, 34]))):
                ctx.plan_advance()
                n_tokens[np.unique(t.leaf_node)] += 1
            assert ctx.check().violations == 0, seed
            _covers(ctx, t, n_tokens)
    assert joined >= 6  # the sweep does reach the plans it is about
    assert apart > 0 or block not in (2, 4, 6)


def test_the_leaf_queries_of_one_search_share_one_list_down_to_their_last_common_node():
    """A chain of 40 nodes of 100 rows with 64 leaf queries at its end: each group of 16 (8 query heads
    per kv head) reads it as one list, so that a leaf query has as many partials as that list has
    chunks; with one list per 64 query rows and segment it would be the same here, but not where a leaf
    query branches off every node: there a group's common part is one list, too."""
    n = 40
    chain = np.arange(-1, n - 1, dtype=np.int32)
    parent = np.concatenate([chain, np.repeat(np.arange(n, dtype=np.int32), 4)])
    n_tok = np.full(parent.size, 100, np.int32)
    off = np.arange(parent.size, dtype=np.int64) * 100
    leaf = np.arange(n, parent.size, dtype=np.int32)
    stats = []
    for opts in ({}, {"cascade_rows": 64}):
        with ets.Context(16, 128, 128, ets.ETS_BF16, -1) as ctx:
            for k, v in opts.items():
                ctx.set_option(k, v)
            ctx.set_option("cascade_chunk", 100000)
            stats.append(ctx.plan(parent, off, n_tok, leaf))
    # by segment: a leaf query below node i has i + 1 shared parts and its own
    assert stats[1].n_partials == 4 * sum(i + 2 for i in range(n))
    # by group: the parts above the group's first branch are one, those below it stay apart
    assert stats[0].n_partials == 4 * sum((i % 4) + 2 for i in range(n))


@pytest.mark.parametrize("hq,d,leaves,root,leaf", [(64, 64, 192, 50000, 16), (64, 64, 256, 8320, 64),
                                                   (64, 64, 320, 12480, 16), (64, 64, 512, 4160, 16)])
def test_a_plan_that_fits_the_static_scratch_by_segment_fits_it(hq, d, leaves, root, leaf):
    """The group kernel's lists can be cut finer than items of 64 query rows: such a plan must not grow
    out of the buffer of ets_tree_decode_attn_static."""
    parent = np.concatenate([[-1], np.zeros(leaves, np.int32)]).astype(np.int32)
    n_tok = np.concatenate([[root], np.full(leaves, leaf)]).astype(np.int32)
    off = np.cumsum(n_tok.astype(np.int64)) - n_tok
    size = []
    for opts in ({}, {"cascade_rows": 64}):
        with ets.Context(8, hq, d, ets.ETS_BF16, -1) as ctx:
            for k, v in opts.items():
                ctx.set_option(k, v)
            size.append(ctx.plan(parent, off, n_tok, np.arange(1, leaves + 1, dtype=np.int32)).workspace_bytes)
            assert ctx.check().violations == 0
    assert size[1] <= ets.ETS_STATIC_SCRATCH_BYTES and size[0] <= ets.ETS_STATIC_SCRATCH_BYTES


def test_the_plan_says_which_kernel_takes_it():
    one = np.array([-1], np.int32)
    for n_tok, leaves, options, mode, rows in [
            (16500, 200, {}, ets.ETS_PLAN_TREE, 128), (16500, 200, {"cascade_rows": 32}, ets.ETS_PLAN_TREE, 32),
            (100, 200, {}, ets.ETS_PLAN_TREE, 64), (16500, 200, {}, ets.ETS_PLAN_FLAT, 64),
            (16500, 200, {"mfma": 0}, ets.ETS_PLAN_TREE, 0), (0, 200, {}, ets.ETS_PLAN_TREE, 0)]:
        with ets.Context(2, 8, 128, ets.ETS_BF16, -1) as ctx:
            with pytest.raises(ets.EtsError):
                ctx.item_rows()
            for k, v in options.items():
                ctx.set_option(k, v)
            ctx.plan(one, np.zeros(1, np.int64), np.array([n_tok], np.int32), np.zeros(leaves, np.int32), mode)
            assert ctx.item_rows() == rows, (n_tok, leaves, options, mode)


@pytest.mark.parametrize("leaves,root,leaf,d,rows", [
    # (8 query heads per kv head: 56 rows are a tile of 64 and a tile of 128, 72 two and two, because 8 rows stay
    # apart, 88 two and one, 136 three and two)
    (7, 60000, 8, 128, 64), (7, 60000, 8, 64, 128), (9, 60000, 8, 128, 64), (9, 60000, 8, 64, 128),
    (11, 60000, 8, 128, 128), (17, 60000, 8, 128, 128),
    (17, 60000, 14000, 128, 64), (17, 60000, 14000, 64, 128), (16, 60000, 8000, 128, 128), (16, 8256, 8, 128, 64)])
def test_rows_that_fill_few_tiles_of_128_stay_with_items_of_64(leaves, root, leaf, d, rows):
    parent = np.concatenate([[-1], np.zeros(leaves, np.int32)]).astype(np.int32)
    n_tok = np.concatenate([[root], np.full(leaves, leaf)]).astype(np.int32)
    off = np.cumsum(n_tok.astype(np.int64)) - n_tok
    with ets.Context(8, 64, d, ets.ETS_BF16, -1) as ctx:
        ctx.plan(parent, off, n_tok, np.arange(1, leaves + 1, dtype=np.int32))
        assert ctx.item_rows() == rows


def test_rows_that_a_leaf_query_reads_by_itself_are_counted_as_such():
    """33 leaf queries under a root, the last four under a longer branch of it, the others under short
    ones: with 8 query heads per kv head the last one's rows stay out of the root's larger items, in a
    list of its own."""
    root, branch, short, leaf = 8320, 9000, 100, 40
    parent = np.array([-1, 0, 1, 2, 3, 0] + [1, 2] + [3] * 5 + [4] * 22 + [5] * 4, np.int32)
    n_tok = np.array([root] + [short] * 4 + [branch] + [leaf] * 33, np.int32)
    off = np.cumsum(n_tok.astype(np.int64)) - n_tok
    with ets.Context(8, 64, 128, ets.ETS_BF16, -1) as ctx:
        st = ctx.plan(parent, off, n_tok, np.arange(6, 39, dtype=np.int32))
        assert ctx.item_rows() == 128
        assert st.cascade_tokens == root + branch + 4 * short and st.stream_tokens == 33 * leaf + root
        assert ctx.check().violations == 0
