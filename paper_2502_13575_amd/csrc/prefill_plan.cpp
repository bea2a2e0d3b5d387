// Planner of step-prefill attention: per distinct leaf node one run list (ancestors'
// rows merged where they are contiguous in the pool and cut into steps of 32, in which the
// rest of one piece is joined with the start of the next; then the node's own rows in
// pieces of 32 counted from its first row), per leaf query
// blocks of rows_per_item / G query tokens.  Leaf queries are taken in depth-first order of their
// nodes, so that workgroups that run at the same time walk the same ancestors.
#include "prefill_plan.h"

#include <algorithm>
#include <functional>
#include <limits>
#include <new>
#include <vector>

namespace ets {
namespace {

ets_status check(const ets_tree& t) {
    if (t.n_nodes < 0 || t.n_leaves < 0) return ETS_ERR_INVALID_ARG;
    if (t.n_nodes > 0 && (!t.parent || !t.tok_offset || !t.n_tokens)) return ETS_ERR_INVALID_ARG;
    if (t.n_leaves > 0 && !t.leaf_node) return ETS_ERR_INVALID_ARG;
    for (int32_t i = 0; i < t.n_nodes; ++i) {
        if (t.parent[i] < -1 || t.parent[i] >= i) return ETS_ERR_BAD_TREE;
        if (t.n_tokens[i] < 0 || t.tok_offset[i] < 0) return ETS_ERR_BAD_TREE;
        if (t.tok_offset[i] > std::numeric_limits<int64_t>::max() - t.n_tokens[i])
            return ETS_ERR_BAD_TREE;
    }
    for (int32_t l = 0; l < t.n_leaves; ++l)
        if (t.leaf_node[l] < 0 || t.leaf_node[l] >= t.n_nodes) return ETS_ERR_BAD_LEAF;
    return ETS_OK;
}

// Query rows per work item.  One workgroup is resident per compute unit, so a launch takes as many
// rounds as its workgroups fill the compute units, and a round costs the cycles that an item of
// that size spends on a run of 32 rows (526 runs in one round: 331 and 529 us).  (A block of at
// most 128 rows costs the same under either size; among items of 256 rows it shortens no round
// that also holds a full one.)  Calls of steps below a path of 960 rows, 8 kv heads x 4 query heads, us with 128 / 256 rows per
// item: 16 steps of 64 tokens 28.4 / 37.2 (one round either way); 16 steps of 65, 96, 128 tokens
// 48.5 / 37.1, 50.3 / 37.8, 53.8 / 43.3 (two rounds against one); 24 steps of 30 to 100 tokens
// 49.6 / 66.9 (two each); 256 steps of 48 tokens 390 / 305 (16 against 8).
constexpr int64_t kComputeUnits = 256, kPrefillRunSmall = 1350, kPrefillRunLarge = 2008;
int64_t rounds_cost(int64_t workgroups, int64_t cycles_per_run) {
    return (workgroups + kComputeUnits - 1) / kComputeUnits * cycles_per_run;
}

// Rounds charge a nearly empty last one in full.  So where they choose 128 rows although that makes
// more items, the workgroups are also handed out one by one, each to the compute unit that is
// free first, and 256 rows stay if that ends 5 % earlier.  (The allowance: on the card a workgroup
// does not always go where the first unit is free, which suits equal items better.)  45 steps of
// 17 to 42 tokens, 8 heads per kv head, 536 items in 2.1 rounds against 896 in 3.5: 104.6 us with
// 128 rows, 89.6 with 256; 42 steps of 36 to 44 tokens, 672 against 1 008: 80.4 and 87.5.
constexpr int64_t kScheduledWorkgroups = 4096;
// Work items are handed out for all kv heads one after the other; where these divide the units, the units
// stay in groups of as many with the same times, and one of each group is enough to follow.
class Schedule {
    size_t units_;
    int32_t copies_;
    std::vector<int64_t> free_at_;  // a heap, earliest on top, once every unit has a workgroup
    int64_t end_ = 0;

public:
    explicit Schedule(int32_t n_kv_heads)
        : units_((size_t)(kComputeUnits % n_kv_heads == 0 ? kComputeUnits / n_kv_heads : kComputeUnits)),
          copies_(kComputeUnits % n_kv_heads == 0 ? 1 : n_kv_heads) {
        free_at_.reserve(units_);
    }
    int64_t end() const { return end_; }
    void add_item(int64_t cycles) {
        for (int32_t c = 0; c < copies_; ++c) add(cycles);
    }

private:
    void add(int64_t cycles) {
        if (free_at_.size() < units_) {
            free_at_.push_back(cycles);
            end_ = std::max(end_, cycles);
            if (free_at_.size() == units_) std::make_heap(free_at_.begin(), free_at_.end(), std::greater<int64_t>());
            return;
        }
        const int64_t at = free_at_[0] + cycles;
        end_ = std::max(end_, at);
        size_t i = 0;  // the top's new time sinks to its place
        for (size_t child = 1; child < units_; child = 2 * i + 1) {
            if (child + 1 < units_ && free_at_[child + 1] < free_at_[child]) ++child;
            if (free_at_[child] >= at) break;
            free_at_[i] = free_at_[child];
            i = child;
        }
        free_at_[i] = at;
    }
};

ets_status build(const ets_shape& shape, const ets_tree& tree, PrefillPlan& p, int64_t kv_elem_bytes) {
    const int32_t N = tree.n_nodes, L = tree.n_leaves;
    const int32_t G = shape.n_q_heads / shape.n_kv_heads;
    p.parent.assign(tree.parent, tree.parent + N);
    p.tok_offset.assign(tree.tok_offset, tree.tok_offset + N);
    p.n_tokens.assign(tree.n_tokens, tree.n_tokens + N);
    p.leaf_node.assign(tree.leaf_node, tree.leaf_node + L);
    p.items.clear();
    p.q_ptr.assign((size_t)L + 1, 0);
    p.item_begin.assign((size_t)L, 0);
    for (int32_t l = 0; l < L; ++l) p.q_ptr[l + 1] = p.q_ptr[l] + p.n_tokens[p.leaf_node[l]];

    // depth-first position of every node: children (larger ids) in id order
    std::vector<int32_t> first_child(N, -1), next_sibling(N, -1), last_child(N, -1), roots;
    for (int32_t i = 0; i < N; ++i) {
        const int32_t par = p.parent[i];
        if (par < 0) {
            roots.push_back(i);
        } else if (first_child[par] < 0) {
            first_child[par] = last_child[par] = i;
        } else {
            next_sibling[last_child[par]] = i;
            last_child[par] = i;
        }
    }
    std::vector<int32_t> dfs_pos(N, 0), stack;
    int32_t pos = 0;
    for (auto r = roots.rbegin(); r != roots.rend(); ++r) stack.push_back(*r);
    while (!stack.empty()) {
        const int32_t n = stack.back();
        stack.pop_back();
        dfs_pos[n] = pos++;
        // push the siblings' chain in reverse so that the smallest id is visited first
        const size_t mark = stack.size();
        for (int32_t c = first_child[n]; c >= 0; c = next_sibling[c]) stack.push_back(c);
        std::reverse(stack.begin() + (std::ptrdiff_t)mark, stack.end());
    }
    std::vector<int32_t> order(L);
    for (int32_t l = 0; l < L; ++l) order[l] = l;
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        return dfs_pos[p.leaf_node[x]] < dfs_pos[p.leaf_node[y]];
    });

    ets_prefill_stats& st = p.stats;
    st = ets_prefill_stats{};
    st.n_leaves = L;
    st.n_q_rows = p.q_ptr[L];
    std::vector<char> live(N, 0);

    std::vector<int32_t> chain;
    std::vector<int32_t> run_begin_of(N, -1), anc_runs_of(N, 0);  // per distinct leaf node
    std::vector<int32_t> plain_runs_of(N, 0);  // ancestors' runs if none were joined
    std::vector<int64_t> anc_tokens_of(N, 0);
    auto steps_of = [](int64_t n) { return (n + kStepRows - 1) / kStepRows; };
    auto append_steps = [&](int64_t tok, int64_t n) {
        const size_t at = p.runs.size();
        p.runs.resize(at + (size_t)steps_of(n));
        for (Run* out = p.runs.data() + at; n > 0; ++out, tok += kStepRows, n -= kStepRows)
            *out = Run{tok, (int32_t)std::min<int64_t>(kStepRows, n), 0};
    };
    // `join`: whether runs may be joined of two pieces
    auto make_runs = [&](bool join) {
        p.runs.clear();
        p.joins = false;
        std::fill(run_begin_of.begin(), run_begin_of.end(), -1);
        std::fill(plain_runs_of.begin(), plain_runs_of.end(), 0);
        for (int32_t oi = 0; oi < L; ++oi) {
            const int32_t v = p.leaf_node[order[oi]];
            const int32_t len = p.n_tokens[v];
            if (run_begin_of[v] < 0 && len > 0) {
                chain.clear();
                for (int32_t x = v; x >= 0; x = p.parent[x]) chain.push_back(x);
                std::reverse(chain.begin(), chain.end());
                run_begin_of[v] = (int32_t)p.runs.size();
                // ancestors: contiguous rows merge, then steps of 32.  A step costs the same however many rows it
                // has, and every node of some hundred tokens used to end in a half-empty one.
                int64_t cur_tok = 0, cur_n = 0, anc_tokens = 0;
                auto flush = [&]() {
                    int64_t joined = 0;
                    plain_runs_of[v] += (int32_t)steps_of(cur_n);
                    if (join && cur_n > 0 && (int32_t)p.runs.size() - run_begin_of[v] > kPrefillFirstRuns)
                        joined = join_rows(p.runs.back(), cur_tok, cur_n);
                    p.joins = p.joins || joined > 0;
                    append_steps(cur_tok + joined, cur_n - joined);
                    cur_n = 0;
                };
                for (size_t c = 0; c + 1 < chain.size(); ++c) {
                    const int32_t n = chain[c];
                    live[n] = 1;
                    if (p.n_tokens[n] <= 0) continue;
                    anc_tokens += p.n_tokens[n];
                    if (cur_n > 0 && cur_tok + cur_n == p.tok_offset[n]) {
                        cur_n += p.n_tokens[n];
                    } else {
                        flush();
                        cur_tok = p.tok_offset[n];
                        cur_n = p.n_tokens[n];
                    }
                }
                flush();
                live[v] = 1;
                anc_runs_of[v] = (int32_t)p.runs.size() - run_begin_of[v];
                anc_tokens_of[v] = anc_tokens;
                append_steps(p.tok_offset[v], len);
                if (p.runs.size() > (size_t)std::numeric_limits<int32_t>::max() - 64)
                    return false;
            }
        }
        return true;
    };
    if (!make_runs(true)) return ETS_ERR_UNSUPPORTED;

    int64_t n_large = 0, n_small = 0;
    for (int32_t l = 0; l < L; ++l) {
        const int64_t q_rows = (int64_t)p.n_tokens[p.leaf_node[l]] * G;
        n_large += (q_rows + kPrefillRowsPerItem - 1) / kPrefillRowsPerItem;
        n_small += (q_rows + kPrefillRowsSmall - 1) / kPrefillRowsSmall;
    }
    n_large *= shape.n_kv_heads;
    n_small *= shape.n_kv_heads;
    auto rows_per_item = [&]() {
        bool small = rounds_cost(n_small, kPrefillRunSmall) < rounds_cost(n_large, kPrefillRunLarge);
        if (small && n_small > n_large && n_small > kComputeUnits && n_small <= kScheduledWorkgroups) {
            auto ends = [&](int32_t rows) {
                Schedule schedule(shape.n_kv_heads);
                for (int32_t oi = 0; oi < L; ++oi) {
                    const int32_t v = p.leaf_node[order[oi]], len = p.n_tokens[v];
                    for (int32_t t0 = 0; t0 < len; t0 += rows / G) {
                        const int32_t n_tok = std::min(rows / G, len - t0);
                        const int64_t runs = anc_runs_of[v] + (t0 + n_tok - 1) / 32 + 1;
                        const int64_t cycles =
                            runs * (n_tok * G <= kPrefillRowsSmall ? kPrefillRunSmall : kPrefillRunLarge);
                        schedule.add_item(cycles);
                    }
                }
                return schedule.end();
            };
            small = ends(kPrefillRowsSmall) * 100 < ends(kPrefillRowsPerItem) * 105;
        }
        return small ? kPrefillRowsSmall : kPrefillRowsPerItem;
    };
    int32_t rows = rows_per_item();
    // The loop that takes joined runs is 1 to 3 % longer, and a launch of few rounds, where a workgroup waits for
    // its loads more than for anything else, gains less by fewer rows.  The time without over the time with, up
    // to four rounds: 0.97 to 1.00 where less than 7 % of the runs are saved; 123 drawn calls where more are: up to
    // 10 % 0.96 to 1.06, geometric mean 1.02, to 15 % 0.98 to 1.08, 1.03, beyond 0.97 to 1.19, 1.07 (5 of
    // them lose more than a hundredth).  More rounds, 77 calls: 2.5 to 5 % 0.99 to 1.03, 1.01, to 8 % 0.98 to
    // 1.05, 1.02, to 15 % 1.00 to 1.08, 1.05, beyond 1.02 to 1.21, 1.08.
    // (Joins that save no run are such a call too.)
    if (p.joins) {
        int64_t plain = 0, saved = 0;  // runs walked by all items
        for (int32_t l = 0; l < L; ++l) {
            const int32_t v = p.leaf_node[l], len = p.n_tokens[v];
            for (int32_t t0 = 0; t0 < len; t0 += rows / G) {
                plain += plain_runs_of[v] + (std::min(t0 + rows / G, len) - 1) / 32 + 1;
                saved += plain_runs_of[v] - anc_runs_of[v];
            }
        }
        const int64_t workgroups = rows == kPrefillRowsSmall ? n_small : n_large;
        if (saved * (workgroups <= 4 * kComputeUnits ? 15 : 40) < plain) {
            if (!make_runs(false)) return ETS_ERR_UNSUPPORTED;
            rows = rows_per_item();
        }
    }
    const int32_t tq = rows / G;  // query tokens per item
    st.rows_per_item = rows;

    std::vector<std::vector<PrefillItem>> per_leaf((size_t)L);
    for (int32_t oi = 0; oi < L; ++oi) {
        const int32_t l = order[oi];
        const int32_t v = p.leaf_node[l];
        const int32_t len = p.n_tokens[v];
        for (int32_t t0 = 0; t0 < len; t0 += tq) {
            PrefillItem it{};
            it.n_tok = std::min(tq, len - t0);
            it.tok0 = t0;
            it.run_begin = run_begin_of[v];
            it.run_end = run_begin_of[v] + anc_runs_of[v] + (t0 + it.n_tok - 1) / 32 + 1;
            it.q_row0 = p.q_ptr[l] + t0;
            it.leaf = l;
            it.n_anc = anc_runs_of[v];
            per_leaf[l].push_back(it);
            // what the block's queries see: ancestors in full, own rows causally
            const int64_t a = t0, b = t0 + it.n_tok;  // own rows visible: a + 1 .. b
            st.visible_pairs += it.n_tok * anc_tokens_of[v] + (b * (b + 1) - a * (a + 1)) / 2;
            for (int32_t r = it.run_begin; r < it.run_end; ++r) st.streamed_tokens += p.runs[r].n;
        }
    }
    // items in the depth-first leaf order; item_begin indexes them per leaf query
    std::vector<int32_t> n_items_of(L, 0);
    for (int32_t oi = 0; oi < L; ++oi) {
        const int32_t l = order[oi];
        n_items_of[l] = (int32_t)per_leaf[l].size();
        for (const PrefillItem& it : per_leaf[l]) p.items.push_back(it);
    }
    {
        // position of leaf query l's first item in p.items
        int32_t cursor = 0;
        std::vector<int32_t> first(L, 0);
        for (int32_t oi = 0; oi < L; ++oi) {
            first[order[oi]] = cursor;
            cursor += n_items_of[order[oi]];
        }
        for (int32_t l = 0; l < L; ++l) p.item_begin[l] = first[l];
    }
    // Launch order.  Depth-first order ends a launch of few rounds on whatever comes last, and the chip waits
    // for its long items: there the longest go first where that ends earlier by a hundredth.  Items of the same
    // length stay in depth-first order.  (1 280 workgroups of 64 steps of 100 to 150 tokens 450 -> 443 us; the model
    // says 7 %, but a workgroup does not always go where a unit is free.  Beyond sixteen rounds it ends less than
    // a hundredth earlier, and what runs together should walk the same ancestors.)
    p.order.resize(p.items.size());
    for (size_t i = 0; i < p.order.size(); ++i) p.order[i] = (int32_t)i;
    if ((int64_t)p.items.size() * shape.n_kv_heads <= kScheduledWorkgroups) {
        auto cycles = [&](int32_t i) {
            const PrefillItem& it = p.items[(size_t)i];
            return (it.run_end - it.run_begin) * (it.n_tok * G <= kPrefillRowsSmall ? kPrefillRunSmall : kPrefillRunLarge);
        };
        auto end_of = [&](const std::vector<int32_t>& order) {
            Schedule schedule(shape.n_kv_heads);
            for (int32_t i : order) schedule.add_item(cycles(i));
            return schedule.end();
        };
        // (an order cannot end before an even share of the work, nor before its longest item)
        int64_t work = 0, most = 0;
        for (int32_t i : p.order) {
            work += cycles(i);
            most = std::max<int64_t>(most, cycles(i));
        }
        const int64_t even = (work * shape.n_kv_heads + kComputeUnits - 1) / kComputeUnits;
        const int64_t end = end_of(p.order);
        if (std::max(even, most) * 100 < end * 99) {
            std::vector<int32_t> longest = p.order;
            std::stable_sort(longest.begin(), longest.end(), [&](int32_t x, int32_t y) { return cycles(x) > cycles(y); });
            if (end_of(longest) * 100 < end * 99) p.order.swap(longest);
        }
    }
    st.n_items = (int64_t)p.items.size();
    st.n_runs = (int64_t)p.runs.size();
    for (int32_t i = 0; i < N; ++i) {
        if (!live[i]) continue;
        st.unique_tokens += p.n_tokens[i];
        if (p.n_tokens[i] > 0)
            st.min_pool_tokens = std::max(st.min_pool_tokens, p.tok_offset[i] + p.n_tokens[i]);
    }
    const int64_t tok_bytes = 2 * (int64_t)shape.n_kv_heads * shape.head_dim * kv_elem_bytes;
    st.unique_kv_bytes = st.unique_tokens * tok_bytes;
    st.streamed_kv_bytes = st.streamed_tokens * tok_bytes;
    // two contractions of head_dim per (query row, visible key row), 2 flops per multiply-add
    st.flops = 4 * (int64_t)shape.head_dim * shape.n_q_heads * st.visible_pairs;
    p.valid = true;
    return ETS_OK;
}

}  // namespace

ets_status build_prefill_plan(const ets_shape& shape, const ets_tree& tree, PrefillPlan& plan,
                              int64_t kv_elem_bytes) {
    plan.valid = false;
    const ets_status s = check(tree);
    if (s != ETS_OK) return s;
    try {
        return build(shape, tree, plan, kv_elem_bytes);
    } catch (const std::bad_alloc&) {
        plan.valid = false;
        return ETS_ERR_NOMEM;
    }
}

bool prefill_cover(const PrefillPlan& p, int32_t leaf, int32_t tok, std::vector<int64_t>& rows) {
    rows.clear();
    // the items of a leaf query are consecutive, in token order
    for (size_t i = (size_t)p.item_begin[leaf]; i < p.items.size() && p.items[i].leaf == leaf; ++i) {
        const PrefillItem& it = p.items[i];
        if (tok < it.tok0 || tok >= it.tok0 + it.n_tok) continue;
        for (int32_t r = it.run_begin; r < it.run_end; ++r) {
            const Run& run = p.runs[r];
            const int64_t kpos = (int64_t)kStepRows * (r - it.run_begin - it.n_anc);
            for (int32_t t = 0; t < run.n; ++t)
                if (kpos + t <= tok) rows.push_back(run_row(run, t));
        }
        return true;
    }
    return false;
}

bool check_prefill_plan(const PrefillPlan& p, const ets_shape& shape, PlanCheck& out) {
    out = PlanCheck{};
    const int G = shape.n_q_heads / shape.n_kv_heads;
    const int64_t n_runs = (int64_t)p.runs.size();
    auto bad = [&](bool cond) {
        if (cond) out.violations += 1;
    };
    bad(p.order.size() != p.items.size());  // every item once
    std::vector<char> seen(p.items.size(), 0);
    for (int32_t i : p.order) bad(i < 0 || (size_t)i >= seen.size() || seen[(size_t)i]++ != 0);
    for (const PrefillItem& it : p.items) {
        out.items += 1;
        bad(it.run_begin < 0 || it.run_end < it.run_begin || it.run_end > n_runs);
        bad(it.n_anc < 0 || it.run_begin + it.n_anc > it.run_end);
        for (int64_t r = it.run_begin; r < it.run_end && r < n_runs; ++r)
            bad(p.runs[(size_t)r].join != 0 && (r < it.run_begin + kPrefillFirstRuns || r >= it.run_begin + it.n_anc));
        bad(it.n_tok < 1 || it.n_tok * G > p.stats.rows_per_item);
        bad(it.leaf < 0 || it.leaf >= p.stats.n_leaves);
        // query tokens past n_tok are clamped to the block's last one by the kernel
        bad(it.q_row0 < 0 || it.q_row0 + it.n_tok > p.stats.n_q_rows);
        for (int64_t r = it.run_begin; r < it.run_end && r < n_runs; ++r) {
            const Run& run = p.runs[(size_t)r];
            bad(!check_step(run, p.stats.min_pool_tokens));
            for (int32_t t = 0; t < run.n; ++t) out.max_pool_row = std::max(out.max_pool_row, run_row(run, t));
        }
    }
    return out.violations == 0;
}

}  // namespace ets
