// Host planner: validates the tree, counts leaf queries per node, compacts
// chains of nodes with identical leaf sets into segments, cuts segments into
// work items for the two attention kernels and numbers the partial results.
//
// Tree semantics after the ETS paper, Sec. 4.1 and App. B: a non-leaf node is
// needed iff some retained leaf is among its descendants, and all trajectories
// through a node share that node's KV.
#include "plan.h"

#include <algorithm>
#include <limits>
#include <new>
#include <utility>

namespace ets {
namespace {

// Whether the planner, left to decide, merges inside the attention launch.
bool fuse_by_default(const ets_stats&) { return false; }

struct Seg {
    int32_t parent_seg = -1;
    int64_t cnt = 0;             // leaf queries at or beneath the segment
    std::vector<int32_t> nodes;  // chain, root side first
    int64_t tokens = 0;
    int32_t ent_begin = 0;       // range in Plan::ent_order
    int32_t own_filled = 0;
    int32_t child_cursor = 0;
    bool cascade = false;
    bool wide = false;           // read by the wide kernel (many query rows)
};

// A list of nodes that the consecutive leaf queries ent_order[ent_begin .. + n_ent) read together:
// one or more segments.  Its chunks take n_chunks partial slots of each of them, from `prefix` on.
struct Shared {
    int32_t ent_begin = 0, n_ent = 0;
    std::vector<int32_t> nodes;
    int64_t tokens = 0;
    int32_t prefix = 0, n_chunks = 0;
    int32_t above = -1;          // the shared list before it on the way from the root
    bool wide = false;
    int32_t tail = 0;            // its last leaf queries, which keep an item of their own
    int32_t slots = -1;          // lists with the same number here end at the same partial slot
};

struct Chunk {
    int32_t run_begin, run_end, tokens;
};

constexpr int64_t kMaxPiecesPerChunk = kTreeAttnMaxSteps;  // step list the kernel keeps in LDS

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t round_up(int64_t a, int64_t m) { return ceil_div(a, m) * m; }

// Small calls over fp32 pools take one launch (direct_attn_kernel): rows per item of such a plan, 0 = two
// launches.  `longest`: rows of the longest path; items16, items32: items of all leaf queries, at least one each, if
// they are cut after 16 or 32 rows.  Two limits:
//  - A compute unit takes a whole path of a kv head, in at most sixteen waves, while two launches spread
//    it.  Time of two launches over that of one, calls of up to 60 leaves: up to two query heads per kv head 1.3 to
//    1.6 at 250 to 400 rows, 1.04 to 1.2 at 450 to 512; four heads 1.2 to 1.45 at 250, 1.04 to 1.15 at 400, 0.87
//    to 1.05 from 430 on; eight heads of 64 0.92 to 1.1 at 300 to 320, 0.83 to 0.95 from 410, of 128 1.02
//    to 1.15 at 340 to 400, 0.83 to 0.96 from 420.
//  - With more waves than the chip holds at once the ends of the items count, each a fold of every query head's
//    sums over the lanes: up to 10 000 partial rows (items times query heads) 16 rows to an item took 0.96 to
//    2.0, with eight heads up to 20 000; beyond, down to 0.65 (364 leaves of 71 rows, 32 heads), where 32
//    rows take 1.03.  32 rows up to 15 000 partial rows 0.85 to 1.7; beyond, 0.58 to 1.3.
// 278 random searches of 8 to 24 leaves: 114 come under the rule, 1.01 to 1.7 times faster, 1.27 in the geometric mean;
// 900 calls of 1 to 2 000 leaves: 700, 1.31, 17 of them 2 to 19 % slower.  The others would mostly lose.
constexpr int64_t kDirectGrain = 16;  // rows of an item: a multiple of
int64_t direct_rows(const ets_shape& shape, int64_t longest, int64_t items16, int64_t items32) {
    const int32_t G = shape.n_q_heads / shape.n_kv_heads, Hq = shape.n_q_heads;
    const int64_t most = G <= 2 ? 512 : G == 4 ? 416 : shape.head_dim == 64 ? 320 : 400;
    if (longest > most) return 0;
    if (longest <= 16 * kDirectWaves && items16 * Hq <= (G == 8 ? 20000 : 10000)) return 16;
    return items32 * Hq <= 15000 ? 32 : 0;
}

// Consecutive pool rows of a node list, before they are cut into steps.
struct Piece {
    int64_t tok;  // first pool row
    int32_t n;    // rows
    bool grows;   // ends a node that holds leaf queries
};

// Appends the (merged) pieces of a node list to `out`.  A node that holds leaf
// queries grows by a token per decode step: the piece that ends such a node is marked
// and nothing is merged behind it.  Returns false if a growing node has no
// rows yet (there is no piece to mark).
bool collect_pieces(const Plan& p, const std::vector<int32_t>& nodes, const std::vector<int64_t>& own,
                    std::vector<Piece>& out) {
    bool ok = true;
    bool closed = true;  // the previous run must not be extended
    for (int32_t n : nodes) {
        const int32_t len = p.n_tokens[n];
        const bool grows = own[n] > 0;
        if (len <= 0) {
            if (grows) ok = false;
            continue;
        }
        const int64_t tok = p.tok_offset[n];
        if (!closed && !out.empty() && out.back().tok + out.back().n == tok &&
            (int64_t)out.back().n + len <= std::numeric_limits<int32_t>::max()) {
            out.back().n += len;
        } else {
            out.push_back(Piece{tok, len, false});
        }
        out.back().grows = grows;
        closed = grows;
    }
    return ok;
}

// Cuts `src` (total `tokens` rows) into chunks of at most `cap` rows, sized
// evenly in multiples of `grain` rows, appending the chunks' runs to plan.runs.  With
// piece > 0 no emitted run is longer than `piece` rows (the matrix-core kernel
// walks its run list in steps of at most 32 rows).  Behind the last run of a marked
// piece (a growing node's tail) an empty spare run is emitted and an AdvEntry recorded;
// returns false if a chunk's step list had no room for a spare.  `join`: a step that the end of a
// piece does not fill goes on in the next piece (see join_rows).
bool cut_runs(Plan& p, const std::vector<Piece>& src, int64_t tokens, int64_t cap, int64_t piece, bool join,
              std::vector<Chunk>& chunks, int64_t grain = 32) {
    chunks.clear();
    if (tokens <= 0) return true;
    bool ok = true;
    cap = std::max<int64_t>(cap, grain);
    int64_t n_chunks = ceil_div(tokens, cap);
    int64_t per = std::min(cap, round_up(ceil_div(tokens, n_chunks), grain));
    size_t ri = 0;
    int64_t used = 0;  // rows of src[ri] already handed out
    int64_t left = tokens;
    while (left > 0) {
        int64_t want = std::min(per, left);
        Chunk c{(int32_t)p.runs.size(), 0, 0};
        int64_t pieces = 0;
        bool open = false;  // the last step may go on in the next run
        while (want > 0 && (piece <= 0 || pieces < kMaxPiecesPerChunk)) {
            const int64_t avail = src[ri].n - used;
            int64_t take = open ? join_rows(p.runs.back(), src[ri].tok, std::min(avail, want)) : 0;
            if (take == 0) {
                take = std::min(avail, want);
                if (piece > 0) take = std::min(take, piece);
                p.runs.push_back(Run{src[ri].tok + used, (int32_t)take, 0});
                ++pieces;
            }
            used += take;
            want -= take;
            c.tokens += (int32_t)take;
            open = join && used == src[ri].n && !src[ri].grows && p.runs.back().n < kStepRows;
            if (used == src[ri].n) {
                if (src[ri].grows) {
                    if (piece > 0 && pieces >= kMaxPiecesPerChunk) {
                        ok = false;
                    } else {
                        const int32_t r_last = (int32_t)p.runs.size() - 1;
                        const int64_t end0 = src[ri].tok + src[ri].n;
                        p.adv.push_back(AdvEntry{r_last, r_last + 1, end0, 1, 0});
                        p.runs.push_back(Run{end0, 0, 0});
                        ++pieces;
                    }
                }
                ++ri;
                used = 0;
            }
        }
        c.run_end = (int32_t)p.runs.size();
        left -= c.tokens;
        chunks.push_back(c);
    }
    return ok;
}

// Fills the slot's copies of its item's steps from the step lists.  Returns whether one of
// them is a run that an advance may extend.
bool fill_unit_steps(const Plan& p, UnitSlot& u, int wave, const std::vector<char>* grows) {
    bool may_grow = false;
    Run* dst[2] = {&u.first, &u.second};
    for (int j = 0; j < 2; ++j) {
        const int k = unit_step_index(u.item, wave, j);
        const int64_t r = (int64_t)u.item.run_begin + k;
        if (k < 0 || r >= u.item.run_end) {
            *dst[j] = Run{0, 0, 0};
            continue;
        }
        *dst[j] = p.runs[(size_t)r];
        if (grows) may_grow = may_grow || (*grows)[(size_t)r];
    }
    return may_grow;
}

// CascadeItem::wave_item of an item that stands in the launch order as `code`.
int32_t unit_kind(const Plan& p, int32_t code, const CascadeItem& it, int64_t G) {
    return code < 0 ? 1 : !p.groups ? 0 : it.n_ent * G <= 16 ? 2 : 3;
}

// The table the matrix-core kernel starts from (see UnitSlot), and the slots whose copies
// of steps an advance has to refresh.
void build_units(Plan& p, int64_t G) {
    const size_t n_units = p.wg_map.size();
    p.units.assign(4 * n_units, UnitSlot{});  // zero: n_ent = 0, nothing to do
    p.adv_slots.clear();
    std::vector<char> grows(p.runs.size(), 0);
    for (const AdvEntry& e : p.adv) grows[(size_t)e.r_last] = grows[(size_t)e.r_spare] = 1;
    const int64_t n_items = (int64_t)p.cascade_items.size();
    for (size_t y = 0; y < n_units; ++y) {
        const int32_t code = p.wg_map[y];
        for (int w = 0; w < 4; ++w) {
            const int64_t idx = code >= 0 ? code : p.n_single + 4 * (-(int64_t)code - 1) + w;
            if (idx >= n_items) continue;
            UnitSlot& u = p.units[4 * y + (size_t)w];
            u.item = p.cascade_items[(size_t)idx];
            u.item.wave_item = unit_kind(p, code, u.item, G);
            if (fill_unit_steps(p, u, w, &grows)) p.adv_slots.push_back((int32_t)(4 * y + (size_t)w));
        }
    }
}

// After an advance: the unit table's copies follow the step lists.
void refresh_units(Plan& p) {
    for (int32_t slot : p.adv_slots) fill_unit_steps(p, p.units[(size_t)slot], slot & 3, nullptr);
}

// Cuts the leaf queries (in depth-first order) into groups of at most `room` consecutive ones, with
// the fewest tokens for the groups to read: the sum over the groups of the shared rows above any of
// their leaf queries.  What two neighbours have in common is read once if they share a group and
// twice if a boundary stands between them, so a boundary costs the rows above both (`costs[i]`:
// between leaf queries i - 1 and i).  Returns the first leaf query of every group, and the end.
std::vector<int32_t> group_leaves(const std::vector<int64_t>& costs, int32_t room) {
    constexpr int64_t kGroupTokens = 32;  // and a group of its own costs about the start of an item
    const int32_t L = (int32_t)costs.size();
    std::vector<int64_t> cost((size_t)L + 1, 0);
    std::vector<int32_t> from((size_t)L + 1, 0);
    for (int32_t j = 1; j <= L; ++j) {
        cost[j] = std::numeric_limits<int64_t>::max();
        for (int32_t i = std::max(0, j - room); i < j; ++i) {
            const int64_t c = cost[i] + costs[i] + kGroupTokens;
            if (c < cost[j]) {
                cost[j] = c;
                from[j] = i;
            }
        }
    }
    std::vector<int32_t> bounds;
    for (int32_t j = L; j > 0; j = from[j]) bounds.push_back(j);
    bounds.push_back(0);
    std::reverse(bounds.begin(), bounds.end());
    return bounds;
}

ets_status validate(const ets_tree& t) {
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

ets_status build(const ets_shape& shape, const PlanOptions& opt, const ets_tree& tree, int mode,
                 bool may_group, Plan& p) {
    const int32_t N = tree.n_nodes, L = tree.n_leaves;
    const int32_t G = shape.n_q_heads / shape.n_kv_heads;
    const int64_t esz = opt.kv_elem_bytes > 0 ? opt.kv_elem_bytes : shape.dtype == ETS_F32 ? 4 : 2;

    p.mode = mode;
    p.parent.assign(tree.parent, tree.parent + N);
    p.tok_offset.assign(tree.tok_offset, tree.tok_offset + N);
    p.n_tokens.assign(tree.n_tokens, tree.n_tokens + N);
    p.leaf_node.assign(tree.leaf_node, tree.leaf_node + L);

    // leaf queries at or beneath every node (children have larger ids)
    std::vector<int64_t> own(N, 0);
    for (int32_t l = 0; l < L; ++l) own[p.leaf_node[l]] += 1;
    p.leaf_count = own;
    for (int32_t i = N - 1; i >= 0; --i)
        if (p.parent[i] >= 0) p.leaf_count[p.parent[i]] += p.leaf_count[i];

    ets_stats& st = p.stats;
    st = ets_stats{};
    st.n_nodes = N;
    st.n_leaves = L;
    for (int32_t i = 0; i < N; ++i) {
        if (p.leaf_count[i] == 0) continue;
        st.live_nodes += 1;
        st.unique_tokens += p.n_tokens[i];
        st.flat_tokens += p.leaf_count[i] * (int64_t)p.n_tokens[i];
        if (p.n_tokens[i] > 0)
            st.min_pool_tokens = std::max(st.min_pool_tokens, p.tok_offset[i] + p.n_tokens[i]);
    }
    const int64_t tok_bytes = 2 * (int64_t)shape.n_kv_heads * shape.head_dim * esz;
    st.unique_kv_bytes = st.unique_tokens * tok_bytes;
    st.flat_kv_bytes = st.flat_tokens * tok_bytes;

    // chain compaction: a live node joins its parent's segment when both have
    // the same leaf set, i.e. the same count
    std::vector<Seg> segs;
    std::vector<int32_t> seg_of(N, -1);
    for (int32_t i = 0; i < N; ++i) {
        if (p.leaf_count[i] == 0) continue;
        const int32_t par = p.parent[i];
        if (par >= 0 && p.leaf_count[par] == p.leaf_count[i]) {
            seg_of[i] = seg_of[par];
        } else {
            Seg s;
            s.parent_seg = par >= 0 ? seg_of[par] : -1;
            s.cnt = p.leaf_count[i];
            seg_of[i] = (int32_t)segs.size();
            segs.push_back(std::move(s));
        }
        Seg& s = segs[seg_of[i]];
        s.nodes.push_back(i);
        s.tokens += p.n_tokens[i];
    }
    st.n_segments = (int64_t)segs.size();

    p.runs.clear();
    p.stream_items.clear();
    p.cascade_items.clear();
    p.wide_items.clear();
    p.ent_order.assign(L, 0);
    p.part_base.assign((size_t)L + 1, 0);
    p.max_cascade_ent = 0;
    p.groups = false;
    p.direct_waves = 0;
    p.adv.clear();
    p.adv_in_place = true;
    p.advances = 0;

    std::vector<Piece> pieces;
    std::vector<Chunk> chunks;
    std::vector<int32_t> stream_tokens;   // per stream item, for ordering
    std::vector<int64_t> cascade_cost;    // per cascade item, for ordering

    // leaf queries in depth-first segment order: the queries beneath a segment
    // form one contiguous range of ent_order
    {
        std::vector<int64_t> seg_own(segs.size(), 0);
        for (int32_t l = 0; l < L; ++l) seg_own[seg_of[p.leaf_node[l]]] += 1;
        int64_t root_cursor = 0;
        for (size_t s = 0; s < segs.size(); ++s) {
            Seg& sg = segs[s];
            if (sg.parent_seg < 0) {
                sg.ent_begin = (int32_t)root_cursor;
                root_cursor += sg.cnt;
            } else {
                Seg& ps = segs[sg.parent_seg];
                sg.ent_begin = ps.child_cursor;
                ps.child_cursor += (int32_t)sg.cnt;
            }
            sg.child_cursor = sg.ent_begin + (int32_t)seg_own[s];
        }
        for (int32_t l = 0; l < L; ++l) {
            Seg& sg = segs[seg_of[p.leaf_node[l]]];
            p.ent_order[sg.ent_begin + sg.own_filled++] = l;
        }
    }

    // Which kernel reads which segment.  The matrix-core kernel reads a shared
    // segment once for all `cnt` leaf queries beneath it but costs one partial
    // result per query and query head (written, then read by the merge); otherwise
    // every query reads the segment itself as part of its own item.  A segment is
    // shared when the KV bytes this saves exceed the partial bytes it adds.
    const bool use_mfma = opt.mfma != 0 && shape.dtype == ETS_BF16;  // head_dim 64 or 128
    const bool cascade_ok = mode == ETS_PLAN_TREE && use_mfma && opt.cascade_min_leaves > 0;
    if (mode == ETS_PLAN_TREE && opt.require_sharing && !cascade_ok) return ETS_ERR_UNSUPPORTED;
    st.shares_nodes = cascade_ok ? 1 : 0;
    const int64_t piece = use_mfma ? 32 : 0;
    p.piece = (int32_t)piece;
    auto grow_end_of = [&](int32_t node) { return p.tok_offset[node] + p.n_tokens[node]; };
    const int64_t partial_bytes = 2 * (int64_t)shape.n_q_heads * (shape.head_dim + 2) * 4;
    constexpr int64_t kTile = 64;
    // wide kernel: one workgroup per compute unit, about t_wide per 64-token tile (1.8 us for items
    // of more than 128 query rows, 1.2 for others).  Off unless asked for: without it a call takes
    // 131 us on 256 leaves with 8 query heads per kv head against 142 to 159 for 512 to 16 rows,
    // 368 on 512 leaves against 425 to 458, 2 056 on 16 searches against 2 129 to 2 213; over E4M3
    // pools 290 on 512 leaves against 291 to 332.  It does not merge, so a plan that uses it keeps
    // the merge launch.
    const int64_t wide_rows = opt.wide_rows >= 0 && shape.head_dim == 128 ? opt.wide_rows : 0;
    const int64_t ent_per_wide = std::max<int64_t>(1, kWideRowsPerItem / G);
    const int64_t t_wide = 1500;
    bool any_wide = false;
    for (Seg& sg : segs) {
        sg.cascade = cascade_ok && sg.cnt >= 2 && sg.cnt >= opt.cascade_min_leaves &&
                     sg.tokens > 0 &&
                     (sg.cnt - 1) * sg.tokens * tok_bytes > sg.cnt * partial_bytes;
        // A segment with many query rows is work for the matrix cores, not for the memory
        // system: items of 64 rows would stream it rows / 64 times through the compute
        // units.  The wide kernel takes 256 rows per item.
        sg.wide = sg.cascade && wide_rows > 0 && sg.cnt * G > wide_rows;
        any_wide = any_wide || sg.wide;
        if (sg.wide) st.wide_tokens += sg.tokens;
    }
    // Items of at most 16 query rows apply weights of 16 bits to V as it is, larger ones weights of 11
    // bits to V in fp16, which ends at 65 504.  Cut into items of 64 query rows, a segment's last leaf queries
    // are in an item of the former kind where at most 16 rows are left over; larger items leave these
    // leaf queries out: nobody gets fewer bits by the larger item.  (16 searches of 256 leaves with
    // 64 query heads, 6 % of the leaf queries' rows: 1 916 us against 1 831 with them inside; one of
    // them 133 against 130, 512 leaves with 32 query heads 368 against 366.)
    auto tail_of = [&](const Seg& sg) {
        const int64_t per64 = std::max<int64_t>(1, kTreeAttnRowsPerItem / G), rest = sg.cnt % per64;
        return (int32_t)(rest * G <= 16 ? rest : 0);
    };
    // Which kernel.  The group kernel applies a tile to 128 query rows in about 1.0 us of a compute unit,
    // where two items of 64 rows of the other one take 1.3 together, reads it half as often and joins
    // segments into one item (see below); but with head_dim 128 only two of its workgroups are resident, so
    // that calls of short items and calls that stream are slower with it.  It takes the plans whose
    // row-parallel tiles (counted at 64 query rows; about 3.3 ns of the whole chip each)
    //  - are more than kGroupMinTiles (fewer: the other kernel's time over this one's is 0.83 to 1.26, median
    //    0.95) and fill at least three tenths of the time the unique bytes take (0.09 to 0.26 of it: 0.92 to 0.99);
    //  - have to fill a larger part the fewer they are: tiles times that part above 3 500 (40 drawn trees,
    //    below 0.90 to 1.07, median 0.99; above 0.97 to 1.29, median 1.06);
    //  - with head_dim 128 become so many fewer tiles of 128 rows (and of a tail's), at 1 / 0.9 of the price, that
    //    this saves a tenth of the time of the unique bytes: a segment of 81 to 128 rows halves its tiles, one of
    //    up to 64 only pays more (108 drawn trees: below 0.86 to 1.14, geometric mean 0.983; above 0.93 to 1.20, 1.045;
    //    with head_dim 64, 52 trees, 0.91 to 1.51, 1.14).
    const int64_t hbm_ns = st.unique_kv_bytes * (esz < 2 ? 2 : 1) / 5500;
    int64_t tiles64 = 0, tiles128 = 0;
    for (const Seg& sg : segs)
        if (sg.cascade && sg.cnt * G > 16) {
            tiles64 += ceil_div(sg.tokens, kTile) * ceil_div(sg.cnt * G, kTreeAttnRowsPerItem) * shape.n_kv_heads;
            const int64_t tail = tail_of(sg);
            tiles128 += ceil_div(sg.tokens, kTile) * shape.n_kv_heads *
                        (ceil_div((sg.cnt - tail) * G, kGroupRowsPerItem) + (tail > 0 ? 1 : 0));
        }
    p.groups = may_group && cascade_ok && !any_wide && opt.cascade_rows == 0 && opt.fuse_merge != 1 &&
               tiles64 > kGroupMinTiles && tiles64 * 11 > hbm_ns &&
               (double)tiles64 * tiles64 * 3.3 > 3500.0 * hbm_ns &&
               (shape.head_dim == 64 || (0.9 * tiles64 - tiles128) * 33 > hbm_ns);
    // Steps of two pieces: the kernel of 64-row items takes them.  (The group kernel keeps the waits for its loads
    // exact, and choosing every row's offset costs it what the steps save: one search of 256 leaves 133.2 ->
    // 131.7 us, 16 of them 1 918 -> 1 913, but 512 leaves over E4M3 pools 262 -> 267.  The wide kernel is off.)
    const bool join = piece == kStepRows && !p.groups && !any_wide;
    const int64_t rows_per_item =
        p.groups ? kGroupRowsPerItem : opt.cascade_rows > 0 ? opt.cascade_rows : kTreeAttnRowsPerItem;
    const int64_t ent_per_item = std::max<int64_t>(1, rows_per_item / G);
    // cost model in nanoseconds: a resident workgroup needs about t_tile per tile of 64
    // tokens whether it waits on memory (few rows) or computes (many rows), and t_item to
    // start and to store its partial results; kResident workgroups are resident (three per
    // compute unit, two of the group kernel with head_dim 128; with head_dim 64 four are, of which the model knows
    // three; what four would change in it was not measured).  Measured: 2.1-2.7 us per tile, 6.5-8.5
    // us per item; the sum predicts the attention launch of the configurations within 5 %.  Group
    // kernel: 1.5 us per tile of up to 64 query rows, 2.0-2.7 of more, 5-8 us per item, of which the
    // model takes one time for all.
    const int64_t t_tile = p.groups ? 2000 : 2500, t_item = 7000;
    const int64_t kResident = p.groups && shape.head_dim == 128 ? 512 : 768;
    // The shared lists.  A segment by itself would cost every leaf query beneath it a partial result,
    // and an item for every ent_per_item of them.  So the leaf queries are grouped, and within a
    // group the segments that the same leaf queries of it read are walked as one list: the path down
    // to a group's last common node is one item, and so is every stretch of a branch below it.
    std::vector<Shared> shared;
    std::vector<int32_t> last_shared(L, -1);  // by entry: the shared list nearest to its leaf
    std::vector<std::pair<int32_t, int32_t>> own_shared;  // (entry, shared segment) read by that entry alone
    // It pays where partial results are a good part of the traffic, and costs L2 hits where they are not:
    // groups walk the same rows at different times, the row groups of one segment at the same time.
    // Joined against by segment, us: 16 searches of 256 leaves with 64 query heads (31 % of the KV bytes in
    // partial results, 7.1 -> 4.1 of them for a leaf query) 1 953 against 1 998, one of them 132 against 142,
    // 58 drawn trees 0.94 to 1.15, geometric mean 1.02; 512 leaves with 32 query heads (8 %) 376 against
    // 369, over E4M3 pools 291 against 283.
    int64_t by_segment = L;
    for (const Seg& sg : segs)
        if (sg.cascade) by_segment += sg.cnt;
    p.min_workspace_bytes = (by_segment - L) * shape.n_q_heads * ((int64_t)shape.head_dim + 2) * 4;
    const bool grouped = p.groups && L >= 2 * ent_per_item &&
                         by_segment * partial_bytes * 8 > st.unique_kv_bytes * (esz < 2 ? 2 : 1);
    if (!grouped) {
        std::vector<int32_t> of_seg(segs.size(), -1);  // the nearest shared list at or above
        for (size_t i = 0; i < segs.size(); ++i) {
            const Seg& sg = segs[i];
            const int32_t above = sg.parent_seg >= 0 ? of_seg[sg.parent_seg] : -1;
            of_seg[i] = above;
            if (!sg.cascade) continue;
            of_seg[i] = (int32_t)shared.size();
            Shared sh;
            sh.ent_begin = sg.ent_begin;
            sh.n_ent = (int32_t)sg.cnt;
            sh.nodes.swap(segs[i].nodes);  // (nobody reads a shared segment by himself)
            sh.tokens = sg.tokens;
            sh.above = above;
            sh.wide = sg.wide;
            sh.tail = p.groups ? tail_of(sg) : 0;
            st.cascade_tokens += sg.tokens;
            shared.push_back(std::move(sh));
        }
        for (int32_t e = 0; e < L; ++e) last_shared[e] = of_seg[seg_of[p.leaf_node[p.ent_order[e]]]];
    } else {
        // rows of shared segments above neighbouring entries
        std::vector<int64_t> above_rows(segs.size(), 0), common(L, 0);
        std::vector<int32_t> level(segs.size(), 0);
        for (size_t i = 0; i < segs.size(); ++i) {
            const Seg& sg = segs[i];
            if (sg.parent_seg >= 0) {
                above_rows[i] = above_rows[sg.parent_seg];
                level[i] = level[sg.parent_seg] + 1;
            }
            if (sg.cascade) above_rows[i] += sg.tokens;
        }
        std::vector<int32_t> leaf_seg(L);
        for (int32_t e = 0; e < L; ++e) leaf_seg[e] = seg_of[p.leaf_node[p.ent_order[e]]];
        for (int32_t e = 1; e < L; ++e) {
            int32_t x = leaf_seg[e - 1], y = leaf_seg[e];
            while (x != y && x >= 0 && y >= 0) {
                if (level[x] >= level[y]) x = segs[x].parent_seg;
                else y = segs[y].parent_seg;
            }
            if (x == y && x >= 0) common[e] = above_rows[x];
        }
        // (a boundary where a tail begins costs less: its segment is read twice there anyway)
        std::vector<int64_t> costs = common;
        for (const Seg& sg : segs)
            if (const int32_t n = tail_of(sg); sg.cascade && n > 0 && n < sg.cnt)
                costs[sg.ent_begin + sg.cnt - n] -= sg.tokens;
        const std::vector<int32_t> bounds = group_leaves(costs, (int32_t)ent_per_item);
        auto slots_of = [&](int32_t e) { return last_shared[e] < 0 ? -1 : shared[last_shared[e]].slots; };
        std::vector<int32_t> in_group(segs.size(), -1), members;
        std::vector<char> counted(segs.size(), 0);  // in cascade_tokens
        for (size_t g = 0; g + 1 < bounds.size(); ++g) {
            const int32_t first = bounds[g], end = bounds[g + 1];
            members.clear();
            for (int32_t e = first; e < end; ++e)
                for (int32_t s = leaf_seg[e]; s >= 0 && in_group[s] != (int32_t)g; s = segs[s].parent_seg) {
                    in_group[s] = (int32_t)g;
                    members.push_back(s);
                }
            std::sort(members.begin(), members.end());  // parents before children
            for (int32_t s : members) {
                const Seg& sg = segs[s];
                if (!sg.cascade) continue;
                const int32_t seg_end = sg.ent_begin + (int32_t)sg.cnt, tail = seg_end - tail_of(sg);
                const int32_t hi = std::min(end, seg_end);
                // the group's entries of the segment, cut where its tail begins and where the entries' partial
                // slots so far differ (a list's slots are numbered alike for all its entries)
                for (int32_t lo = std::max(first, sg.ent_begin), next; lo < hi; lo = next) {
                    for (next = lo + 1; next < hi && slots_of(next) == slots_of(lo);) ++next;
                    const int32_t cut = lo < tail && tail < next ? tail : next;
                    // Lists of both parts, of a single entry too, keep their slots alike for what the
                    // entries on both sides read together further down.
                    const bool pair = cut < next && next - lo > 2 && common[cut] > above_rows[s];
                    const bool lists[2] = {pair || cut - lo > 1, pair || next - cut > 1};
                    bool made = true;
                    for (int k = 0; k < 2; ++k) {
                        const int32_t from = k ? cut : lo, to = k ? next : cut, n = to - from;
                        if (n == 0) continue;
                        if (!lists[k]) {
                            own_shared.push_back({from, s});
                            continue;
                        }
                        int32_t list = last_shared[from];
                        if (list < 0 || last_shared[to - 1] != list || shared[list].n_ent != n) {
                            Shared sh;
                            sh.ent_begin = from;
                            sh.n_ent = n;
                            sh.above = list;
                            list = (int32_t)shared.size();
                            sh.slots = k && pair && made ? list - 1 : list;
                            shared.push_back(std::move(sh));
                            std::fill(last_shared.begin() + from, last_shared.begin() + to, list);
                        } else {
                            made = false;  // (these entries are all that read the list above)
                        }
                        Shared& sh = shared[list];
                        sh.nodes.insert(sh.nodes.end(), sg.nodes.begin(), sg.nodes.end());
                        sh.tokens += sg.tokens;
                        if (n > 1 && !counted[s]) {
                            counted[s] = 1;
                            st.cascade_tokens += sg.tokens;
                        }
                    }
                }
            }
        }
        std::sort(own_shared.begin(), own_shared.end());
    }
    // segments that the leaf query of entry e reads by itself, leaf first
    auto own_segs = [&](int32_t e, std::vector<int32_t>& out) {
        out.clear();
        for (int32_t s = seg_of[p.leaf_node[p.ent_order[e]]]; s >= 0; s = segs[s].parent_seg)
            if (!segs[s].cascade ||
                (grouped && std::binary_search(own_shared.begin(), own_shared.end(), std::make_pair(e, s))))
                out.push_back(s);
    };
    // the items of a shared list: f(its first entry, counted in the list, and how many)
    auto for_items = [&](const Shared& sh, auto f) {
        const int64_t per_item = sh.wide ? ent_per_wide : ent_per_item;
        const int64_t body = sh.n_ent - (sh.wide ? 0 : sh.tail);
        for (int64_t e0 = 0; e0 < body; e0 += per_item) f(e0, std::min(per_item, body - e0));
        if (body < sh.n_ent) f(body, sh.n_ent - body);
    };
    int64_t own_total = 0, longest_own = 0, work_ns = 0, wide_work_ns = 0;
    int64_t own_items[2] = {0, 0};  // of what the leaf queries read themselves, cut after 16 and 32 rows
    int64_t items_est = L;  // one item per leaf query for what it reads itself, plus:
    for (const Shared& sh : shared) {
        if (sh.n_ent == 1) own_total += sh.tokens;  // (beside a list of others: read by one leaf query)
        if (sh.wide) {
            wide_work_ns += ceil_div(sh.tokens, kTile) * ceil_div(sh.n_ent, ent_per_wide) * t_wide *
                            shape.n_kv_heads;
            continue;
        }
        for_items(sh, [&](int64_t, int64_t n) {
            work_ns += ceil_div(sh.tokens, kTile) * t_tile * shape.n_kv_heads;
            items_est += 1;
        });
    }
    std::vector<int32_t> reads;
    for (int32_t e = 0; e < L; ++e) {
        own_segs(e, reads);
        int64_t tokens = 0;
        for (int32_t s : reads) {
            tokens += segs[s].tokens;
            work_ns += ceil_div(segs[s].tokens, kTile) * t_tile * shape.n_kv_heads;
        }
        own_total += tokens;
        longest_own = std::max(longest_own, tokens);
        for (int i = 0; i < 2; ++i) own_items[i] += std::max<int64_t>(ceil_div(tokens, 16 << i), 1);
    }
    st.stream_tokens = own_total;
    const int64_t direct_cap = shape.dtype == ETS_F32 && opt.stream_chunk <= 0 && L > 0
                                   ? direct_rows(shape, longest_own, own_items[0], own_items[1]) : 0;
    const bool direct = direct_cap > 0;
    // time the whole call is expected to take: the larger of the HBM time of the
    // unique bytes (at ~5.5 TB/s) and the modelled work spread over the resident
    // workgroups; no single item should take more than half of it: finer items balance no
    // better (the launch order starts the long ones first) and every further chunk of a
    // shared segment costs one more partial result for each leaf query beneath it
    // (measured on the configurations: the optimum lies at 45-55 % of the call time)
    // (1-byte pools are budgeted like 2-byte ones: their launch is bound by the number
    // of loads, not by their bytes, and finer items would only add partial results)
    // (plus the start and the end of the items on the critical path, which is what a small
    // call mostly consists of)
    const int64_t call_ns =
        std::max(hbm_ns, (work_ns + items_est * t_item * shape.n_kv_heads) / kResident) +
        2 * t_item;
    const int64_t item_budget_ns = std::max<int64_t>(call_ns / 2, 4 * t_tile);

    // wide items: no longer than a quarter of the time their launch is expected to take on
    // 256 compute units, and not so short that start-up dominates
    const int64_t wide_budget_ns = std::max<int64_t>(wide_work_ns / 256 / 4, 16 * t_wide);

    int64_t scap = opt.stream_chunk;
    if (direct) {
        scap = direct_cap;
    } else if (scap <= 0) {
        if (use_mfma) {
            scap = item_budget_ns / t_tile * kTile;
        } else {
            scap = round_up(ceil_div(own_total * shape.n_kv_heads, 2048), 32);
            scap = std::min<int64_t>(std::max<int64_t>(scap, 64), 2048);
        }
    }

    // shared lists: chunk counts first (they fix the slot numbering)
    std::vector<std::vector<Chunk>> shared_chunks(shared.size());
    for (size_t i = 0; i < shared.size(); ++i) {
        Shared& sh = shared[i];
        sh.prefix = sh.above < 0 ? 0 : shared[sh.above].prefix + shared[sh.above].n_chunks;
        int64_t ccap = opt.cascade_chunk;
        if (ccap <= 0 && sh.wide)
            ccap = wide_budget_ns / t_wide * kTile;
        else if (ccap <= 0)
            ccap = item_budget_ns / t_tile * kTile;
        pieces.clear();
        if (!collect_pieces(p, sh.nodes, own, pieces)) p.adv_in_place = false;
        if (!cut_runs(p, pieces, sh.tokens, ccap, piece, join, shared_chunks[i]))
            p.adv_in_place = false;
        sh.n_chunks = (int32_t)shared_chunks[i].size();
    }

    // per leaf query: the segments of its chain that no shared item reads are read
    // by the query itself, as one run list cut into items
    std::vector<int32_t> ent_pos(L, 0);
    for (int32_t i = 0; i < L; ++i) ent_pos[p.ent_order[i]] = i;
    {
        std::vector<int32_t> own_nodes;
        int64_t slot = 0;
        for (int32_t l = 0; l < L; ++l) {
            p.part_base[l] = (int32_t)slot;
            const int32_t e = ent_pos[l];
            const int32_t shared_slots =
                last_shared[e] < 0 ? 0 : shared[last_shared[e]].prefix + shared[last_shared[e]].n_chunks;
            slot += shared_slots;
            own_nodes.clear();
            own_segs(e, reads);
            for (size_t i = reads.size(); i-- > 0;)
                own_nodes.insert(own_nodes.end(), segs[reads[i]].nodes.begin(), segs[reads[i]].nodes.end());
            pieces.clear();
            if (!collect_pieces(p, own_nodes, own, pieces)) p.adv_in_place = false;
            int64_t tokens = 0;
            for (const Piece& x : pieces) tokens += x.n;
            if (!cut_runs(p, pieces, tokens, scap, piece, join, chunks, direct ? kDirectGrain : 32))
                p.adv_in_place = false;
            if (direct) p.direct_waves = std::max(p.direct_waves, std::max(1, (int32_t)chunks.size()));
            int32_t c_idx = 0;
            for (const Chunk& c : chunks) {
                if (slot >= std::numeric_limits<int32_t>::max()) return ETS_ERR_UNSUPPORTED;
                if (use_mfma) {
                    p.cascade_items.push_back(CascadeItem{c.run_begin, c.run_end, ent_pos[l], 1,
                                                          shared_slots + c_idx, c.tokens, p.groups ? 0 : 1, 0});
                    cascade_cost.push_back(ceil_div(c.tokens, kTile) * t_tile);
                    p.max_cascade_ent = std::max(p.max_cascade_ent, 1);
                } else {
                    p.stream_items.push_back(
                        StreamItem{l, c.run_begin, c.run_end, (int32_t)slot});
                    stream_tokens.push_back(c.tokens);
                }
                ++c_idx;
                ++slot;
            }
            if (slot >= std::numeric_limits<int32_t>::max()) return ETS_ERR_UNSUPPORTED;
        }
        p.part_base[L] = (int32_t)slot;
    }

    std::vector<int64_t> wide_cost;
    for (size_t i = 0; i < shared.size(); ++i) {
        const Shared& sh = shared[i];
        for (int32_t c = 0; c < sh.n_chunks; ++c) {
            const Chunk& ch = shared_chunks[i][c];
            const int64_t per_item = sh.wide ? ent_per_wide : ent_per_item;
            const int32_t sole = !p.groups && sh.n_ent <= per_item ? 1 : 0;
            for_items(sh, [&](int64_t e0, int64_t n) {
                const int32_t ne = (int32_t)n;
                const CascadeItem it{ch.run_begin, ch.run_end, sh.ent_begin + (int32_t)e0, ne,
                                     sh.prefix + c, ch.tokens, sole, 0};
                if (sh.wide) {
                    p.wide_items.push_back(it);
                    wide_cost.push_back(ceil_div(ch.tokens, kTile) * ceil_div((int64_t)ne * G, 32));
                } else {
                    p.cascade_items.push_back(it);
                    cascade_cost.push_back(ceil_div(ch.tokens, kTile) * t_tile);
                    p.max_cascade_ent = std::max(p.max_cascade_ent, ne);
                }
            });
        }
    }

    // longest items first, so that the tail of each launch is made of short ones
    if (!direct) {
        std::vector<int32_t> idx(p.stream_items.size());
        for (size_t i = 0; i < idx.size(); ++i) idx[i] = (int32_t)i;
        std::stable_sort(idx.begin(), idx.end(), [&](int32_t a, int32_t b) {
            return stream_tokens[a] > stream_tokens[b];
        });
        std::vector<StreamItem> sorted(idx.size());
        for (size_t i = 0; i < idx.size(); ++i) sorted[i] = p.stream_items[idx[i]];
        p.stream_items.swap(sorted);
    }
    {
        std::vector<int32_t> idx(p.wide_items.size());
        for (size_t i = 0; i < idx.size(); ++i) idx[i] = (int32_t)i;
        std::stable_sort(idx.begin(), idx.end(),
                         [&](int32_t a, int32_t b) { return wide_cost[a] > wide_cost[b]; });
        std::vector<CascadeItem> sorted(idx.size());
        for (size_t i = 0; i < idx.size(); ++i) sorted[i] = p.wide_items[idx[i]];
        p.wide_items.swap(sorted);
    }
    {
        std::vector<int32_t> idx(p.cascade_items.size());
        for (size_t i = 0; i < idx.size(); ++i) idx[i] = (int32_t)i;
        std::stable_sort(idx.begin(), idx.end(), [&](int32_t a, int32_t b) {
            return cascade_cost[a] > cascade_cost[b];
        });
        // Small items with at most 16 query rows follow the others (both groups longest
        // first): one wave walks such an item alone, four of them share a workgroup,
        // which divides the number of short workgroups the device has to start by four.
        std::vector<CascadeItem> sorted;
        sorted.reserve(idx.size());
        // A lone wave needs about 2.5 us per 16-token unit; such an item should not
        // last longer than a quarter of the time the whole call is expected to take.  Group kernel: 1.5 us and
        // six tenths; at most 256 tokens instead, 65 drawn trees, 0.95 to 1.16 times as long, geometric
        // mean 1.01, 128 tokens 0.97 to 1.29, 1.05, no such items 0.98 to 1.68, 1.18.
        const int64_t wave_cap = std::min<int64_t>(
            opt.wave_items, p.groups ? call_ns * 6 / 10 / 1500 * 16 : hbm_ns / 4 / 2500 * 16);
        auto small = [&](const CascadeItem& it) {
            return (int64_t)it.n_ent * G <= 16 && it.n_tokens <= wave_cap;
        };
        for (size_t i = 0; i < idx.size(); ++i)
            if (!small(p.cascade_items[idx[i]])) sorted.push_back(p.cascade_items[idx[i]]);
        p.n_single = (int32_t)sorted.size();
        for (size_t i = 0; i < idx.size(); ++i)
            if (small(p.cascade_items[idx[i]])) sorted.push_back(p.cascade_items[idx[i]]);
        p.cascade_items.swap(sorted);
        // Launch order.  Items with many query rows keep a workgroup slot busy for a long
        // time per byte they bring in from memory; items with few rows (a leaf's private
        // rows, segments shared by a handful of leaves) stream at the memory system's pace.
        // The device hands workgroups out in index order, so the two kinds are merged into
        // one sequence in which each advances at the same fraction of its total tokens:
        // memory traffic and arithmetic are then spread evenly over the launch instead of
        // following each other.  Within a kind the order stays longest first.
        const int64_t n_w = ((int64_t)p.cascade_items.size() - p.n_single + 3) / 4;
        std::vector<std::pair<int64_t, int32_t>> heavy, light;  // (tokens, code)
        for (int32_t i = 0; i < p.n_single; ++i) {
            const CascadeItem& it = p.cascade_items[(size_t)i];
            ((int64_t)it.n_ent * G > 16 ? heavy : light).push_back({it.n_tokens, i});
        }
        for (int64_t g = 0; g < n_w; ++g) {
            int64_t tok = 0;
            for (int64_t k = 4 * g; k < std::min<int64_t>(4 * g + 4, (int64_t)p.cascade_items.size() - p.n_single); ++k)
                tok += p.cascade_items[(size_t)(p.n_single + k)].n_tokens;
            light.push_back({tok, (int32_t)(-g - 1)});
        }
        p.wg_map.clear();
        p.wg_map.reserve(heavy.size() + light.size());
        // Longest first, whatever the kind, where the merged sequence would end the launch on a long item:
        //  - in units of few rounds over the resident workgroups.  Group kernel: the merged sequence is 3 to
        //    15 % slower up to three rounds, and as much faster from there on.  The other kernel, 82 drawn trees,
        //    merged over longest first: 0.98 to 1.24 up to five rounds, median 1.02 (64 diverging leaves 34.4 ->
        //    33.0 us, 100 leaves with head_dim 64 26.0 -> 23.7, 196 leaves of one query head 29.3 -> 24.6);
        //    0.95 to 1.03, median 0.98, from there to eight rounds, 0.96 to 1.03, median 0.99, beyond (12
        //    searches of 292 leaves 387 against 405);
        //  - where an item with many rows is handed out so late, at the same fraction of the tokens as the others,
        //    that it lasts a fifth of the call longer than is left of it (8 searches of 45 leaves under prompts of
        //    3 500 rows and a few short steps 101 us merged, 86 longest first; 4 of 137 120 and 99; 512
        //    leaves under one root of 33 000 rows 1 037 and 617; up to an eighth of the call 0.97 to 1.02).
        const int64_t n_units = ((int64_t)heavy.size() + (int64_t)light.size()) * shape.n_kv_heads;
        double overrun = 0;  // parts of the call (the items stand longest first)
        int64_t total = 0, handed = 0;
        for (const auto& x : heavy) total += x.first;
        for (const auto& x : heavy) {
            handed += x.first;
            overrun = std::max(overrun, (double)handed / total - 1 + (double)(ceil_div(x.first, kTile) * t_tile) / call_ns);
        }
        if (opt.interleave && (n_units < (p.groups ? 3 : 5) * kResident || overrun > 0.2)) {
            auto duration = [&](const std::pair<int64_t, int32_t>& u) {  // tenths of a microsecond
                if (u.second >= 0) {
                    const CascadeItem& it = p.cascade_items[(size_t)u.second];
                    const int64_t rows = (int64_t)it.n_ent * G;
                    if (!p.groups)  // (tiles of up to 64 rows; four waves that walk 16 tokens each)
                        return rows > 16 ? ceil_div(u.first, kTile) * 25 : ceil_div(u.first, kTile) * 16;
                    return rows > 64 ? ceil_div(u.first, kTile) * 21 : rows > 32 ? ceil_div(u.first, kTile) * 16
                           : rows > 16 ? ceil_div(u.first, kTile) * 14 : ceil_div(u.first, 2 * kTile) * 16;
                }
                // four small items
                const size_t first = (size_t)(p.n_single + 4 * (-(int64_t)u.second - 1));
                int64_t n = 0;
                for (size_t k = first; k < std::min(first + 4, p.cascade_items.size()); ++k)
                    n = std::max<int64_t>(n, p.cascade_items[k].n_tokens);
                return p.groups ? ceil_div(n, 32) * 16 : ceil_div(n, 16) * 14;
            };
            std::vector<std::pair<int64_t, int32_t>> all;
            for (const auto* kind : {&heavy, &light})
                for (const auto& u : *kind) all.push_back({duration(u), u.second});
            std::stable_sort(all.begin(), all.end(), [](const std::pair<int64_t, int32_t>& a, const std::pair<int64_t, int32_t>& b) {
                return a.first > b.first;
            });
            for (const auto& u : all) p.wg_map.push_back(u.second);
        } else if (!opt.interleave) {
            for (int32_t i = 0; i < p.n_single; ++i) p.wg_map.push_back(i);
            for (int64_t g = 0; g < n_w; ++g) p.wg_map.push_back((int32_t)(-g - 1));
        } else {
            auto by_tokens = [](const std::pair<int64_t, int32_t>& a,
                                const std::pair<int64_t, int32_t>& b) { return a.first > b.first; };
            // Where there are many of them (group kernel), items of more than 256 tokens come in the order of
            // their leaf queries, not of their lengths: neighbours walk the same rows from the root, and
            // what runs at the same time finds them in L2 (16 searches of 256 leaves: 10.8 GB read past L2
            // and 2 058 us in order of length, 8.9 GB and 1 893 us so).
            const bool by_place = p.groups && (int64_t)heavy.size() * shape.n_kv_heads > 8 * kResident;
            auto before = [&](const std::pair<int64_t, int32_t>& a, const std::pair<int64_t, int32_t>& b) {
                if (!by_place) return a.first > b.first;
                const bool la = a.first > 256, lb = b.first > 256;
                if (la != lb) return la;
                return p.cascade_items[(size_t)a.second].ent_begin < p.cascade_items[(size_t)b.second].ent_begin;
            };
            std::stable_sort(heavy.begin(), heavy.end(), before);
            std::stable_sort(light.begin(), light.end(), by_tokens);
            int64_t tot_h = 0, tot_l = 0, done_h = 0, done_l = 0;
            for (const auto& x : heavy) tot_h += std::max<int64_t>(x.first, 1);
            for (const auto& x : light) tot_l += std::max<int64_t>(x.first, 1);
            size_t ih = 0, il = 0;
            while (ih < heavy.size() || il < light.size()) {
                // the kind that lags behind in its own total goes next (fractions compared
                // without division: done_h / tot_h <= done_l / tot_l)
                const bool take_heavy =
                    il >= light.size() ||
                    (ih < heavy.size() && (__int128)done_h * tot_l <= (__int128)done_l * tot_h);
                if (take_heavy) {
                    p.wg_map.push_back(heavy[ih].second);
                    done_h += std::max<int64_t>(heavy[ih++].first, 1);
                } else {
                    p.wg_map.push_back(light[il].second);
                    done_l += std::max<int64_t>(light[il++].first, 1);
                }
            }
        }
    }

    if (p.runs.size() >= (size_t)std::numeric_limits<int32_t>::max() ||
        p.wg_map.size() >= (size_t)std::numeric_limits<int32_t>::max() / 16)
        return ETS_ERR_UNSUPPORTED;
    build_units(p, G);
    {
        std::vector<int32_t> first(N, -1);
        p.adv_node.clear();
        p.adv_src.clear();
        p.adv_last_row.clear();
        for (int32_t l = 0; l < L; ++l) {
            const int32_t n = p.leaf_node[l];
            if (first[n] >= 0) continue;
            first[n] = l;
            p.adv_node.push_back(n);
            p.adv_src.push_back(l);
            p.adv_last_row.push_back(p.n_tokens[n] > 0 ? grow_end_of(n) - 1 : kNoRow);
        }
        p.adv_room = piece > 0 ? 32 : std::numeric_limits<int32_t>::max();
    }
    p.ent_base.resize((size_t)L);
    for (int32_t i = 0; i < L; ++i) p.ent_base[i] = p.part_base[p.ent_order[i]];
    st.n_partials = p.part_base[L];
    // the kernels number partial rows, (leaf, head) pairs and workgroups with 32-bit integers
    const int64_t i32_max = std::numeric_limits<int32_t>::max();
    if (st.n_partials * shape.n_q_heads >= i32_max || (int64_t)L * shape.n_q_heads >= i32_max ||
        (int64_t)p.stream_items.size() * shape.n_kv_heads >= i32_max)
        return ETS_ERR_UNSUPPORTED;
    st.n_stream_items = (int64_t)p.stream_items.size();
    st.n_cascade_items = (int64_t)p.cascade_items.size();
    p.item_rows = p.cascade_items.empty() ? 0 : (int32_t)rows_per_item;
    st.n_wide_items = (int64_t)p.wide_items.size();
    st.workspace_bytes = st.n_partials * shape.n_q_heads * ((int64_t)shape.head_dim + 2) * 4;
    // The matrix-core kernel can run the merge itself when it writes every partial and every
    // leaf query has at least one (the wave that stores a leaf's last partial merges them).
    // (the merging kernel addresses the workspace with 32-bit byte offsets)
    bool can_fuse = use_mfma && L > 0 && p.stream_items.empty() && p.wide_items.empty() &&
                    !p.cascade_items.empty() &&
                    st.n_partials * shape.n_q_heads * shape.head_dim * 4 < (int64_t(1) << 31);
    for (int32_t l = 0; can_fuse && l < L; ++l) can_fuse = p.part_base[l + 1] > p.part_base[l];
    p.fused = can_fuse && (opt.fuse_merge == 1 || (opt.fuse_merge < 0 && fuse_by_default(st)));
    st.merge_fused = p.fused ? 1 : 0;
    p.valid = true;
    return ETS_OK;
}

}  // namespace

constexpr int32_t kMinJoinedRows = 8;
int32_t join_rows(Run& r, int64_t tok, int64_t avail) {
    const int32_t first = r.n, take = (int32_t)std::min<int64_t>(avail, kStepRows - first);
    const int64_t gap = tok - first - r.tok;
    if (r.join != 0 || first <= 0 || take <= 0 || gap > kMaxJoinGap || gap < -kMaxJoinGap) return 0;
    if (gap < 0 && (first + take < kStepRows || tok + take > r.tok)) return 0;
    if (first + take < kMinJoinedRows) return 0;
    r.n += take;
    r.join = join_code(first, gap);
    return take;
}

bool check_step(const Run& run, int64_t pool_rows) {
    if (run.n < 0 || run.n > kStepRows || run.tok < 0) return false;
    const StepSpan s = span_of(run.tok, run.n, run.join);
    const Join j = join_of(run.join);
    for (int32_t t = 0; t < kStepRows; ++t) {
        const int64_t off = (int64_t)t + (t < j.first ? s.low_shift : s.high_shift);
        if (t >= run.n) {
            if (off < s.size) return false;
            continue;
        }
        const int64_t row = run_row(run, t);
        if (off < 0 || off >= s.size || s.base + off != row || row < 0 || row >= pool_rows) return false;
    }
    return true;
}

void advance_tree(Plan& plan) {
    ets_stats& st = plan.stats;
    const int64_t tok_bytes = st.unique_tokens > 0 ? st.unique_kv_bytes / st.unique_tokens : 0;
    for (int32_t n : plan.adv_node) {
        plan.n_tokens[n] += 1;
        st.unique_tokens += 1;
        st.flat_tokens += plan.leaf_count[n];
        st.min_pool_tokens =
            std::max(st.min_pool_tokens, plan.tok_offset[n] + (int64_t)plan.n_tokens[n]);
    }
    if (tok_bytes > 0) {
        st.unique_kv_bytes = st.unique_tokens * tok_bytes;
        st.flat_kv_bytes = st.flat_tokens * tok_bytes;
    }
}

bool advance_in_place(Plan& plan) {
    if (!plan.valid || !plan.adv_in_place || plan.adv_room <= 0) return false;
    for (const AdvEntry& e : plan.adv) {
        Run& last = plan.runs[e.r_last];
        if (e.mergeable && (plan.piece == 0 || last.n < plan.piece)) {
            last.n += 1;
        } else {
            Run& spare = plan.runs[e.r_spare];
            if (spare.n == 0) spare.tok = e.end0 + plan.advances;
            spare.n += 1;
        }
    }
    refresh_units(plan);
    plan.advances += 1;
    plan.adv_room -= 1;
    advance_tree(plan);
    return true;
}

void chain_of(const Plan& plan, int32_t leaf, std::vector<int32_t>& out) {
    const size_t first = out.size();
    for (int32_t x = plan.leaf_node[leaf]; x >= 0; x = plan.parent[x]) out.push_back(x);
    std::reverse(out.begin() + (std::ptrdiff_t)first, out.end());
}

ets_status build_plan(const ets_shape& shape, const PlanOptions& opt, const ets_tree& tree,
                      int mode, Plan& plan) {
    plan.valid = false;
    if (mode != ETS_PLAN_TREE && mode != ETS_PLAN_FLAT) return ETS_ERR_INVALID_ARG;
    ets_status s = validate(tree);
    if (s != ETS_OK) return s;
    try {
        s = build(shape, opt, tree, mode, true, plan);
        // The group kernel's plans mostly have fewer partial results, but their shared lists can be cut finer: a
        // plan that fits the static scratch with items of 64 query rows keeps them if it would not fit
        // otherwise.  (The other plan has at least a partial result for every leaf query of a shared segment.)
        if (s == ETS_OK && plan.groups && plan.stats.workspace_bytes > ETS_STATIC_SCRATCH_BYTES &&
            plan.min_workspace_bytes <= ETS_STATIC_SCRATCH_BYTES) {
            Plan by64;
            if (build(shape, opt, tree, mode, false, by64) == ETS_OK &&
                by64.stats.workspace_bytes <= ETS_STATIC_SCRATCH_BYTES)
                plan = std::move(by64);
        }
        return s;
    } catch (const std::bad_alloc&) {
        plan.valid = false;
        return ETS_ERR_NOMEM;
    }
}

bool check_plan(const Plan& p, const ets_shape& shape, PlanCheck& out) {
    out = PlanCheck{};
    const int64_t L = (int64_t)p.leaf_node.size();
    const int G = shape.n_q_heads / shape.n_kv_heads;
    const int per_block = std::max(1, 16 / G);  // entries whose rows make up a 16-row block
    const int64_t n_runs = (int64_t)p.runs.size();
    out.entry_table_entries = (int64_t)p.ent_order.size() + kEntryPadding;
    auto bad = [&](bool cond) {
        if (cond) out.violations += 1;
    };
    auto entry_leaf = [&](int64_t idx) -> int64_t {  // padding entries hold zero
        return idx < (int64_t)p.ent_order.size() ? p.ent_order[(size_t)idx] : 0;
    };
    bad(p.ent_base.size() != p.ent_order.size());
    // every partial slot has exactly one writer: the merge reads all of a leaf's slots, and the
    // merge inside the attention launch starts when as many have arrived as the leaf has slots
    std::vector<char> written((size_t)std::max<int64_t>(p.stats.n_partials, 0), 0);
    auto writes = [&](int64_t slot) {
        if (slot < 0 || slot >= (int64_t)written.size() || written[(size_t)slot]++) out.violations += 1;
    };
    for (size_t i = 0; i < p.cascade_items.size(); ++i) {
        const CascadeItem& it = p.cascade_items[i];
        const bool wave_item = (int64_t)i >= p.n_single;
        out.items += 1;
        // the step list
        bad(it.run_begin < 0 || it.run_end < it.run_begin || it.run_end > n_runs);
        if (!wave_item) bad(it.run_end - it.run_begin > kTreeAttnMaxSteps);
        for (int64_t r = it.run_begin; r < it.run_end && r < n_runs; ++r) {
            const Run& run = p.runs[(size_t)r];
            bad(!check_step(run, p.stats.min_pool_tokens));
            for (int32_t t = 0; t < run.n; ++t) out.max_pool_row = std::max(out.max_pool_row, run_row(run, t));
        }
        // the entries: every wave loads 16 consecutive entries from its block's first one
        const int64_t R = (int64_t)it.n_ent * G;
        bad(it.n_ent < 1 || R > (p.groups ? kGroupRowsPerItem : kTreeAttnRowsPerItem) || it.ent_begin < 0 ||
            (int64_t)it.ent_begin + it.n_ent > L);
        if (wave_item) bad(R > 16);
        const bool rowpar = R > 16;
        const int n_blocks = (int)((R + 15) / 16);
        for (int blk = 0; blk < (rowpar ? n_blocks : 1); ++blk) {
            const int64_t first = (int64_t)it.ent_begin + (16 * blk) / G;
            const int64_t last_loaded = first + 15;
            out.max_entry_index = std::max(out.max_entry_index, last_loaded);
            out.max_entry_overreach = std::max(
                out.max_entry_overreach, last_loaded - ((int64_t)it.ent_begin + it.n_ent - 1));
            bad(last_loaded >= out.entry_table_entries);
            // the entries whose query rows the wave fetches (rows past R included)
            for (int k = 0; k < per_block; ++k) {
                const int64_t leaf = entry_leaf(first + k);
                bad(leaf < 0 || leaf >= std::max<int64_t>(L, 1));
            }
        }
        // the partial rows it writes
        for (int32_t e = 0; e < it.n_ent && (int64_t)it.ent_begin + e < L; ++e) {
            const int32_t leaf = p.ent_order[(size_t)(it.ent_begin + e)];
            const int64_t slot = (int64_t)p.part_base[(size_t)leaf] + it.slot_off;
            bad(it.slot_off < 0 || slot >= p.part_base[(size_t)leaf + 1]);
            writes(slot);
            out.max_partial_row =
                std::max(out.max_partial_row, slot * shape.n_q_heads + shape.n_q_heads - 1);
        }
    }
    // wide items: a lane looks up the entry of its own query row, clamped to the item's last
    for (const CascadeItem& it : p.wide_items) {
        out.items += 1;
        bad(it.run_begin < 0 || it.run_end < it.run_begin || it.run_end > n_runs);
        bad(it.n_ent < 1 || (int64_t)it.n_ent * G > kWideRowsPerItem || it.ent_begin < 0 ||
            (int64_t)it.ent_begin + it.n_ent > L);
        out.max_entry_index = std::max(out.max_entry_index, (int64_t)it.ent_begin + it.n_ent - 1);
        for (int64_t r = it.run_begin; r < it.run_end && r < n_runs; ++r) {
            const Run& run = p.runs[(size_t)r];
            bad(run.n < 0 || run.n > 32 || run.tok < 0 || run.join != 0);
            if (run.n > 0) {
                bad(run.tok + run.n > p.stats.min_pool_tokens);
                out.max_pool_row = std::max(out.max_pool_row, run.tok + run.n - 1);
            }
        }
        for (int32_t e = 0; e < it.n_ent && (int64_t)it.ent_begin + e < L; ++e) {
            const int32_t leaf = p.ent_order[(size_t)(it.ent_begin + e)];
            const int64_t slot = (int64_t)p.part_base[(size_t)leaf] + it.slot_off;
            bad(it.slot_off < 0 || slot >= p.part_base[(size_t)leaf + 1]);
            writes(slot);
            out.max_partial_row =
                std::max(out.max_partial_row, slot * shape.n_q_heads + shape.n_q_heads - 1);
        }
    }
    for (size_t i = 0; p.direct_waves > 0 && i < p.stream_items.size(); ++i)
        bad(p.stream_items[i].slot != (int64_t)i);
    for (int64_t l = 0; p.direct_waves > 0 && l < L; ++l)
        bad(p.part_base[(size_t)l + 1] - p.part_base[(size_t)l] > std::min(p.direct_waves, kDirectWaves));
    for (const StreamItem& it : p.stream_items) {
        out.items += 1;
        bad(it.run_begin < 0 || it.run_end < it.run_begin || it.run_end > n_runs);
        bad(it.entry < 0 || it.entry >= L);
        if (it.entry >= 0 && it.entry < L)
            bad(it.slot < p.part_base[(size_t)it.entry] || it.slot >= p.part_base[(size_t)it.entry + 1]);
        writes(it.slot);
        out.max_partial_row = std::max(
            out.max_partial_row, (int64_t)it.slot * shape.n_q_heads + shape.n_q_heads - 1);
        for (int64_t r = it.run_begin; r < it.run_end && r < n_runs; ++r) {
            const Run& run = p.runs[(size_t)r];
            bad(run.n < 0 || run.tok < 0 || run.join != 0);
            if (run.n > 0) {
                bad(run.tok + run.n > p.stats.min_pool_tokens);
                out.max_pool_row = std::max(out.max_pool_row, run.tok + run.n - 1);
            }
        }
    }
    // the unit table says what the launch order and the step lists say
    bad(p.units.size() != 4 * p.wg_map.size());
    for (size_t y = 0; y < p.wg_map.size() && 4 * y + 3 < p.units.size(); ++y) {
        const int32_t code = p.wg_map[y];
        for (int w = 0; w < 4; ++w) {
            const UnitSlot& u = p.units[4 * y + (size_t)w];
            const int64_t idx = code >= 0 ? code : p.n_single + 4 * (-(int64_t)code - 1) + w;
            if (idx < 0 || idx >= (int64_t)p.cascade_items.size()) {
                bad(u.item.n_ent != 0);
                continue;
            }
            const CascadeItem& it = p.cascade_items[(size_t)idx];
            bad(u.item.run_begin != it.run_begin || u.item.run_end != it.run_end ||
                u.item.ent_begin != it.ent_begin || u.item.n_ent != it.n_ent ||
                u.item.slot_off != it.slot_off || u.item.sole_reader != it.sole_reader ||
                u.item.wave_item != unit_kind(p, code, it, G));
            const Run* held[2] = {&u.first, &u.second};
            for (int j = 0; j < 2; ++j) {
                const int k = unit_step_index(u.item, w, j);
                const int64_t r = (int64_t)it.run_begin + k;
                if (k >= 0 && r < it.run_end && r < n_runs)
                    bad(held[j]->tok != p.runs[(size_t)r].tok || held[j]->n != p.runs[(size_t)r].n ||
                        held[j]->join != p.runs[(size_t)r].join);
                else
                    bad(held[j]->n != 0);
            }
        }
    }
    // the launch order names every item that takes a workgroup and every group of small
    // items exactly once
    {
        const int64_t n_w = ((int64_t)p.cascade_items.size() - p.n_single + 3) / 4;
        bad((int64_t)p.wg_map.size() != p.n_single + n_w);
        std::vector<char> seen_single((size_t)p.n_single, 0), seen_group((size_t)n_w, 0);
        for (int32_t code : p.wg_map) {
            if (code >= 0) {
                if (code >= p.n_single || seen_single[(size_t)code]++) out.violations += 1;
            } else {
                const int64_t g = -(int64_t)code - 1;
                if (g >= n_w || seen_group[(size_t)g]++) out.violations += 1;
            }
        }
    }
    bad(out.max_partial_row >= p.stats.n_partials * shape.n_q_heads);
    for (char w : written) bad(w != 1);
    if (p.fused) {
        // only the matrix-core kernel's own items count arrivals, and a leaf query without a
        // partial would never be merged
        bad(!p.stream_items.empty() || !p.wide_items.empty());
        for (int64_t l = 0; l < L; ++l) bad(p.part_base[(size_t)l + 1] <= p.part_base[(size_t)l]);
    }
    return out.violations == 0;
}

bool leaf_cover(const Plan& plan, int32_t leaf, std::vector<int64_t>& rows,
                int32_t& n_partials) {
    const int32_t base = plan.part_base[leaf];
    n_partials = plan.part_base[leaf + 1] - base;
    // run range of every slot of this leaf, taken from the work items themselves
    std::vector<std::pair<int32_t, int32_t>> by_slot((size_t)n_partials, {-1, -1});
    bool ok = true;
    auto put = [&](int32_t slot, int32_t rb, int32_t re) {
        const int32_t k = slot - base;
        if (k < 0 || k >= n_partials || by_slot[k].first >= 0) {
            ok = false;
            return;
        }
        by_slot[k] = {rb, re};
    };
    for (const StreamItem& it : plan.stream_items)
        if (it.entry == leaf) put(it.slot, it.run_begin, it.run_end);
    for (const std::vector<CascadeItem>* items : {&plan.cascade_items, &plan.wide_items})
        for (const CascadeItem& it : *items)
            for (int32_t i = 0; i < it.n_ent; ++i)
                if (plan.ent_order[it.ent_begin + i] == leaf)
                    put(base + it.slot_off, it.run_begin, it.run_end);
    rows.clear();
    for (const auto& rr : by_slot) {
        if (rr.first < 0) {
            ok = false;
            continue;
        }
        for (int32_t r = rr.first; r < rr.second; ++r)
            for (int32_t t = 0; t < plan.runs[r].n; ++t) rows.push_back(run_row(plan.runs[r], t));
    }
    return ok;
}

}  // namespace ets
