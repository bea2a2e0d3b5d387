// Step-prefill attention on the matrix cores: one workgroup of four wavefronts = one
// block of query tokens of a leaf query's node, one kv head.
//
// Scoring a new step with the reward model is a prefill of that step's tokens over the
// tree of cached steps: query token i of the node sees every row of the node's strict
// ancestors and rows 0..i of the node itself.  A workgroup takes up to 256 query rows
// (256 / G consecutive tokens x the G query heads of the kv head) through its runs with 64 rows per
// wave, or 32 where the item has at most 128 (template parameter NB: blocks of 32 rows per
// wave; below, NB = 2): the ancestors' rows, then the node's own rows up to its last token, 64
// rows (two runs of at most 32) at a time through LDS.  It keeps the running softmax of its rows
// in registers:
// there are no partial results and no merge, the normalised output leaves at the end.
// Every K/V row a workgroup reads (512 bytes per kv head) meets 256 query rows, 256 flop
// per byte: with 128 rows the walk was bound by the 5.8 TB/s at which L2 and the memory
// side cache feed the compute units, not by the matrix cores.  Blocks of the same node
// and of sibling nodes run next to each other and find their shared ancestors in L2.
//
// Bound: the issue of instructions next to the matrix cores.  One wave per SIMD owns 64 query
// rows (two blocks of 32), so that every K and V fragment read from LDS feeds two matrix
// instructions: with 32 rows per wave, eight waves read 128 KB per run, 640 of the 1 024
// cycles that the matrix instructions take even without a bank conflict.  Lane l = (n, g),
// n = l % 32, g = l / 32.  Per run of 32 rows and block of 32 query rows:
//   S^T = K Q^T     8 x v_mfma_f32_32x32x16_bf16: run rows on M, query rows on N.  A = K
//                   rows from the LDS tile (lane (n, g): row n, d = 16 kk + 8 g .. + 7),
//                   B = Q in registers.  Lane (n, g) receives query row n against run
//                   rows 8 c + 4 g + r (c, r = 0..3);
//   hide            rows past the end of a short run (t >= n_run) get -3.4e38 from one more matrix
//                   instruction, in every run alike: with steps of some forty tokens every second
//                   run is a short one;
//   mask            rows of the querying node: row t counts iff kpos + t <= i_row, kpos being
//                   the run's position inside the node.  Runs that are seen in full branch past it;
//   softmax         against a per-row reference that is raised only when a score exceeds
//                   it by 2^8 in weight (then one cross-lane exchange);
//   O^T += V^T P^T  8 x v_mfma_f32_32x32x16_f16: d on M (4 blocks of 32), query rows on
//                   N, run rows on the contraction (2 halves of 16).  P rounded to fp16
//                   sits in the B layout as it is when contraction slot 8 g + 4 c' + r
//                   of half t stands for run row 16 t + 8 c' + 4 g + r; V, converted to
//                   fp16 while it is staged, is written to LDS as A fragments in that
//                   slot order.
// The work on a run is software pipelined inside the wave (prefill_unit), and the pipeline
// runs on across tiles.  Three tile buffers rotate, so that the next tile can be staged
// while the previous one may still be read by a slower wave: one barrier per tile (new
// contents visible), and the staging is spread over the gaps of the matrix instructions.
// K and V are fetched with range-checked buffer loads two and a half tiles ahead of their
// use (two register sets alternate; one tile ahead left the waves waiting for memory).
// Each wave fetches and stages half a run (16 rows, 16 bytes per lane and load) of K and of V.
// A run that its node does not fill goes on in the next piece of the path (Run::join): a run costs the same
// however many rows it has, and with nodes of some hundred tokens 4 to 6 % of the walk, with nodes of 16 to
// 64 up to 40 %, were rows that are not there.  128 steps of 10 to 14 tokens over 100 such steps, 8 heads:
// 240 -> 163 us; 64 steps of 100 to 150 tokens over 16, E4M3 pools: 447 -> 443; 256 ragged steps of 8 heads
// 7.55 -> 7.25 ms.
// The run list can be long (a path of thousands of rows), so its descriptors travel through
// a ring of 256 entries in LDS that is refilled 128 at a time: tile t reads descriptors up to
// 2 t + 9, and a refill at tile t writes those from 2 t + 128 on, 60 tiles ahead of their use.
//
// Measured against eight waves of 32 rows: 256 workgroups of 256 rows over one path of 16.8 k rows,
// 526 runs: 529 us = 1.0 us per run (585), of 128 rows: 331 us = 0.63 us per run (355).  38 k query
// tokens of 8 heads each over 5.4 k rows: 7.7 ms (8.5); 512 steps of up to 512 tokens over 13 k rows:
// 32.6 ms (36.0).  In that launch the matrix pipes are busy 55 % of the cycles; a
// wave issues for 66 % of its time, waits to issue for 12 % and for data or at barriers for 22 %.
// With joined runs the same launch takes 31.9 ms = 997 TFLOP/s (without, in turn on one box, 32.9).
//
// The same kernel serves decode attention for tree segments that MANY leaf queries share
// (template parameter DECODE): there the 256 query rows of a work item are up to 256 / G
// leaf queries x the G query heads of the kv head, every row sees every row of the item's
// runs, and instead of a normalised output the workgroup leaves the unnormalised partial
// (o, m, l) of each query row in the decode workspace, where the log-sum-exp merge picks
// it up.  A root prompt shared by 512 leaves is 2048 query rows per kv head: that is this
// kernel's shape of problem (bound by the matrix cores), not the streaming kernel's.
#pragma once

#include "device_utils.hpp"
#include "prefill_plan.h"
#include "tree_attn_kernel.hpp"

namespace ets {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

#define ETS_INLINE __attribute__((always_inline))  // a lambda the wave's registers pass through

constexpr int kPrefillThreads = 256;  // four waves of up to 64 query rows

// The matrix instructions of the inner loop, with the register file of every operand named: a
// wave holds 128 registers of O, 64 of Q, 32 of scores, 32 of weights, 64 of rows in flight and
// 48 of fragments.  What the vector unit works on (scores, weights, and O when it is scaled) goes to
// the ordinary registers; what only memory, LDS and matrix instructions touch (Q, fragments)
// to the accumulation registers.  Left to itself the compiler puts every accumulator on the
// other side and spills.
// The compiler does not know what these statements are, so the wait states between a matrix
// instruction and its neighbours are the code's own business: mfma_result_wait() before the
// vector unit reads a result that may be younger than 18 issue slots, and no vector instruction
// that writes an operand within two slots of its use.  (Accumulating into the same registers
// needs none; fragments come from LDS and are waited for as usual.)  Where a sequence of them starts,
// behind code that may copy registers, the first one waits its two slots itself (0 to 0.4 % of a
// call), and the rows are waited for where the loop is left.  Inside a sequence it rests on the
// register allocator not placing a copy in front of an instruction, as is the case with the compiler
// of ROCm 7.2.0; tests/test_matrix_wait_states.py follows every path of the built code.
__device__ __forceinline__ void mfma_scores_first(f32x16_t& s, u32x4_t k, bf16x8_t q) {
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "a"(k), "a"(q));
}
__device__ __forceinline__ void mfma_scores(f32x16_t& s, u32x4_t k, bf16x8_t q) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "a"(k), "a"(q));
}
// s += rows x low, see `missing` in prefill_item.
__device__ __forceinline__ void mfma_hide(f32x16_t& s, u32x2_t rows, u32x2_t low) {
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x8_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(rows), "a"(low));
}
__device__ __forceinline__ void mfma_apply(f32x16_t& o, u32x4_t v, u32x4_t p) {
    asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(o) : "a"(v), "v"(p));
}
__device__ __forceinline__ void mfma_apply_first(f32x16_t& o, u32x4_t v, u32x4_t p) {
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(o) : "a"(v), "v"(p));
}
__device__ __forceinline__ void mfma_result_wait(f32x16_t (&o)[4]) {
    asm volatile("s_nop 15\n\ts_nop 15" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]), "+v"(o[3]));
}
__device__ __forceinline__ void mfma_result_wait(f32x16_t& s) {
    asm volatile("s_nop 15\n\ts_nop 15" : "+v"(s));
}

// Masks the run rows the lane's query does not see (lim = rows of the run it sees, may
// be <= 0).  Score i stands for run row 8 (i / 4) + 4 g + i % 4.
__device__ __forceinline__ void prefill_mask(f32x16_t& s, int g, int lim) {
    const int rem = lim - 4 * g;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = (8 * (i >> 2) + (i & 3)) < rem ? s[i] : -INFINITY;
}

// Two weights rounded to fp16 (nearest even), the first in the low half.
__device__ __forceinline__ uint32_t f16_pair(float lo, float hi) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{lo, hi}), f16x2_t));
}

// K rows in LDS: 16 units of 16 bytes and one of padding (a fragment read takes one unit of 32
// rows: 17 n visits every bank group once whichever sixteen rows meet).
constexpr int kPrefillKRow = 17;
// V^T fragments in LDS.  The 16 rows of half a run are kept as 16-byte slots, one per output
// element d = 8 a + x and row group g: the eight contraction slots that lane (d % 32, g) of d
// block d / 32 feeds to the matrix instruction.  Slot (x, g, a) sits at 36 x + 16 g + a: a writer's
// 16 lanes (all a) and the sixteen lanes of a read that meet ({0..3, 12..15, 20..27} or {4..11,
// 16..19, 28..31} of 8 a + x) then touch every bank group once (34 x + .. takes 256 cycles
// for 32 reads of four waves instead of 160), and both address them with one register and
// constant offsets.
constexpr int kVFragX = 36 * 16;        // bytes between elements x and x + 1
constexpr int kVFragHalf = 8 * kVFragX; // bytes of half a run

// A condition that hardly ever holds: its code is kept out of the way.  With one wave per SIMD a
// branch that is taken costs about 100 cycles until instructions arrive from its target.
#define ETS_RARE(x) __builtin_expect(!!(x), 0)

// What a wave carries from run to run: NB blocks of 32 query rows.
template <int NB>
struct PrefillState {
    bf16x8_t qf[NB][8];   // query rows as B operands
    f32x16_t s[2];        // NB = 2: scores of the newest run, per block; NB = 1: of two runs in turn
    f32x16_t oacc[NB][4]; // d block x: lane (n, g) holds d = 32 x + 8 c + 4 g + r at index 4 c + r
    u32x4_t kf[8];        // K fragments of the run after it
    float m[NB], nmc[NB];  // reference score of the lane's row (-inf: none yet); minus the same times
                         // scale_log2e (0 without one)
    float lsum[NB];       // sum of the weights of the runs that are through
    float rsum[NB];       // sum of the weights of the run under way
    float alpha[NB];      // factor of oacc after the application under way, if it is to be scaled
    float p_even, p_last;  // weights under way: of an even score, and the newest one
    float pair;           // sum of the last two
};
constexpr int kEarlyWeights = 4;  // weights of block 0 beside the scores of block 1
constexpr int kLateWeights = 8;   // weights of block 1 that the next stage computes

// Largest of a lane's scores.  (The instruction itself: around fmaxf the compiler first
// canonicalises values whose origin it does not know, one more instruction for each.)
__device__ __forceinline__ float prefill_max(const f32x16_t& s) {
    float mx;
    asm volatile(
        "v_max_f32 %0, %1, %2\n\tv_max3_f32 %0, %0, %3, %4\n\tv_max3_f32 %0, %0, %5, %6\n\t"
        "v_max3_f32 %0, %0, %7, %8\n\tv_max3_f32 %0, %0, %9, %10\n\tv_max3_f32 %0, %0, %11, %12\n\t"
        "v_max3_f32 %0, %0, %13, %14\n\tv_max3_f32 %0, %0, %15, %16"
        : "=&v"(mx)
        : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]), "v"(s[4]), "v"(s[5]), "v"(s[6]), "v"(s[7]),
          "v"(s[8]), "v"(s[9]), "v"(s[10]), "v"(s[11]), "v"(s[12]), "v"(s[13]), "v"(s[14]), "v"(s[15]));
    return mx;
}
// Raises the row's reference to the largest score of the run when one exceeds it by more than
// the margin.  What has been gathered under the old reference is scaled: the sum at once, the
// output rows when the caller has applied the weights still under way.
template <int NB>
__device__ __forceinline__ void prefill_raise(PrefillState<NB>& st, int j, float mx, float scale_log2e) {
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));  // the row's other half of the run
    const float m_new = fmaxf(st.m[j], mx);
    // (a row that has seen nothing yet keeps -inf, and what it gathered is zero)
    st.alpha[j] = st.m[j] == -INFINITY ? 0.f : fast_exp2((st.m[j] - m_new) * scale_log2e);
    st.nmc[j] = m_new == -INFINITY ? 0.f : -m_new * scale_log2e;
    st.m[j] = m_new;
    st.lsum[j] *= st.alpha[j];
}
template <int NB>
__device__ __forceinline__ void scale_rows(PrefillState<NB>& st, int j) {
    mfma_result_wait(st.oacc[j]);
#pragma unroll
    for (int x = 0; x < 4; ++x) st.oacc[j][x] *= st.alpha[j];
}

// Weight i of block j, taken against the row's reference score, in two steps so that nothing
// waits for the exponential.  The empty statements hold the arithmetic where it is written: the
// compiler would otherwise sink it behind the next branch, away from the matrix instructions.
// A run's weights are summed in pairs into a sum of the run, and that goes to the row's sum once:
// as many additions as adding each weight to the row's sum, a sixteenth of them rounded at its
// size (300 runs of equal weights: the log-sum-exp is off by 5e-6 at most instead of 7e-5).
template <int NB>
__device__ __forceinline__ void weight_begin(PrefillState<NB>& st, const f32x16_t& s, int j, int i,
                                             float scale_log2e) {
    st.p_last = fast_exp2(fmaf(s[i], scale_log2e, st.nmc[j]));
}
template <int NB>
__device__ __forceinline__ void weight_end(PrefillState<NB>& st, u32x4_t (&pf)[2][2], int j, int i) {
    if (i & 1) {
        st.pair = st.p_even + st.p_last;
        uint32_t h = f16_pair(st.p_even, st.p_last);
        asm volatile("" : "+v"(h));
        pf[j][i >> 3][(i & 7) >> 1] = h;
        if (i == 15) {
            st.lsum[j] += st.rsum[j] + st.pair;
            asm volatile("" : "+v"(st.lsum[j]));
        }
    } else {
        // (a pair is added to the run's sum beside the next even weight: one addition to each gap)
        if (i >= 2) {
            st.rsum[j] = i == 2 ? st.pair : st.rsum[j] + st.pair;
            asm volatile("" : "+v"(st.rsum[j]));
        }
        st.p_even = st.p_last;
    }
}

// One pipeline stage of a wave: the scores of run u + 1 and the application of run u.
//   A, block 0   scores(u + 1)  ||  the last weights of block 1 of run u
//   A, block 1   scores(u + 1)  ||  block 0 of run u + 1: mask, maximum, first weights
//   B            apply(u)       ||  its other weights; block 1: mask, maximum, first weights
// Written in the order in which it is to be issued: matrix and vector instructions of one wave
// overlap only when they alternate in program order, and a scheduling fence keeps each group
// together.  A matrix instruction takes 32 cycles and 8 of issue, which leaves 24 for other
// instructions behind it (measured: 6 multiply-adds are free, the seventh costs its 4 cycles);
// a weight takes 18 (an exponential 8, a multiply-add and an addition 4 each, half a conversion
// 2), so a run's 32 weights, the staging and the rest fill the 32 gaps of a stage almost completely
// and have to be spread evenly.  The scores of a block are read by the vector unit behind
// three later matrix instructions (24 passes; the result takes 16).  Fragments are read from LDS
// eight matrix steps ahead of their use: kf holds the K fragments of run u + 1 on entry and
// of run u + 2 on exit, read behind `before_b` (a workgroup barrier where that run's tile has
// just been staged).
//   v_run, k_after   LDS byte addresses: the lane's slot of run u's V^T fragments, and its row of
//                    run u + 2's K
//   fill(k)          k = 0..15: the caller's work beside A;  fill_b(i), i = 0..15: beside B
//   missing, low     operands of mfma_hide for run u + 1 (HIDE)
//   hidden, mask(s, j)  whether rows of run u + 1 are newer than a query token, and what hides
//                    them from block j's scores s
//   rare, rare_b(s, j)  the same for the last block, with whatever else of the caller's is rarely to be done
//                    ahead of fill_b(3): one branch for both
template <bool HIDE, class Fill, class Mask, class Before, class Rare, class FillB>
__device__ __forceinline__ void prefill_unit(PrefillState<2>& st, const char* __restrict__ v_run,
                                             const char* __restrict__ k_after,
                                             u32x4_t (&pf_cur)[2][2], u32x4_t (&pf)[2][2],
                                             float scale_log2e, float raise_margin, u32x2_t missing,
                                             u32x2_t low, bool hidden, Fill fill, Mask mask,
                                             Before before_b, bool rare, Rare rare_b, FillB fill_b) {
    u32x4_t vf[8];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        if (kk == 0) mfma_scores_first(st.s[0], st.kf[0], st.qf[0][0]);
        else mfma_scores(st.s[0], st.kf[kk], st.qf[0][kk]);
        __builtin_amdgcn_sched_barrier(0);
        vf[kk] = load16(v_run + (kk >> 2) * kVFragHalf + (kk & 3) * 64);  // half kk / 4, d block kk % 4
        if (kk > 0) weight_end(st, pf_cur, 1, 16 - kLateWeights + kk - 1);
        weight_begin(st, st.s[1], 1, 16 - kLateWeights + kk, scale_log2e);
        fill(kk);
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (HIDE) mfma_hide(st.s[0], missing, low);
    bool raised0 = false, raised1 = false;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        if (kk == 0) mfma_scores_first(st.s[1], st.kf[0], st.qf[1][0]);
        else mfma_scores(st.s[1], st.kf[kk], st.qf[1][kk]);
        __builtin_amdgcn_sched_barrier(0);
        if (kk == 0) weight_end(st, pf_cur, 1, 15);
        fill(8 + kk);
        if (kk == 2 && ETS_RARE(hidden)) mask(st.s[0], 0);
        if (kk == 3) {
            const float mx = prefill_max(st.s[0]);
            raised0 = __any(mx > st.m[0] + raise_margin);
            if (ETS_RARE(raised0)) prefill_raise(st, 0, mx, scale_log2e);
        }
        if (kk > 8 - kEarlyWeights) weight_end(st, pf, 0, kk - 9 + kEarlyWeights);
        if (kk >= 8 - kEarlyWeights) weight_begin(st, st.s[0], 0, kk - 8 + kEarlyWeights, scale_log2e);
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (HIDE) mfma_hide(st.s[1], missing, low);
    before_b();
    __builtin_amdgcn_sched_barrier(0);
    // the other weights of block 0, then those of block 1 that are not late
    constexpr int kRest0 = 16 - kEarlyWeights, kRest = kRest0 + 16 - kLateWeights;
    auto begin = [&](int k) {
        if (k < kRest0) weight_begin(st, st.s[0], 0, kEarlyWeights + k, scale_log2e);
        else weight_begin(st, st.s[1], 1, k - kRest0, scale_log2e);
    };
    auto end = [&](int k) {
        if (k < 0) weight_end(st, pf, 0, kEarlyWeights - 1);
        else if (k < kRest0) weight_end(st, pf, 0, kEarlyWeights + k);
        else weight_end(st, pf, 1, k - kRest0);
    };
    int k = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        // half t of the run, d block x, query block j
        const int t = i >> 3, x = (i >> 1) & 3, j = i & 1;
        if (i == 0) mfma_apply_first(st.oacc[j][x], vf[4 * t + x], pf_cur[j][t]);
        else mfma_apply(st.oacc[j][x], vf[4 * t + x], pf_cur[j][t]);
        __builtin_amdgcn_sched_barrier(0);
        if (j == 1) st.kf[i >> 1] = load16(k_after + 32 * (i >> 1));
        if (i == 2 && ETS_RARE(rare)) rare_b(st.s[1], 1);
        if (i == 3) {
            const float mx = prefill_max(st.s[1]);
            raised1 = __any(mx > st.m[1] + raise_margin);
            if (ETS_RARE(raised1)) prefill_raise(st, 1, mx, scale_log2e);
        } else {
            // one weight beside an instruction, two beside every third until none is too many
            end(k - 1);
            begin(k++);
            if (i % 3 == 0 && kRest - k > 15 - i - (i < 3 ? 1 : 0)) {
                end(k - 1);
                begin(k++);
            }
        }
        fill_b(i);
        __builtin_amdgcn_sched_barrier(0);
    }
    static_assert(kRest == 20, "15 instructions take a weight, five of them two");
    end(kRest - 1);
    if (ETS_RARE(raised0)) scale_rows(st, 0);
    if (ETS_RARE(raised1)) scale_rows(st, 1);
}

// The same for one block of 32 query rows per wave (small launches, see build_prefill_plan).  The
// scores alternate between st.s[ODD] (run u, complete) and st.s[1 - ODD] (run u + 1):
//   A   scores(u + 1), rows past the end of a short run hidden  ||  weights of run u
//   B   apply(u)       ||  staging and loads; mask and maximum of run u + 1
template <int ODD, class Fill, class Before, class Rare, class FillB>
__device__ __forceinline__ void prefill_unit1(PrefillState<1>& st, const char* __restrict__ v_run,
                                              const char* __restrict__ k_after, u32x4_t (&pf)[2][2],
                                              float scale_log2e, float raise_margin, u32x2_t missing,
                                              u32x2_t low, Fill fill, Before before_b, bool rare,
                                              Rare rare_b, FillB fill_b) {
    u32x4_t vf[8];
    f32x16_t& s_cur = st.s[ODD];
    f32x16_t& s_next = st.s[1 - ODD];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        if (kk == 0) mfma_scores_first(s_next, st.kf[0], st.qf[0][0]);
        else mfma_scores(s_next, st.kf[kk], st.qf[0][kk]);
        __builtin_amdgcn_sched_barrier(0);
        vf[kk] = load16(v_run + (kk >> 2) * kVFragHalf + (kk & 3) * 64);
        if (kk > 0) weight_end(st, pf, 0, 2 * kk - 1);
        weight_begin(st, s_cur, 0, 2 * kk, scale_log2e);
        weight_end(st, pf, 0, 2 * kk);
        weight_begin(st, s_cur, 0, 2 * kk + 1, scale_log2e);
        fill(2 * kk);
        fill(2 * kk + 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    mfma_hide(s_next, missing, low);
    weight_end(st, pf, 0, 15);
    before_b();
    __builtin_amdgcn_sched_barrier(0);
    bool raised = false;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i == 0) mfma_apply_first(st.oacc[0][i & 3], vf[i], pf[0][i >> 2]);
        else mfma_apply(st.oacc[0][i & 3], vf[i], pf[0][i >> 2]);
        __builtin_amdgcn_sched_barrier(0);
        st.kf[i] = load16(k_after + 32 * i);
        if (i == 2 && ETS_RARE(rare)) rare_b(s_next, 0);
        if (i == 3) {
            const float mx = prefill_max(s_next);
            raised = __any(mx > st.m[0] + raise_margin);
            if (ETS_RARE(raised)) prefill_raise(st, 0, mx, scale_log2e);
        }
        fill_b(2 * i);
        fill_b(2 * i + 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (ETS_RARE(raised)) scale_rows(st, 0);
}

// LDS of a workgroup: three tile buffers (K rows, behind them the V^T fragments [run][half]) and the
// ring of run descriptors.
constexpr int kPrefillKRowB = 16 * kPrefillKRow;  // bytes of a K row (272)
constexpr int kPrefillKB = 64 * kPrefillKRowB;    // K tile: 64 rows
constexpr int kPrefillBufB = kPrefillKB + 4 * kVFragHalf;
constexpr int kPrefillRing = 256;

// A work item, in the terms both modes share: its runs, and the number of row groups (query tokens,
// or leaf queries) whose G heads make up its query rows.
struct PrefillWork {
    int run_begin, run_end, n_grp;
    int tok0;           // step prefill: first query token, as an index into its node
    int n_anc;          // and the runs ahead of the node's own
    int64_t q_row0;     // and its query row
    int ent_begin;      // decode: first entry of its leaf queries
    int slot_off;       // and the partial slot's offset in each
};

// The work item with 128 NB query rows (32 NB per wave), see prefill_attn_kernel.
template <bool FP8, bool DECODE, bool JOINS, int NB>
__device__ __forceinline__ void prefill_item(
    const PrefillWork& it, char* __restrict__ smem, u32x4_t* __restrict__ sm_desc,
    const void* __restrict__ k_pool, const void* __restrict__ v_pool, int64_t pool_tokens,
    const bf16_t* __restrict__ q, const Run* __restrict__ runs, int g_shift, float scale_log2e_base,
    const HeadScales& k_scales, const HeadScales& v_scales, float* __restrict__ out,
    float* __restrict__ lse, const int32_t* __restrict__ ent_order,
    const int32_t* __restrict__ ent_base, float2* __restrict__ ws_ml) {
    constexpr int D = 128;
    constexpr int WROWS = 32 * NB;         // query rows per wave
    constexpr bool HIDE = !JOINS || NB == 1;  // how the missing rows of short runs are hidden, see missing_of
    constexpr int KROW_B = kPrefillKRowB, KS_B = kPrefillKB, BUF_B = kPrefillBufB, RING = kPrefillRing;
    static_assert(4 * WROWS == (NB == 2 ? kPrefillRowsPerItem : kPrefillRowsSmall), "rows per workgroup");

    const int n_kv_heads = (int)gridDim.x;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sw = w >> 1;   // which run of a tile this wave fetches
    const int hw = w & 1;    // which 16-row half of that run
    const int lane = threadIdx.x & 63;
    const int a = lane & 15;  // when loading: 16-byte piece of a row
    const int b = lane >> 4;  // when loading: row group
    const int n = lane & 31;  // in the matrix layouts: query row / run row / d
    const int g = lane >> 5;
    const int h = blockIdx.x;
    const float scale_log2e = FP8 ? scale_log2e_base * k_scales.of(h) : scale_log2e_base;
    const int run_begin = it.run_begin, run_end = it.run_end, n_grp = it.n_grp, tok0 = it.tok0;
    const int ent_begin = it.ent_begin, slot_off = it.slot_off;
    const int64_t q_row0 = it.q_row0;
    const int n_anc = it.n_anc;
    const int G = 1 << g_shift;
    const int n_q_heads = n_kv_heads << g_shift;
    const int n_runs = run_end - run_begin;
    const int n_tiles = (n_runs + 1) >> 1;
    const Run* my_runs = runs + run_begin;
    const float raise_margin = 8.0f / scale_log2e;  // raw-score distance of 2^8 in weight

    // the wave's 16 rows of K (rows b + 4 i) and of V (rows 4 b + i) of two tiles in flight:
    // a register set is busy from the issue of its loads until its tile is staged, two
    // tiles later; two sets alternate
    using raw_t = std::conditional_t<FP8, u32x2_t, u32x4_t>;
    struct RawTile {
        raw_t k[4], v[4];
    };
    RawTile raw0, raw1;
    constexpr uint32_t stride_b = FP8 ? D : D * 2;
    const int64_t plane = (int64_t)h * pool_tokens;
    const uint32_t piece = a * (FP8 ? 8 : 16);
    const uint32_t k_lane_off = (uint32_t)(16 * hw + b) * stride_b + piece;
    const uint32_t v_lane_off = (uint32_t)(16 * hw + 4 * b) * stride_b + piece;
    auto load_piece = [](__amdgpu_buffer_rsrc_t rs, uint32_t off) -> raw_t {
        if constexpr (FP8)
            return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0));
        else
            return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    };
    // a run's rows through a descriptor that covers exactly the run: rows past the end of
    // a short run read as zero (and are hidden); an empty run (past the end of the
    // list) is staged as zeros.  Always eight loads (an empty run's descriptor covers nothing:
    // every lane reads zero without a memory access), so that the number of loads in
    // flight is known at every wait.
    struct RunRsrc {
        __amdgpu_buffer_rsrc_t k, v;
    };
    auto rsrc_of = [&](const Run& sd, int size) {
        // (uniform, and said to be so: a run that was carried round the loop may sit in vector
        // registers, and loads through a descriptor made there go lane by lane)
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)sd.tok);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)sd.tok >> 32));
        const int64_t base = (plane + (int64_t)(((uint64_t)hi << 32) | lo)) * (int64_t)stride_b;
        char* kb = const_cast<char*>(reinterpret_cast<const char*>(k_pool)) + base;
        char* vb = const_cast<char*>(reinterpret_cast<const char*>(v_pool)) + base;
        const int bytes = __builtin_amdgcn_readfirstlane(size) * (int)stride_b;
        return RunRsrc{__builtin_amdgcn_make_buffer_rsrc(kb, 0, bytes, 0x00020000),
                       __builtin_amdgcn_make_buffer_rsrc(vb, 0, bytes, 0x00020000)};
    };
    // The lane's offsets of its eight rows.  They stay the same but for a run of two pieces, where each
    // row is on one side of the join: changed for its loads and put back for the next run, out of the way.
    // (Chosen at every load, a compare and a select each, they made every run 5 % longer.  In the
    // prologue even the way round that code shows, 27.4 us against 27.1 for 16 steps of 64 tokens: the
    // planner keeps joined runs out of it.  Without JOINS the compiler forms them as it likes and no join word is
    // carried: with both held there too, 16 steps of 64 tokens took 28.27 us instead of 28.05.)
    auto plain_row = [&](int i) {
        return i < 4 ? k_lane_off + (uint32_t)(4 * i) * stride_b : v_lane_off + (uint32_t)(i - 4) * stride_b;
    };
    uint32_t row_off[8];
    auto plain_rows = [&]() {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            row_off[i] = plain_row(i);
            asm volatile("" : "+v"(row_off[i]));
        }
    };
    if constexpr (JOINS) plain_rows();
    int joins = 0;  // whether row_off is of a joined run
    auto joined_rows = [&](Run& sd) {  // returns the rows that its loads may reach
        joins = __builtin_amdgcn_readfirstlane(sd.join);
        if (joins == 0) {
            plain_rows();
            return (int)sd.n;
        }
        const int32_t join = __builtin_amdgcn_readfirstlane(sd.join);
        const StepSpan span = span_of(sd.tok, __builtin_amdgcn_readfirstlane(sd.n), join);
        const int first = join_of(join).first;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = 16 * hw + (i < 4 ? b + 4 * i : 4 * b + i - 4);
            row_off[i] = (uint32_t)(row + (row < first ? span.low_shift : span.high_shift)) * stride_b + piece;
            asm volatile("" : "+v"(row_off[i]));
        }
        sd.tok = span.base;
        return span.size;
    };
    auto issue_load = [&](const RunRsrc& rs, RawTile& raw, int i) {  // i = 0..7
        const uint32_t off = JOINS ? row_off[i] : plain_row(i);
        if (i < 4) raw.k[i] = load_piece(rs.k, off);
        else raw.v[i - 4] = load_piece(rs.v, off);
    };
    auto issue_loads = [&](const Run& sd, RawTile& raw) {  // a run of consecutive rows
        const RunRsrc rs = rsrc_of(sd, sd.n);
#pragma unroll
        for (int i = 0; i < 8; ++i) issue_load(rs, raw, i);
    };
    // K: row-major rows of 272 bytes.  V: lane (a, b) holds run rows 16 hw + 4 b + i
    // (i = 0..3) at d = 8 a + x (x = 0..7); the four rows at one d are half (b >> 1) of slot
    // (x, b & 1, a).
    char* const k_dst = smem + (32 * sw + 16 * hw + b) * KROW_B + a * 16;  // + 4 i rows
    char* const v_dst = smem + KS_B + (sw * 2 + hw) * kVFragHalf + (16 * (b & 1) + a) * 16 + (b >> 1) * 8;
    auto stage_k = [&](char* dst, const RawTile& raw, int i) {  // i = 0..3
        *reinterpret_cast<u32x4_t*>(dst + 4 * i * KROW_B) = widen_raw(raw.k[i]);
    };
    u32x2_t v_even = {0u, 0u}, v_odd = {0u, 0u};  // E4M3: two elements, of rows 0 and 1 so far
    auto stage_v = [&](char* dst, const RawTile& raw, int x) {  // element x = 0..7 of the piece, in order
        if constexpr (FP8) {
            // one conversion yields two elements of a row: two rows of elements x and x + 1, then the
            // other two and both stores
            const int r = 2 * (x & 1);
            const bool high = x & 2;
            const uint32_t lo = high ? e4m3x2_to_f16x2<true>(raw.v[r][x >> 2])
                                     : e4m3x2_to_f16x2<false>(raw.v[r][x >> 2]);
            const uint32_t hi = high ? e4m3x2_to_f16x2<true>(raw.v[r + 1][x >> 2])
                                     : e4m3x2_to_f16x2<false>(raw.v[r + 1][x >> 2]);
            v_even[x & 1] = low_halves(lo, hi);
            v_odd[x & 1] = high_halves(lo, hi);
            if (x & 1) {
                *reinterpret_cast<u32x2_t*>(dst + (x - 1) * kVFragX) = v_even;
                *reinterpret_cast<u32x2_t*>(dst + x * kVFragX) = v_odd;
            }
        } else {
            auto halves = [](float lo, float hi) {
                return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
            };
            auto at = [&](int i) { return (x & 1) ? bf16_hi(raw.v[i][x >> 1]) : bf16_lo(raw.v[i][x >> 1]); };
            *reinterpret_cast<u32x2_t*>(dst + x * kVFragX) =
                u32x2_t{halves(at(0), at(1)), halves(at(2), at(3))};
        }
    };
    // descriptor of run idx from the ring (same address in every lane); runs past the end of the
    // list are empty there
    auto desc_at = [&](int idx) { return sm_desc + (idx & (RING - 1)); };
    auto run_of = [&](const u32x4_t& d) {
        uint32_t lo = __builtin_amdgcn_readfirstlane(d[0]);
        uint32_t hi = __builtin_amdgcn_readfirstlane(d[1]);
        uint32_t rows = __builtin_amdgcn_readfirstlane(d[2]);
        uint32_t join = JOINS ? __builtin_amdgcn_readfirstlane(d[3]) : 0u;
        asm volatile("" : "+s"(lo), "+s"(hi), "+s"(rows));  // carried round the loop in scalar registers
        if constexpr (JOINS) asm volatile("" : "+s"(join));
        return Run{(int64_t)(((uint64_t)hi << 32) | lo), (int32_t)rows, (int32_t)join};
    };
    auto run_at = [&](int idx) { return idx < n_runs ? my_runs[idx] : Run{0, 0, 0}; };

    // prologue: the first two tiles, the first 256 descriptors, the query rows
    issue_loads(run_at(sw), raw0);
    u32x4_t desc_raw = {0u, 0u, 0u, 0u};
    if ((int)threadIdx.x < min(n_runs, RING))
        desc_raw = load16(reinterpret_cast<const char*>(my_runs + threadIdx.x));
    issue_loads(run_at(2 + sw), raw1);

    // row r = 64 w + 32 j + n of the item (block j of the wave) is token r >> g_shift of the
    // block, query head r & (G - 1) of the kv head's group; rows past the block repeat its last
    // token (decode: row r is leaf query r >> g_shift of the item, in ent_order)
    auto group_of = [&](int r) { return min(r >> g_shift, n_grp - 1); };
    // a wave whose rows all lie past the block's last token (the last block of a node
    // is rarely full) only fetches and stages
    const bool active = ((WROWS * w) >> g_shift) < n_grp;
    const int i_first = tok0 + group_of(WROWS * w);  // the wave's first query token
    PrefillState<NB> st;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int r = WROWS * w + 32 * j + n;
        int64_t q_row = q_row0 + group_of(r);
        if constexpr (DECODE) q_row = ent_order[ent_begin + group_of(r)];
        const bf16_t* qp = q + (q_row * n_q_heads + h * G + (r & (G - 1))) * D;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) st.qf[j][kk] = as_bf16x8(load16(qp + 16 * kk + 8 * g));
    }

    sm_desc[threadIdx.x] = desc_raw;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        st.m[j] = -INFINITY;
        st.nmc[j] = st.lsum[j] = 0.f;
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int i = 0; i < 16; ++i) st.oacc[j][x][i] = 0.f;
    }
    // tile 0, and the half of tile 1 that precedes the first stage (see do_tile)
#pragma unroll
    for (int i = 0; i < 4; ++i) stage_k(k_dst, raw0, i);
#pragma unroll
    for (int x = 0; x < 8; ++x) stage_v(v_dst, raw0, x);
    issue_loads(run_at(4 + sw), raw0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        stage_k(k_dst + BUF_B, raw1, i);
        stage_v(v_dst + BUF_B, raw1, i);
    }
    __syncthreads();  // descriptors and the first tile are in LDS; of the second, K is

    // the first run of which the wave's first query token does not see every row
    const int first_hidden = n_anc + ((i_first + 1) >> 5);
    // Which rows of a run do not count: t >= n, and in step prefill kpos + t > the query token's
    // index (kpos: the run's position inside the querying node).
    struct Extent {
        int n, idx;  // of one run, uniform
    };
    auto extent_of = [&](uint32_t rows, int idx) ETS_INLINE {
        Extent e{(int)__builtin_amdgcn_readfirstlane(rows), idx};
        asm volatile("" : "+s"(e.n), "+s"(e.idx));  // carried round the loop in scalar registers
        return e;
    };
    auto hides = [&](const Extent& e) ETS_INLINE -> bool {
        // (once more said to be uniform, see rsrc_of)
        const int n_rows = __builtin_amdgcn_readfirstlane(e.n);
        const bool missing = !HIDE && n_rows < kStepRows;
        if constexpr (DECODE) return missing;  // the query is newer than every row
        return missing || __builtin_amdgcn_readfirstlane(e.idx) >= first_hidden;
    };
    // Rows past the end of a short run: they read as zero and score zero, and an outer product of
    // one contraction slot adds -3.4e38 to them, for every run alike.  `missing`: A operand,
    // 1 in the slot for those rows; `low`: B operand, the number in every column.  (A compare per
    // score behind a branch took 2 to 9 % more on steps of 25 to 150 tokens, 262 steps of 24..80
    // tokens over 4 kv heads 587 us -> 533; where all runs are full the instruction costs 0 to 1 %.)
    // With the rests of nodes joined few runs are short, and with two blocks to a wave the compares take over,
    // the same that hide what is newer than the query: 256 ragged steps of 8 heads 7.4 -> 7.2 ms by both.
    const int row_or_none = g == 0 ? n : -1;
    u32x2_t low = {g == 0 ? 0xFF7Fu : 0u, 0u};
    if constexpr (HIDE) asm volatile("" : "+a"(low));
    auto missing_of = [&](const Extent& e) ETS_INLINE {
        u32x2_t r = {row_or_none >= __builtin_amdgcn_readfirstlane(e.n) ? 0x3F80u : 0u, 0u};
        if constexpr (HIDE) asm volatile("" : "+v"(r));  // (here, not next to the matrix instruction)
        return r;
    };
    // (three matrix instructions, 24 issue slots, stand between a block's scores and its mask)
    auto mask = [&](f32x16_t& s, int j, const Extent& e) ETS_INLINE {
        const int kpos = kStepRows * (e.idx - n_anc);
        int lim = DECODE ? kStepRows : tok0 + group_of(WROWS * w + 32 * j + n) - kpos + 1;
        if constexpr (!HIDE) lim = min(lim, e.n);
        prefill_mask(s, g, lim);
    };
    auto rows_at = [&](int idx) ETS_INLINE {
        return reinterpret_cast<const uint32_t*>(desc_at(idx))[2];
    };

    const char* const k_src = smem + n * KROW_B + g * 16;  // the lane's row of a run's K fragments
    const char* const v_src = smem + KS_B + (n & 7) * kVFragX + (16 * g + (n >> 3)) * 16;
    u32x4_t pf_a[2][2], pf_b[2][2];    // weights of the even and of the odd run of a tile
    Extent e_next;                     // of the run whose scores come next
    Run load_next;                     // the run to be fetched next
    // scores and weights of the first run
    auto first_run = [&]() ETS_INLINE {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            st.kf[kk] = load16(k_src + 32 * kk);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if (kk == 0) mfma_scores_first(st.s[j], st.kf[0], st.qf[j][0]);
                else mfma_scores(st.s[j], st.kf[kk], st.qf[j][kk]);
            }
        }
        e_next = extent_of(rows_at(0), 0);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if constexpr (HIDE) mfma_hide(st.s[j], missing_of(e_next), low);
            mfma_result_wait(st.s[j]);
            if (hides(e_next)) mask(st.s[j], j, e_next);
            prefill_raise(st, j, prefill_max(st.s[j]), scale_log2e);
            // (with one block the weights belong to the first stage; all exponentials ahead of the
            // sums, so that they do not wait for one another)
            const int n_weights = NB == 1 ? 0 : j == 0 ? 16 : 16 - kLateWeights;
            float p[16];
#pragma unroll
            for (int i = 0; i < n_weights; ++i) {
                weight_begin(st, st.s[j], j, i, scale_log2e);
                p[i] = st.p_last;
            }
#pragma unroll
            for (int i = 0; i < n_weights; ++i) {
                st.p_last = p[i];
                weight_end(st, pf_a, j, i);
            }
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) st.kf[x] = load16(k_src + 32 * KROW_B + 32 * x);
        e_next = extent_of(rows_at(1), 1);
    };

    // Tile t, in buffer `cur` (t % 3).  Tile t + 1 goes to `nxt` from the register set `oth`, K and
    // half of V beside the previous tile's second stage, the rest beside this tile's first,
    // in front of the barrier; the set then takes the rows of tile t + 3.  Tile t + 2 follows
    // from `own` into the third buffer, whose last readers (tile t - 1) are behind that
    // barrier.
    int cur = 0, nxt = BUF_B, aft = 2 * BUF_B;
    load_next = run_of(*desc_at(6 + sw));
    auto do_tile = [&](int tile, RawTile& own, RawTile& oth, auto computes) ETS_INLINE {
        // ring refill: when run 128 k starts (k >= 1), runs [128 (k + 1), 128 (k + 2)) take
        // the slots of the 128 runs that were finished before it; they are used from 60
        // tiles later on
        if (ETS_RARE(tile > 0 && (tile & 63) == 0 && w < 2)) {
            const int idx = 2 * tile + 128 + (int)threadIdx.x;
            u32x4_t d = {0u, 0u, 0u, 0u};
            if (idx < n_runs) d = load16(reinterpret_cast<const char*>(my_runs + idx));
            sm_desc[idx & (RING - 1)] = d;
        }
        if constexpr (decltype(computes)::value) {
            char* const v_nxt = v_dst + nxt;
            char* const v_aft = v_dst + aft;
            char* const k_aft = k_dst + aft;
            const char* const vs = v_src + cur;
            const char* const ks = k_src + nxt;
            RunRsrc rs;
            uint32_t d_e;
            u32x4_t d_run;
            int size = load_next.n;
            auto finish = [&](int k) ETS_INLINE {
                if (k >= 8 && k < 11) stage_v(v_nxt, oth, k - 4);
                if (k == 13) stage_v(v_nxt, oth, 7);
            };
            auto begin = [&](int k) ETS_INLINE {
                if (k >= 8 && k < 11) stage_v(v_aft, own, k - 8);
                if (k >= 12) stage_k(k_aft, own, k - 12);
                if (k == 13) stage_v(v_aft, own, 3);
            };
            auto loads = [&](int i) ETS_INLINE {
                if (i == 4) d_e = rows_at(2 * tile + 2);
                // (behind the last branch of the stage: carried over one, a resource descriptor would
                // move to vector registers)
                if (i == 5) {
                    rs = rsrc_of(load_next, size);
                }
                if (i >= 6 && i < 14) issue_load(rs, oth, i - 6);
                if (i == 14) e_next = extent_of(d_e, 2 * tile + 2);
            };
            auto descs = [&](int i) ETS_INLINE {
                if (i == 4) d_e = rows_at(2 * tile + 3);
                // (without JOINS its first twelve bytes, in two reads)
                if (i == 5) {
                    if constexpr (JOINS) {
                        d_run = *desc_at(2 * tile + 8 + sw);
                    } else {
                        const u32x2_t tok = *reinterpret_cast<const u32x2_t*>(desc_at(2 * tile + 8 + sw));
                        d_run = u32x4_t{tok[0], tok[1], 0u, 0u};
                    }
                }
                if (!JOINS && i == 6) d_run[2] = rows_at(2 * tile + 8 + sw);
                if (i == 13) e_next = extent_of(d_e, 2 * tile + 3);
                if (i == 14) load_next = run_of(d_run);
            };
            const Extent e1 = e_next;
            const bool joined = JOINS && (__builtin_amdgcn_readfirstlane(load_next.join) | joins) != 0;
            auto mask1 = [&](f32x16_t& s, int j) ETS_INLINE { mask(s, j, e1); };
            auto rare1 = [&](f32x16_t& s, int j) ETS_INLINE {
                if (hides(e1)) mask(s, j, e1);
                if constexpr (JOINS)
                    if (joined) size = joined_rows(load_next);
            };
            if constexpr (NB == 2)
                prefill_unit<HIDE>(st, vs, ks, pf_a, pf_b, scale_log2e, raise_margin, missing_of(e1), low, hides(e1),
                                   finish, mask1, []() { __syncthreads(); }, hides(e1) || joined, rare1, loads);
            else
                prefill_unit1<0>(st, vs, ks, pf_a, scale_log2e, raise_margin, missing_of(e1), low, finish,
                                 []() { __syncthreads(); }, hides(e1) || joined, rare1, loads);
            const Extent e2 = e_next;
            auto mask2 = [&](f32x16_t& s, int j) ETS_INLINE { mask(s, j, e2); };
            if constexpr (NB == 2)
                prefill_unit<HIDE>(st, vs + 2 * kVFragHalf, ks + 32 * KROW_B, pf_b, pf_a, scale_log2e,
                                   raise_margin, missing_of(e2), low, hides(e2), begin, mask2, []() {}, hides(e2),
                                   mask2, descs);
            else
                prefill_unit1<1>(st, vs + 2 * kVFragHalf, ks + 32 * KROW_B, pf_b, scale_log2e,
                                 raise_margin, missing_of(e2), low, begin, []() {}, hides(e2), mask2, descs);
        } else {
#pragma unroll
            for (int x = 4; x < 8; ++x) stage_v(v_dst + nxt, oth, x);
            __syncthreads();
            const int size = JOINS ? joined_rows(load_next) : (int)load_next.n;
            const RunRsrc rs = rsrc_of(load_next, size);
#pragma unroll
            for (int i = 0; i < 8; ++i) issue_load(rs, oth, i);
            load_next = run_of(*desc_at(2 * tile + 8 + sw));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                stage_k(k_dst + aft, own, i);
                stage_v(v_dst + aft, own, i);
            }
        }
        const int free_buf = cur;
        cur = nxt;
        nxt = aft;
        aft = free_buf;
    };
    // (nothing but the exit branches off inside the loops: the waits for a register set then leave
    // the other set's loads in flight)
    auto walk = [&](auto computes) ETS_INLINE {
        for (int tile = 0;;) {
            do_tile(tile, raw0, raw1, computes);
            if (++tile >= n_tiles) break;
            do_tile(tile, raw1, raw0, computes);
            if (++tile >= n_tiles) break;
        }
        // (here, where the loop is left, so that no copy of the rows comes before it)
        if constexpr (decltype(computes)::value)
#pragma unroll
            for (int j = 0; j < NB; ++j) mfma_result_wait(st.oacc[j]);
        __syncthreads();  // every wave is done with the tiles: the epilogue reuses the buffers
    };
    if (!active) {
        walk(std::false_type{});  // only fetches and stages, through the same barriers
        // (The compiler joins the two ways behind this one.  A load that still counts as outstanding here makes
        // the other way wait for all of its own before the first product, 0.4 us: of its registers, too.)
        __builtin_amdgcn_s_waitcnt(0);
        return;
    }
    first_run();
    walk(std::true_type{});

    // rows out through the wave's own LDS region (a block's 32 rows padded to 132 floats), so that
    // whole 512-byte rows are stored: normalised in step prefill, unnormalised next to (m, l) in
    // decode
    constexpr int OROW = 132;
    static_assert(4 * 32 * OROW * 4 <= 3 * BUF_B, "four regions");
    float* ob = reinterpret_cast<float*>(smem) + w * (32 * OROW);
    const int col = (lane & 31) * 4;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int r_lane = WROWS * w + 32 * j + n;
        // row of the lane's query in `out` (and in lse / ws_ml)
        int64_t out_row = q_row0 + group_of(r_lane);
        if constexpr (DECODE) out_row = ent_base[ent_begin + group_of(r_lane)] + slot_off;
        out_row = out_row * n_q_heads + h * G + (r_lane & (G - 1));
        float l = st.lsum[j];
        l += __shfl_xor(l, 32, 64);
        float inv = 1.0f;
        if constexpr (!DECODE) {
            inv = 1.0f / l;
            if constexpr (FP8) inv *= v_scales.of(h);
        }
        if (g == 0 && (r_lane >> g_shift) < n_grp) {
            if constexpr (DECODE)
                ws_ml[out_row] = make_float2(st.m[j] * scale_log2e, l);
            else
                lse[out_row] = (st.m[j] * scale_log2e + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
        }
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                *reinterpret_cast<float4*>(ob + n * OROW + 32 * x + 8 * c + 4 * g) =
                    make_float4(st.oacc[j][x][4 * c] * inv, st.oacc[j][x][4 * c + 1] * inv,
                                st.oacc[j][x][4 * c + 2] * inv, st.oacc[j][x][4 * c + 3] * inv);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int rr = 2 * k + (lane >> 5);  // row of the block that the lane stores
            const int r = WROWS * w + 32 * j + rr;
            int64_t row_out = (q_row0 + (r >> g_shift)) * n_q_heads + h * G + (r & (G - 1));
            if constexpr (DECODE) row_out = __shfl(out_row, rr, 64);  // lane rr (g = 0) holds it
            const float4 v = *reinterpret_cast<const float4*>(ob + rr * OROW + col);
            if ((r >> g_shift) < n_grp) *reinterpret_cast<float4*>(out + row_out * D + col) = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// JOINS: whether runs of two pieces may be among the plan's (the others' loop is the shorter one: 16 steps
// of 64 tokens 27.4 us, with joins allowed for 27.7, 8 steps of 16 tokens 7.65 and 7.8).
// FP8: the pools hold E4M3 codes (128-byte rows, 8 bytes per lane and load); the codes are
// widened while the tile is staged (K to bf16, V straight to the fp16 fragments), the kv
// head's K scale enters the score scale and its V scale multiplies the normalised rows.
// DECODE: `items_raw` are CascadeItem (leaf queries ent_order[ent_begin .. + n_ent), at most
// 256 / G of them), `out` is the partial workspace ws_o, `lse` is unused, and ent_order,
// ent_base, ws_ml are the decode plan's tables; otherwise `items_raw` are PrefillItem and
// the last three arguments are unused.
// An item of at most 128 query rows (the last block of a node, a short step, a segment of few leaf
// queries) is walked with 32 rows per wave: 1 350 cycles per run instead of the 2 008 that a wave
// of 64 rows takes however many of them are in use.  Calls against 64 rows per wave throughout, us:
// 256 steps of 16 tokens, 4 heads per kv head, 248 -> 173; of 20 to 150 tokens 547 -> 516; of 32 to
// 256 tokens, 1 head, 319 -> 298; 8 heads 1 484 -> 1 466; decode of 256 leaf queries with
// segments of more than 16 query rows as wide items 183 -> 163.
template <bool FP8, bool DECODE, bool JOINS>
__global__ __launch_bounds__(kPrefillThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void prefill_attn_kernel(
    const void* __restrict__ k_pool, const void* __restrict__ v_pool, int64_t pool_tokens,
    const bf16_t* __restrict__ q, const Run* __restrict__ runs,
    const void* __restrict__ items_raw, int item_base, int g_shift, float scale_log2e_base,
    HeadScales k_scales, HeadScales v_scales, float* __restrict__ out, float* __restrict__ lse,
    const int32_t* __restrict__ ent_order, const int32_t* __restrict__ ent_base,
    float2* __restrict__ ws_ml) {
    static_assert(!DECODE || kPrefillRowsPerItem == kWideRowsPerItem, "rows per workgroup");
    __shared__ u32x4_t smem[3 * kPrefillBufB / 16];
    __shared__ u32x4_t sm_desc[kPrefillRing];
    PrefillWork work{};
    if constexpr (DECODE) {
        const CascadeItem it = static_cast<const CascadeItem*>(items_raw)[item_base + (int)blockIdx.y];
        work.run_begin = it.run_begin;
        work.run_end = it.run_end;
        work.n_grp = it.n_ent;
        work.ent_begin = it.ent_begin;
        work.slot_off = it.slot_off;
    } else {
        const PrefillItem it = static_cast<const PrefillItem*>(items_raw)[item_base + (int)blockIdx.y];
        work.run_begin = it.run_begin;
        work.run_end = it.run_end;
        work.n_grp = it.n_tok;
        work.tok0 = it.tok0;
        work.n_anc = it.n_anc;
        work.q_row0 = it.q_row0;
    }
    char* const lds = reinterpret_cast<char*>(smem);
    if (work.n_grp << g_shift <= kPrefillRowsSmall)
        prefill_item<FP8, DECODE, JOINS, 1>(work, lds, sm_desc, k_pool, v_pool, pool_tokens, q, runs, g_shift,
                                     scale_log2e_base, k_scales, v_scales, out, lse, ent_order, ent_base,
                                     ws_ml);
    else
        prefill_item<FP8, DECODE, JOINS, 2>(work, lds, sm_desc, k_pool, v_pool, pool_tokens, q, runs, g_shift,
                                     scale_log2e_base, k_scales, v_scales, out, lse, ent_order, ent_base,
                                     ws_ml);
}

}  // namespace ets
