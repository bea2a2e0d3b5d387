// Tree attention where shared rows meet many query rows: the kernel of plans whose work items hold
// groups of leaf queries, up to 128 query rows each (the planner says which plans, see build()).
//
// Arithmetic, layouts and results per query row are those of tree_attn_kernel.hpp: scores in fp32 by
// bf16 matrix instructions, weights against a lazily raised reference, fp16 weights on V converted
// to fp16 in items of more than 16 query rows, bf16 head plus remainder on bf16 V in the others, one
// unnormalised partial (o, m, l) per query row.  What differs is the split:
//   R > 64   a wave takes two blocks of 16 query rows through both steps of a 64-token tile: every
//            fragment read from LDS feeds two matrix instructions, and a tile is fetched and staged
//            once for 128 rows;
//   R > 16   the two waves of a pair compute the step they fetched, each for its own row blocks, and
//            the pairs add up their results behind the walk;
//   R <= 16  every wave walks 32-token steps that it fetched itself, alone (small items) or every
//            fourth one (results folded through LDS).
// Two register sets take turns, so that a tile is requested two tiles ahead and staged into the second of
// two LDS buffers while the first is read: one barrier per tile.  Step lists stand in LDS or in the lanes
// of a register: a scalar load in the loop returns in no order, and every wait for LDS would wait for it.
// The conversion of the next tile stands beside the last matrix instructions of the current one, and is
// pinned there: hoisted ahead of them, as the compiler did, it waits for loads a tile too early.
// 252 registers and 72.5 KB of LDS with head_dim 128: two workgroups per compute unit (three with 64).
//
// Bound of a tile: the issue of one wave's chain.  (Of a call, items of more than 64 rows take half of the
// slot time or less, e.g. 48 of 117 us on 256 leaves with 64 query heads.)  A tile takes a wave of 32 query rows 4 200 cycles alone and 4 500
// with a second workgroup beside it (issue of the loads 450, a step of 32 tokens 1 750, barrier 170), of
// which the matrix pipe is busy 1 024: 1.0 us of a compute unit per 128 x 64, against 1.27 for two
// tiles of 64 rows with three workgroups of the other kernel.  Calls that also stream meet the bandwidth
// behind L2 first: 512 leaves read 2.0 GB past L2 in 370 us.  Whole calls, the other kernel -> this one,
// us: 16 searches of 256 leaves with 64 query heads 2 061 -> 1 957, one of them 145 -> 132; 512 leaves
// with 32 query heads 368 -> 369, over E4M3 pools 272 -> 264; drawn trees beyond the planner's lines 0.93 to
// 1.20, 1.045 in the mean, with head_dim 64 0.91 to 1.51, 1.14.  Not faster: segments walked by resident
// workgroups in lists made by the planner (no slot idle, but every tile as much longer).
#pragma once

#include "tree_attn_kernel.hpp"

namespace ets {

static_assert(kGroupRowsPerItem == 128, "4 waves x 32 rows");

// What a wave of a row-parallel item carries from step to step: NB blocks of 16 query rows.
template <int D, int NB>
struct GroupState {
    bf16x8_t qf[NB][D / 32];   // query rows as B operands
    f32x4_t oacc[NB][D / 16];  // lane (a, b): row a of the block, output block x
    float m[NB], lsum[NB];     // reference score and sum of weights of the lane's row
};

// Largest of a lane's eight scores.  (The instructions themselves: around fmaxf the compiler first
// canonicalises every value.  It does not see what reads the results of the matrix instructions
// here, so the wait for them is part of the statement.)
__device__ __forceinline__ float max_of(const f32x4_t& lo, const f32x4_t& hi) {
    float mx;
    asm volatile(
        "s_nop 15\n\tv_max3_f32 %0, %1, %2, %3\n\tv_max3_f32 %0, %0, %4, %5\n\t"
        "v_max3_f32 %0, %0, %6, %7\n\tv_max_f32 %0, %0, %8"
        : "=&v"(mx)
        : "v"(lo[0]), "v"(lo[1]), "v"(lo[2]), "v"(lo[3]), "v"(hi[0]), "v"(hi[1]), "v"(hi[2]), "v"(hi[3]));
    return mx;
}

// One step of a row-parallel item: 32 staged tokens (V already fp16) against the wave's NB blocks of
// 16 query rows; every fragment read from LDS feeds NB matrix instructions.  The scores of tokens that
// a short step does not have (they read as zero) start from -inf instead of 0.
// Matrix and vector instructions of a wave overlap where they alternate in program order: the
// weights of the second block are computed beside the application of the first, and the caller's
// fill(x), x = 0 .. D / 16 - 1, stands beside the application of the last.
template <int D, int NB, class Fill>
__device__ __forceinline__ void group_step(const u32x4_t* __restrict__ ks_lane,
                                          const u32x4_t* __restrict__ vs_lane,
                                          int b, int n_valid, GroupState<D, NB>& st,
                                          float scale_log2e, float raise_margin, Fill fill) {
    constexpr int KROW = k_row_units<D>();
    constexpr int NKK = D / 32, NX = D / 16;
    // scores S^T = K Q^T, the fragments requested two products ahead
    f32x4_t s[NB][2];
    if (n_valid < 32) {
        int rem = n_valid - 4 * b;
        asm volatile("" : "+v"(rem));  // (here: hoisted, the compares' operands take registers)
#pragma unroll
        for (int i = 0; i < 8; ++i) s[0][i >> 2][i & 3] = 16 * (i >> 2) + (i & 3) >= rem ? -INFINITY : 0.f;
#pragma unroll
        for (int j = 1; j < NB; ++j) {
            s[j][0] = s[0][0];
            s[j][1] = s[0][1];
        }
    } else {
#pragma unroll
        for (int j = 0; j < NB; ++j) s[j][0] = s[j][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    u32x4_t kf[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        kf[0][t] = ks_lane[16 * t * KROW];
        kf[1][t] = ks_lane[16 * t * KROW + 4];
    }
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
                s[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kf[kk & 1][t]), st.qf[j][kk],
                                                                  s[j][t], 0, 0, 0);
            if (kk + 2 < NKK) kf[kk & 1][t] = ks_lane[16 * t * KROW + 4 * (kk + 2)];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // the V^T fragments are requested before the softmax arithmetic
    u32x4_t vf[NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) vf[x] = vs_lane[x * 64];
    __builtin_amdgcn_sched_barrier(0);
    // lane holds row a of the block, tokens 4 b + i (first half) and 16 + 4 b + i (second half)
    float mx[NB];
    bool above = false;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        mx[j] = max_of(s[j][0], s[j][1]);
        above = above || mx[j] > st.m[j] + raise_margin;
    }
    if (__any(above)) {
        // raise the reference of every row to its running maximum
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            float x = fmaxf(mx[j], __shfl_xor(mx[j], 16, 64));
            x = fmaxf(x, __shfl_xor(x, 32, 64));
            const float m_new = fmaxf(st.m[j], x);
            const float alpha = fast_exp2((st.m[j] - m_new) * scale_log2e);
            st.lsum[j] *= alpha;
#pragma unroll
            for (int y = 0; y < NX; ++y) st.oacc[j][y] *= alpha;
            st.m[j] = m_new;
        }
    }
    f16x8_t pf[NB];
    float mc[NB], psum[NB];
    auto weight = [&](int j, int i) {
        const float p = fast_exp2(fmaf(s[j][i >> 2][i & 3], scale_log2e, -mc[j]));
        psum[j] = i ? psum[j] + p : p;
        pf[j][i] = (_Float16)p;
    };
#pragma unroll
    for (int j = 0; j < NB; ++j)  // (a row that has seen nothing yet: every score is -inf, every weight 0)
        mc[j] = st.m[j] == -INFINITY ? 0.f : st.m[j] * scale_log2e;
#pragma unroll
    for (int i = 0; i < 8; ++i) weight(0, i);
    st.lsum[0] += psum[0];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            st.oacc[j][x] =
                __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(vf[x]), pf[j], st.oacc[j][x], 0, 0, 0);
            if (j + 1 < NB) {
#pragma unroll
                for (int i = 8 * x / NX; i < 8 * (x + 1) / NX; ++i) weight(NB - 1, i);
            } else {
                fill(x);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (j + 1 < NB) st.lsum[NB - 1] += psum[NB - 1];
    }
}

// A step that one wave fetched itself, against a single block of query rows.  K rows and V^T
// fragments (bf16) sit in the wave's own LDS region.  The weight enters the P V product as a bf16 head
// plus its bf16 remainder, one matrix instruction each.
template <int D>
__device__ __forceinline__ void private_step(const u32x4_t* __restrict__ ks_lane,
                                                  const u32x4_t* __restrict__ vs_lane, int b,
                                                  int n_valid, const bf16x8_t (&qf)[D / 32],
                                                  f32x4_t (&oacc)[D / 16], float& m, float& lsum,
                                                  float scale_log2e, float raise_margin) {
    constexpr int KROW = k_row_units<D>();
    constexpr int NKK = D / 32, NX = D / 16;
    f32x4_t s[2];
    {
        int rem = n_valid - 4 * b;
        asm volatile("" : "+v"(rem));  // (here: hoisted, the compares' operands take registers)
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i >> 2][i & 3] = 16 * (i >> 2) + (i & 3) >= rem ? -INFINITY : 0.f;
    }
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
        for (int t = 0; t < 2; ++t)
            s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ks_lane[16 * t * KROW + 4 * kk]), qf[kk],
                                                           s[t], 0, 0, 0);
    // lane holds row a, tokens 4 b + i and 16 + 4 b + i
    float mx = max_of(s[0], s[1]);
    if (__any(mx > m + raise_margin)) {
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m, mx);
        const float alpha = fast_exp2((m - m_new) * scale_log2e);
        lsum *= alpha;
#pragma unroll
        for (int x = 0; x < NX; ++x) oacc[x] *= alpha;
        m = m_new;
    }
    const float mc = m * scale_log2e;
    float psum = 0.f;
    bf16x8_t head, rest;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float p = fast_exp2(fmaf(s[i >> 2][i & 3], scale_log2e, -mc));
        psum = i ? psum + p : p;
        head[i] = (__bf16)p;
        rest[i] = (__bf16)(p - (float)head[i]);
    }
#pragma unroll
    for (int x = 0; x < NX; ++x) {
        const bf16x8_t v = as_bf16x8(vs_lane[x * 64]);
        oacc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, head, oacc[x], 0, 0, 0);
        oacc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, rest, oacc[x], 0, 0, 0);
    }
    lsum += psum;
}

template <bool FP8, int D = 128>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 3, D == 128 ? 2 : 3))) void group_attn_kernel(
    const void* __restrict__ k_pool, const void* __restrict__ v_pool, int64_t pool_tokens,
    const bf16_t* __restrict__ q, const Run* __restrict__ steps,
    const UnitSlot* __restrict__ units, int unit_base,
    const int32_t* __restrict__ ent_order, const int32_t* __restrict__ ent_base, int g_shift,
    float scale_log2e_base, HeadScales k_scales,
    float* __restrict__ ws_o, float2* __restrict__ ws_ml) {
    static_assert(D == 128 || D == 64, "head_dim");
    const int n_kv_heads = (int)gridDim.x;
    constexpr int KROW = k_row_units<D>();
    constexpr int NKK = D / 32;            // matrix instructions of a score product
    constexpr int NX = D / 16;             // V^T fragments (blocks of 16 output elements)
    constexpr int PPR = D / 8;             // 16-byte pieces (8 elements) per row
    constexpr int RPL = 64 / PPR;          // K rows one load instruction of a wave covers
    constexpr int NKL = 16 / RPL;          // K loads per 16 tokens
    constexpr int KS_UNITS = 64 * KROW;    // K tile: 64 padded rows
    constexpr int VS_UNITS = 2 * NX * 64;  // V^T fragments: [step][x][lane]
    constexpr int BUF_UNITS = KS_UNITS + VS_UNITS;
    constexpr int WAVE_UNITS = 2 * BUF_UNITS / 4;  // a wave's own region
    static_assert(32 * KROW + NX * 64 <= WAVE_UNITS, "a private step");
    // two tiles: K rows, then V^T fragments; reused for folds and on the way out
    __shared__ u32x4_t smem[2 * BUF_UNITS];
    __shared__ float sm_m[4][16];
    __shared__ float sm_l[4][16];
    __shared__ u32x4_t sm_desc[kTreeAttnMaxSteps];  // step list of a row-parallel item

    // wave index, made known-uniform so that per-wave descriptors come through scalar loads
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sw = w >> 1;  // which step of a tile this wave fetches
    const int hw = w & 1;   // which 16-token half of that step
    const int h = blockIdx.x;  // kv head; consecutive workgroups share an item
    // E4M3 pools: the K scale of this kv head is part of the score scale
    const float scale_log2e = FP8 ? scale_log2e_base * k_scales.of(h) : scale_log2e_base;
    const int G = 1 << g_shift;
    const int n_q_heads = n_kv_heads << g_shift;
    const float raise_margin = 8.0f / scale_log2e;  // raw-score distance of 2^8 in weight
    const int64_t plane = (int64_t)h * pool_tokens;  // first row of this kv head

    // A workgroup takes one item, or four small items, one per wave, which then works alone; the
    // planner's launch order says which.  One table read (uniform per wave: scalar loads) brings the item
    // and the first two steps the wave fetches.
    const int lane = threadIdx.x & 63;
    const int a = lane & 15;  // 16-byte piece of a row when loading; MFMA row/column index
    const int b = lane >> 4;  // token sub-index when loading; MFMA contraction group kg
    const UnitSlot* my_unit = units + 4 * (unit_base + (int)blockIdx.y) + w;
    const CascadeItem it = my_unit->item;
    const Run first_step = my_unit->first, second_step = my_unit->second;
    const bool wave_item = it.wave_item == 1;
    if (it.n_ent == 0) return;
    const int R = it.n_ent << g_shift;
    const int n_blocks = (R + 15) >> 4;
    const int n_steps = it.run_end - it.run_begin;
    const int n_tiles = (n_steps + 1) >> 1;
    const Run* my_steps = steps + it.run_begin;

    using raw_t = std::conditional_t<FP8, u32x2_t, u32x4_t>;
    constexpr uint32_t stride_b = FP8 ? D : D * 2;  // bytes between the tokens of a head plane
    constexpr uint32_t piece_b = FP8 ? 8 : 16;      // bytes of a lane's 8 elements
    // K: a load covers RPL consecutive rows, the lane's piece pa of row rb: token
    // RPL i + rb of the half (head_dim 128: pa = a, rb = b).
    // V: contraction slot 4 hw + j of group b = token 4 b + j of the half.  With head_dim 128
    // the lane's piece is a, of which it transposes all 8 elements; with head_dim 64 a row
    // has 8 pieces, lanes 2 p and 2 p + 1 both fetch piece p and transpose one half each
    // (output element 4 a + x of fragment x).
    const int pa = lane & (PPR - 1), rb = lane / PPR;
    const int va = D == 128 ? a : a >> 1;
    const uint32_t k_lane_off = (uint32_t)rb * stride_b + pa * piece_b;
    const uint32_t v_lane_off = (uint32_t)(4 * b) * stride_b + va * piece_b;
    // 16 HALVES tokens of a step from its token `from` on, requested into a register set.  Buffer loads:
    // the rows are addressed through a descriptor that covers exactly them (base = the first row at this
    // kv head, size = the rows of the step from there on), so a load is a scalar descriptor plus a 32-bit
    // lane offset, and rows past the end of a ragged step read as zero instead of needing clamped
    // addresses (they are masked later).  Always the same number of loads (an empty descriptor covers
    // nothing: every lane reads zero without a memory access), so that the waits behind them are
    // exact.  Returns the rows there are.
    auto issue = [&](const Run& sd, int from, auto& raw, auto halves, auto aux_tag) {
        constexpr int HALVES = decltype(halves)::value;
        // cache policy of the loads: 2 = non-temporal, in items of at most 16 query rows, whose rows are mostly
        // one leaf query's own; rows of larger items are mostly read by further ones
        // (uniform, and said to be so: carried round a loop a step may sit in vector registers)
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)sd.tok);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)sd.tok >> 32));
        const int n = max(0, (int)__builtin_amdgcn_readfirstlane(sd.n) - from);
        const int64_t base = (plane + from + (int64_t)(((uint64_t)hi << 32) | lo)) * (int64_t)stride_b;
        char* kb = const_cast<char*>(reinterpret_cast<const char*>(k_pool)) + base;
        char* vb = const_cast<char*>(reinterpret_cast<const char*>(v_pool)) + base;
        const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(kb, 0, n * (int)stride_b, 0x00020000);
        const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(vb, 0, n * (int)stride_b, 0x00020000);
#pragma unroll
        for (int t = 0; t < HALVES; ++t) {
            // (the row stepping rides in the instructions' immediate offsets, which are range-checked with
            // the lane offset; hoisted out of the loop it would take a register for each)
            uint32_t k_off = k_lane_off, v_off = v_lane_off;
            asm volatile("" : "+v"(k_off), "+v"(v_off));
            if (t > 0) {
                k_off += 16 * t * stride_b;
                v_off += 16 * t * stride_b;
            }
#pragma unroll
            for (int i = 0; i < NKL; ++i)
                raw.k[NKL * t + i] = load_row_piece<FP8>(kr, k_off + (uint32_t)(RPL * i) * stride_b, 0, aux_tag);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                raw.v[4 * t + i] = load_row_piece<FP8>(vr, v_off + (uint32_t)i * stride_b, 0, aux_tag);
        }
        return n;
    };
    using cached_t = std::integral_constant<int, 0>;
    using streamed_t = std::integral_constant<int, 2>;
    // The leaf query and the partial slot of a row block's row a.  A block's entries may run up to 15
    // past the item's own, which is what the tables' zero padding is for: those name leaf query 0 or a
    // neighbouring item's leaf queries, whose rows are read and never written.  Requested ahead of
    // the first tile: vector loads return in order.
    const int head = h * G + (a & (G - 1));
    auto entry_of = [&](const int32_t* table, int block) {
        return table[it.ent_begin + ((16 * block + a) >> g_shift)];
    };
    // Q rows of a block as B operands: lane (column a = query row, group b) holds
    // q[row][32 kk + 8 b .. + 8)
    auto load_q = [&](int ent, bf16x8_t (&qf)[NKK]) {
        const bf16_t* qp = q + ((int64_t)ent * n_q_heads + head) * D;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) qf[kk] = as_bf16x8(load16(qp + 32 * kk + 8 * b));
    };

    // Partial results leave through the wave's LDS region.  Lane (a, b) holds row a, d = 32 b + 8 i + x
    // (head_dim 64: d = 16 b + 4 i + x): written from there, every store instruction would
    // touch 64 different cache lines with 16 bytes each.  Rows are padded by 4 floats, and each
    // store instruction writes whole rows (two of 512 bytes, or four of 256).
    constexpr int OROW = D + 4;
    static_assert(32 * OROW * 4 <= WAVE_UNITS * 16, "two blocks");
    float* const ob = reinterpret_cast<float*>(smem + w * WAVE_UNITS);
    auto put_rows = [&](int at, const f32x4_t (&oacc)[NX]) {  // a block, as the wave's at-th
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float* p = ob + (16 * at + a) * OROW + (D / 4) * b + (D / 16) * i;
            *reinterpret_cast<float4*>(p) =
                make_float4(oacc[0][i], oacc[1][i], oacc[2][i], oacc[3][i]);
            if constexpr (D == 128)
                *reinterpret_cast<float4*>(p + 4) =
                    make_float4(oacc[4][i], oacc[5][i], oacc[6][i], oacc[7][i]);
        }
    };
    // The wave's at-th block, row block blk of the item, from LDS to the workspace.  `ent_slot`: first
    // partial slot of the lane's row's leaf query.
    auto store_rows = [&](int at, int blk, int ent_slot, float m, float l) {
        const int r_lane = 16 * blk + a;
        const int32_t out_row = (ent_slot + it.slot_off) * n_q_heads + head;
        if (b == 0 && r_lane < R) {
            ws_ml[out_row] = make_float2(m * scale_log2e, l);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        constexpr int LPR = D / 4;       // lanes that store a row, 16 bytes each
        constexpr int RPS = 64 / LPR;    // rows per store instruction
        const int col = (lane & (LPR - 1)) * 4;
#pragma unroll
        for (int k = 0; k < 16 / RPS; ++k) {
            const int r = RPS * k + lane / LPR;              // row of the block this lane stores
            const int32_t row_out = __shfl(out_row, r, 64);  // lane r holds row r (a = r, b = 0)
            const float4 v = *reinterpret_cast<const float4*>(ob + (16 * at + r) * OROW + col);
            if (16 * blk + r < R) {
                *reinterpret_cast<float4*>(ws_o + (int64_t)row_out * D + col) = v;
            }
        }
    };

    if (R <= 16) {
        // ---- At most 16 query rows: nothing is shared between waves, so every wave walks steps that it
        // fetched itself through its own LDS region, with no workgroup barrier in the loop.  A small
        // item is walked by this wave alone (all its steps); others by the four waves together (steps
        // w, 4 + w, ..).
        struct RawStep {
            raw_t k[2 * NKL], v[8];
        };
        RawStep raw0, raw1;
        u32x4_t* const ksw = smem + w * WAVE_UNITS;
        u32x4_t* const vsw = ksw + 32 * KROW;
        // K rows as they are, V as bf16 A fragments: lane (a, b) holds tokens 4 b .. + 3 of both halves at the
        // elements of its piece (head_dim 64: of its half of the piece)
        auto stage = [&](const RawStep& raw) {
#pragma unroll
            for (int i = 0; i < 2 * NKL; ++i) ksw[(RPL * i + rb) * KROW + pa] = widen_raw(raw.k[i]);
            u32x4_t vw[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) vw[i] = widen_raw(raw.v[i]);
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                const uint32_t sel = (x & 1) ? 0x07060302u : 0x05040100u;
                u32x4_t t;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t lo = D == 128 ? vw[2 * i][(x >> 1) & 3] : (a & 1) ? vw[2 * i][2 + ((x >> 1) & 1)] : vw[2 * i][(x >> 1) & 1];
                    const uint32_t hi = D == 128 ? vw[2 * i + 1][(x >> 1) & 3] : (a & 1) ? vw[2 * i + 1][2 + ((x >> 1) & 1)] : vw[2 * i + 1][(x >> 1) & 1];
                    t[i] = __builtin_amdgcn_perm(hi, lo, sel);
                }
                vsw[x * 64 + lane] = t;
            }
        };
        const int first = wave_item ? 0 : w, stride = wave_item ? 1 : 4;
        const int n_own = wave_item ? n_steps : (n_steps + 3) >> 2;
        constexpr std::integral_constant<int, 2> whole{};
        const int ent = entry_of(ent_order, 0), ent_slot = entry_of(ent_base, 0);
        int n_cur = issue(first_step, 0, raw0, whole, streamed_t{});
        bf16x8_t qf[NKK];
        load_q(ent, qf);
        int n_next = issue(second_step, 0, raw1, whole, streamed_t{});
        // The wave's steps ahead, one to a lane, 64 at a time: a scalar load in the loop would come back in no
        // order, so that every wait for LDS would wait for it too.
        auto steps_from = [&](int k) {
            const int idx = first + (k + lane) * stride;
            u32x4_t d = load16(my_steps + min(idx, n_steps - 1));
            if (idx >= n_steps) d[2] = 0;
            return d;
        };
        u32x4_t held = steps_from(0);
        auto own_step = [&](int k) {  // for k in order
            if ((k & 63) == 0) held = steps_from(k);
            const uint32_t lo = __builtin_amdgcn_readlane(held[0], k & 63), hi = __builtin_amdgcn_readlane(held[1], k & 63);
            return Run{(int64_t)(((uint64_t)hi << 32) | lo), (int32_t)__builtin_amdgcn_readlane(held[2], k & 63), 0};
        };
        f32x4_t oacc[NX];
        float m = -INFINITY, lsum = 0.f;
#pragma unroll
        for (int x = 0; x < NX; ++x) oacc[x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        stage(raw0);
        Run sd_far = own_step(2);
        // step k of the wave is staged; step k + 1 is in flight in `nxt`; step k + 2 goes to `far`, and the
        // one after it is looked up
        auto do_step = [&](int k, RawStep& far, RawStep& nxt) {
            const int n_far = issue(sd_far, 0, far, whole, streamed_t{});
            sd_far = own_step(k + 3);
            if (n_cur > 0)
                private_step<D>(ksw + a * KROW + b, vsw + lane, b, n_cur, qf, oacc, m, lsum,
                                     scale_log2e, raise_margin);
            // the wave's LDS accesses complete in order; keep the compiler from moving them
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            stage(nxt);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            n_cur = n_next;
            n_next = n_far;
        };
        for (int k = 0;;) {
            do_step(k, raw0, raw1);
            if (++k >= n_own) break;
            do_step(k, raw1, raw0);
            if (++k >= n_own) break;
        }
        float l = lsum;
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (!wave_item) {
            // The four waves hold the same rows over disjoint tokens (a wave that saw no
            // token has m = -inf, l = 0); waves 1..3 hand their results to wave 0 through
            // LDS, so the item still yields one partial per query row.
            if (b == 0) {
                sm_m[w][a] = m;
                sm_l[w][a] = l;
            }
            __syncthreads();  // also: every wave is done with its tile region
            const float ms = fmaxf(fmaxf(sm_m[0][a], sm_m[1][a]), fmaxf(sm_m[2][a], sm_m[3][a]));
            const float f_own = fast_exp2((m - ms) * scale_log2e);
            f32x4_t* fold = reinterpret_cast<f32x4_t*>(smem) + lane;
            if (w != 0) {
#pragma unroll
                for (int x = 0; x < NX; ++x) fold[((w - 1) * NX + x) * 64] = oacc[x] * f_own;
            }
            __syncthreads();
            if (w != 0) return;
            l *= f_own;
#pragma unroll
            for (int k = 1; k < 4; ++k)
                l += sm_l[k][a] * fast_exp2((sm_m[k][a] - ms) * scale_log2e);
            m = ms;
#pragma unroll
            for (int x = 0; x < NX; ++x)
                oacc[x] = oacc[x] * f_own + fold[x * 64] + fold[(NX + x) * 64] + fold[(2 * NX + x) * 64];
        }
        put_rows(0, oacc);
        store_rows(0, 0, ent_slot, m, l);
        return;
    }

    // ---- More query rows: the tile is staged in LDS once and used by all waves.
    // Wave w fetches half hw of step 2 tile + sw of every tile.
    struct RawUnit {
        raw_t k[NKL], v[4];
    };
    RawUnit raw0, raw1;
    constexpr std::integral_constant<int, 1> half{};
    // Part k of the wave's half step into a tile buffer: its NKL pieces of K rows, then one
    // element of every V piece at a time: this half's four contraction slots (8 of the 16 bytes)
    // of a V^T fragment, converted to fp16 for the P V product once for all row blocks: element
    // x of the lane's 16-byte piece (head_dim 64: of the lane's half of it), tokens 4 b .. 4 b + 3.
    // (The statements that pin the pieces keep the conversion, and with it the wait for the loads, where it
    // is written; `place` tells the copies apart, which would otherwise be joined ahead of the branch
    // between them.)
    u32x2_t v_even = {0u, 0u}, v_odd = {0u, 0u};  // E4M3: two elements, of tokens 4 b and 4 b + 1 so far
    auto stage_part = [&](u32x4_t* buf, const RawUnit& raw, int k, auto place) {  // (in order)
        if (k < NKL) {
            raw_t piece = raw.k[k];
            asm volatile("; %1" : "+v"(piece) : "n"(decltype(place)::value));
            buf[(32 * sw + 16 * hw + RPL * k + rb) * KROW + pa] = widen_raw(piece);
        } else {
            const int x = k - NKL;
            u32x2_t* const vs2 = reinterpret_cast<u32x2_t*>(buf + KS_UNITS) + (sw * NX * 64 + lane) * 2 + hw;
            if constexpr (FP8) {
                // one conversion yields two elements of a row: two rows of elements x and x + 1, then the
                // other two and both stores (head_dim 64: codes 4 (a & 1) .. + 3 of the piece)
                const int r = 2 * (x & 1);
                uint32_t two[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    uint32_t codes = D == 128 ? raw.v[r + i][x >> 2] : (a & 1) ? raw.v[r + i][1] : raw.v[r + i][0];
                    asm volatile("; %1" : "+v"(codes) : "n"(decltype(place)::value));
                    two[i] = (x & 2) ? e4m3x2_to_f16x2<true>(codes) : e4m3x2_to_f16x2<false>(codes);
                }
                v_even[x & 1] = low_halves(two[0], two[1]);
                v_odd[x & 1] = high_halves(two[0], two[1]);
                if (x & 1) {
                    vs2[(x - 1) * 128] = v_even;
                    vs2[x * 128] = v_odd;
                }
            } else {
                float f[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t dw = D == 128 ? raw.v[i][(x >> 1) & 3]
                                           : (a & 1) ? raw.v[i][2 + ((x >> 1) & 1)] : raw.v[i][(x >> 1) & 1];
                    asm volatile("; %1" : "+v"(dw) : "n"(decltype(place)::value));
                    f[i] = (x & 1) ? bf16_hi(dw) : bf16_lo(dw);
                }
                vs2[x * 128] = u32x2_t{__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[0], f[1])),
                                       __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[2], f[3]))};
            }
        }
    };
    auto stage = [&](u32x4_t* buf, const RawUnit& raw, auto place) {
#pragma unroll
        for (int k = 0; k < NKL + NX; ++k) stage_part(buf, raw, k, place);
    };
    // More than 64 rows: a wave takes row blocks 2 w and 2 w + 1 through both steps of every tile.
    // Up to 64: the waves of a pair (2 sw, 2 sw + 1) compute the step they have fetched, each for its
    // own row blocks (two of them when the item has more than two, else one); behind the walk the
    // two waves that hold a block over different steps add up their results.
    auto walk = [&](auto blocks, auto both_steps) __attribute__((always_inline)) {
        constexpr int NB = decltype(blocks)::value;
        constexpr bool quad = decltype(both_steps)::value;
        const int blk0 = NB * (quad ? w : hw);
        const bool active = blk0 < n_blocks;  // others only fetch and stage
        // (a block that the item does not have repeats the last one and is not stored)
        int ent[NB], slot[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            ent[j] = entry_of(ent_order, min(blk0 + j, n_blocks - 1));
            slot[j] = entry_of(ent_base, min(blk0 + j, n_blocks - 1));
        }
        // the item's step list goes to LDS once, zeros behind the last
        static_assert(kTreeAttnMaxSteps == 256, "one descriptor per thread");
        u32x4_t desc_raw = load16(my_steps + min((int)threadIdx.x, n_steps - 1));
        if ((int)threadIdx.x >= n_steps) desc_raw[2] = 0;
        issue(first_step, 16 * hw, raw0, half, cached_t{});
        GroupState<D, NB> st;
#pragma unroll
        for (int j = 0; j < NB; ++j) load_q(ent[j], st.qf[j]);
        issue(second_step, 16 * hw, raw1, half, cached_t{});
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            st.m[j] = -INFINITY;
            st.lsum[j] = 0.f;
#pragma unroll
            for (int x = 0; x < NX; ++x) st.oacc[j][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
        sm_desc[threadIdx.x] = desc_raw;
        stage(smem, raw0, std::integral_constant<int, 0>{});
        __syncthreads();
        // Rows of the steps of a tile that the wave computes, packed (the first in the low half), and the step
        // it fetches.  Read from LDS at the start of a tile and made scalar at its end.
        auto rows_at = [&](int tile) -> uint32_t {
            const int idx = min(2 * tile, kTreeAttnMaxSteps - 2);
            if constexpr (quad) return sm_desc[idx][2] | sm_desc[idx + 1][2] << 16;
            else return sm_desc[idx + sw][2];
        };
        auto desc_at = [&](int tile) { return sm_desc[min(2 * tile + sw, kTreeAttnMaxSteps - 1)]; };
        auto step_of = [&](const u32x4_t& d, int tile) {
            const uint32_t lo = __builtin_amdgcn_readfirstlane(d[0]), hi = __builtin_amdgcn_readfirstlane(d[1]);
            const int n = __builtin_amdgcn_readfirstlane(d[2]);
            return Run{(int64_t)(((uint64_t)hi << 32) | lo), 2 * tile + sw < kTreeAttnMaxSteps ? n : 0, 0};
        };
        uint32_t rows = __builtin_amdgcn_readfirstlane(rows_at(0));
        uint32_t rows_next = __builtin_amdgcn_readfirstlane(rows_at(1));
        Run sd_far = step_of(desc_at(2), 2);
        // Tile t stands in `buf`; tile t + 1 is in flight in `nxt` and goes to the other buffer,
        // whose readers are behind the last barrier; tile t + 2 is requested into `far`.
        auto do_tile = [&](int tile, u32x4_t* buf, u32x4_t* other, RawUnit& far, RawUnit& nxt) {
            issue(sd_far, 16 * hw, far, half, cached_t{});
            u32x4_t d_far = desc_at(tile + 3);
            uint32_t rows_after = rows_at(tile + 2);
            auto compute = [&](int c, int n_valid, auto fill) {
                group_step<D, NB>(buf + (32 * c + a) * KROW + b, buf + KS_UNITS + c * NX * 64 + lane,
                                 b, n_valid, st, scale_log2e, raise_margin, fill);
            };
            constexpr int PARTS = NKL + NX;
            constexpr std::integral_constant<int, 2> beside{};
            if (!active) {
                stage(other, nxt, std::integral_constant<int, 1>{});
            } else if constexpr (quad) {
                compute(0, rows & 0xFFFF, [&](int x) {
                    if (x < PARTS / 2) stage_part(other, nxt, x, beside);
                });
                compute(1, rows >> 16, [&](int x) {
                    if (x < PARTS / 2) stage_part(other, nxt, PARTS / 2 + x, beside);
                });
            } else {
                compute(sw, rows, [&](int x) {
#pragma unroll
                    for (int k = PARTS * x / NX; k < PARTS * (x + 1) / NX; ++k) stage_part(other, nxt, k, beside);
                });
            }
            __syncthreads();
            asm volatile("" : "+v"(d_far), "+v"(rows_after));  // (here, not where they were read)
            sd_far = step_of(d_far, tile + 3);
            rows = rows_next;
            rows_next = __builtin_amdgcn_readfirstlane(rows_after);
        };
        for (int tile = 0;;) {
            do_tile(tile, smem, smem + BUF_UNITS, raw0, raw1);
            if (++tile >= n_tiles) break;
            do_tile(tile, smem + BUF_UNITS, smem, raw1, raw0);
            if (++tile >= n_tiles) break;
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            st.lsum[j] += __shfl_xor(st.lsum[j], 16, 64);
            st.lsum[j] += __shfl_xor(st.lsum[j], 32, 64);
        }
        if constexpr (quad) {
            if (!active) return;
#pragma unroll
            for (int j = 0; j < NB; ++j) put_rows(j, st.oacc[j]);
#pragma unroll 1
            for (int j = 0; j < NB && blk0 + j < n_blocks; ++j)
                store_rows(j, blk0 + j, j ? slot[NB - 1] : slot[0], j ? st.m[NB - 1] : st.m[0],
                           j ? st.lsum[NB - 1] : st.lsum[0]);
        } else {
            // Both waves of a row group hold its blocks over their own steps.  Each of them stores one block,
            // the first wave the first, and gets the other's share of it through LDS.
            constexpr int FOLD = NX * 64 + 32;  // units of a block: rows, then (m, l)
            static_assert(4 * FOLD <= 2 * BUF_UNITS, "four blocks");
            auto hand_over = [&](int j) {
                u32x4_t* fold = smem + w * FOLD;
#pragma unroll
                for (int x = 0; x < NX; ++x) fold[x * 64 + lane] = __builtin_bit_cast(u32x4_t, st.oacc[j][x]);
                reinterpret_cast<float2*>(fold + NX * 64)[lane] = make_float2(st.m[j], st.lsum[j]);
            };
            if (NB == 2 && sw == 1) {
                hand_over(0);
                // (its own block from here on)
                st.m[0] = st.m[NB - 1];
                st.lsum[0] = st.lsum[NB - 1];
                slot[0] = slot[NB - 1];
#pragma unroll
                for (int x = 0; x < NX; ++x) st.oacc[0][x] = st.oacc[NB - 1][x];
            } else {
                hand_over(NB - 1);
            }
            __syncthreads();
            const u32x4_t* fold = smem + (w ^ 2) * FOLD;
            const float2 ml = reinterpret_cast<const float2*>(fold + NX * 64)[lane];
            // (a wave without a step has m = -inf, l = 0, o = 0)
            const float ms = fmaxf(st.m[0], ml.x);
            const float f_own = fast_exp2((st.m[0] - ms) * scale_log2e);
            const float f_got = fast_exp2((ml.x - ms) * scale_log2e);
            const float l = st.lsum[0] * f_own + ml.y * f_got;
#pragma unroll
            for (int x = 0; x < NX; ++x)
                st.oacc[0][x] = st.oacc[0][x] * f_own + __builtin_bit_cast(f32x4_t, fold[x * 64 + lane]) * f_got;
            __syncthreads();
            const int blk = blk0 + (NB == 2 ? sw : 0);
            if ((NB == 1 && sw == 1) || blk >= n_blocks) return;
            put_rows(0, st.oacc[0]);
            store_rows(0, blk, slot[0], ms, l);
        }
    };
    if (R > 64) walk(std::integral_constant<int, 2>{}, std::true_type{});
    else if (R > 32) walk(std::integral_constant<int, 2>{}, std::false_type{});
    else walk(std::integral_constant<int, 1>{}, std::false_type{});
}

}  // namespace ets
