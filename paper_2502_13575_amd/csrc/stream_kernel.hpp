// Per-leaf streaming attention: one wavefront = one (work item, kv head).
//
// A work item names one leaf query and a list of pool runs (its private
// suffix of the tree, or in the flat baseline its whole root->leaf chain).
// The wave streams the runs' K and V rows from HBM with 16-byte loads that
// cover whole head rows contiguously (D * sizeof(T) bytes per token and head),
// keeps the G query heads of the kv head in registers, and carries a running
// (max, sum, weighted V) per query head: the online form of the softmax whose
// result is defined by out = sum_t exp(s_t - lse) V_t.  It writes one
// unnormalised partial (o, m, l) per query head; the merge kernel combines the
// partials along the leaf's chain.  m is kept in log2 units (scores are
// pre-multiplied by log2 e) so that exp2 can be used throughout.
#pragma once

#include "device_utils.hpp"
#include "merge_kernel.hpp"
#include "plan.h"

namespace ets {

// The running state of a wave: per query head the reference, the sum of weights and, in lane
// (b, a), the a-th 16 bytes' elements of the weighted V over the tokens of lane group b.
template <typename T, int D, int G>
struct StreamState {
    static constexpr int EPL = Vec16<T>::N;  // elements per lane per load
    static constexpr int LPT = D / EPL;      // lanes per token row
    float m[G], l[G], o[G][EPL];
};

// Walks the runs of an item; behind it every lane holds the sums over all tokens.
template <typename T, int D, int G, int U>
__device__ __forceinline__ void stream_walk(StreamState<T, D, G>& st, const StreamItem& item, int lane, int h,
                                            int n_q_heads, const T* __restrict__ k_pool,
                                            const T* __restrict__ v_pool, int64_t pool_tokens,
                                            const T* __restrict__ q, const Run* __restrict__ runs,
                                            float scale_log2e) {
    constexpr int EPL = StreamState<T, D, G>::EPL, LPT = StreamState<T, D, G>::LPT;
    constexpr int TPS = 64 / LPT;     // tokens per wave-wide load
    static_assert(LPT >= 2 && LPT <= 64 && TPS >= 1, "unsupported row size");
    float (&m)[G] = st.m;
    float (&l)[G] = st.l;
    float (&o)[G][EPL] = st.o;
    const int a = lane % LPT;  // which 16-byte piece of the row
    const int b = lane / LPT;  // which token of the step
    constexpr int64_t row_stride = D;  // pools are [kv head][pool row][D]

    float qf[G][EPL];
    {
        const T* qp = q + ((int64_t)item.entry * n_q_heads + (int64_t)h * G) * D + a * EPL;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            Vec16<T> v;
            v.load(qp + g * D);
            v.unpack(qf[g]);
#pragma unroll
            for (int i = 0; i < EPL; ++i) qf[g][i] *= scale_log2e;
        }
    }

#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = -INFINITY;
        l[g] = 0.f;
#pragma unroll
        for (int i = 0; i < EPL; ++i) o[g][i] = 0.f;
    }

    for (int r = item.run_begin; r < item.run_end; ++r) {
        const Run run = runs[r];
        const int64_t base = ((int64_t)h * pool_tokens + run.tok) * (int64_t)D + a * EPL;
        const T* kb = k_pool + base;
        const T* vb = v_pool + base;
        for (int t0 = 0; t0 < run.n; t0 += TPS * U) {
            Vec16<T> kraw[U], vraw[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int tok = min(t0 + u * TPS + b, run.n - 1);  // clamp: stays inside the run
                kraw[u].load(kb + tok * row_stride);
                vraw[u].load(vb + tok * row_stride);
            }
            float s[U][G];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float kf[EPL];
                kraw[u].unpack(kf);
                const bool valid = t0 + u * TPS + b < run.n;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    float acc = 0.f;
#pragma unroll
                    for (int i = 0; i < EPL; ++i) acc = fmaf(qf[g][i], kf[i], acc);
                    acc = group_sum<LPT>(acc);
                    s[u][g] = valid ? acc : -INFINITY;
                }
            }
            float alpha[G], mu[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float mn = m[g];
#pragma unroll
                for (int u = 0; u < U; ++u) mn = fmaxf(mn, s[u][g]);
                mu[g] = (mn == -INFINITY) ? 0.f : mn;
                alpha[g] = fast_exp2(m[g] - mu[g]);
                m[g] = mn;
                l[g] *= alpha[g];
#pragma unroll
                for (int i = 0; i < EPL; ++i) o[g][i] *= alpha[g];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float vf[EPL];
                vraw[u].unpack(vf);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float p = fast_exp2(s[u][g] - mu[g]);
                    l[g] += p;
#pragma unroll
                    for (int i = 0; i < EPL; ++i) o[g][i] = fmaf(p, vf[i], o[g][i]);
                }
            }
        }
    }

    // fold the TPS token lanes of the wave together
#pragma unroll
    for (int g = 0; g < G; ++g) {
        float mt = m[g];
#pragma unroll
        for (int off = LPT; off < 64; off <<= 1) mt = fmaxf(mt, __shfl_xor(mt, off, 64));
        const float mu = (mt == -INFINITY) ? 0.f : mt;
        const float f = fast_exp2(m[g] - mu);
        float lt = l[g] * f;
#pragma unroll
        for (int off = LPT; off < 64; off <<= 1) lt += __shfl_xor(lt, off, 64);
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            float x = o[g][i] * f;
#pragma unroll
            for (int off = LPT; off < 64; off <<= 1) x += __shfl_xor(x, off, 64);
            o[g][i] = x;
        }
        m[g] = mt;
        l[g] = lt;
    }
}

template <typename T, int D, int G, int U>
__global__ __launch_bounds__(64) void stream_attn_kernel(
    const T* __restrict__ k_pool, const T* __restrict__ v_pool, int64_t pool_tokens,
    const T* __restrict__ q, const Run* __restrict__ runs, const StreamItem* __restrict__ items,
    int n_kv_heads,
    float scale_log2e, float* __restrict__ ws_o, float2* __restrict__ ws_ml) {
    const int h = blockIdx.x % n_kv_heads;
    const StreamItem item = items[blockIdx.x / n_kv_heads];
    const int lane = threadIdx.x;
    const int n_q_heads = n_kv_heads * G;
    StreamState<T, D, G> st;
    stream_walk<T, D, G, U>(st, item, lane, h, n_q_heads, k_pool, v_pool, pool_tokens, q, runs, scale_log2e);
    constexpr int EPL = StreamState<T, D, G>::EPL;
    const int a = lane % StreamState<T, D, G>::LPT;
    if (lane != a) return;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int64_t row = (int64_t)item.slot * n_q_heads + h * G + g;
        float4* dst = reinterpret_cast<float4*>(ws_o + row * D + a * EPL);
#pragma unroll
        for (int i = 0; i < EPL / 4; ++i)
            dst[i] = make_float4(st.o[g][4 * i], st.o[g][4 * i + 1], st.o[g][4 * i + 2], st.o[g][4 * i + 3]);
        if (a == 0) ws_ml[row] = make_float2(st.m[g], st.l[g]);
    }
}

// LDS of direct_attn_kernel with this many waves.
constexpr int direct_lds_bytes(int waves, int D, int G) { return waves * G * (D * 4 + 8); }

// A small call over fp32 pools in one launch: a workgroup takes a leaf query's whole path for one kv
// head, a wave each of its items (at most sixteen, in slot order from part_base[leaf] on; waves past the
// last one idle), and merges their results through LDS as merge_kernel does through the workspace.
// Bound: the chain of dependent round trips (items -> runs -> rows -> fold -> output) and the launch
// itself; the merge launch it saves is a second such chain behind the first one's end.  8 leaves of 80 rows
// 9.2 -> 5.8 us, 32 of 300 rows with 16 query heads of 64 9.2 -> 7.9; the rule stands in plan.cpp.
// LDS goes by the waves that there are: with room for sixteen (66 KB with eight query heads of 128) two workgroups
// fit a compute unit, 179 leaves of 19 rows 4 kv heads x 8 query heads of 128, 20.7 us; so 11.8.
template <typename T, int D, int G, int U>
__global__ __launch_bounds__(64 * kDirectWaves) void direct_attn_kernel(
    const T* __restrict__ k_pool, const T* __restrict__ v_pool, int64_t pool_tokens,
    const T* __restrict__ q, const Run* __restrict__ runs, const StreamItem* __restrict__ items,
    const int32_t* __restrict__ part_base, int n_kv_heads, float scale_log2e, HeadScales v_scales,
    void* __restrict__ out, int out_bf16, float* __restrict__ lse) {
    // [wave][G * D] weighted V, then [wave][G] (m, l): direct_lds_bytes for the waves that there are
    extern __shared__ float4 direct_lds[];
    static_assert(alignof(float4) == 16 && D % 4 == 0, "rows are written 16 bytes at a time");
    float* const sm_o = reinterpret_cast<float*>(direct_lds);
    float2* const sm_ml = reinterpret_cast<float2*>(sm_o + (blockDim.x >> 6) * (G * D));
    const int h = blockIdx.x % n_kv_heads;
    const int leaf = blockIdx.x / n_kv_heads;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int n_q_heads = n_kv_heads * G;
    const int first = part_base[leaf], n_items = part_base[leaf + 1] - first;
    if (w < n_items) {
        StreamState<T, D, G> st;
        stream_walk<T, D, G, U>(st, items[first + w], lane, h, n_q_heads, k_pool, v_pool, pool_tokens, q, runs,
                                scale_log2e);
        constexpr int EPL = StreamState<T, D, G>::EPL;
        const int a = lane % StreamState<T, D, G>::LPT;
        if (lane == a) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float4* dst = reinterpret_cast<float4*>(sm_o + w * (G * D) + g * D + a * EPL);
#pragma unroll
                for (int i = 0; i < EPL / 4; ++i)
                    dst[i] = make_float4(st.o[g][4 * i], st.o[g][4 * i + 1], st.o[g][4 * i + 2], st.o[g][4 * i + 3]);
                if (a == 0) sm_ml[w * G + g] = make_float2(st.m[g], st.l[g]);
            }
        }
    }
    __syncthreads();
    const int64_t row0 = (int64_t)leaf * n_q_heads + h * G;
    for (int e = threadIdx.x; e < G * D; e += blockDim.x) {
        const int g = e / D;
        float ms = -INFINITY, l = 0.f, acc = 0.f;
        for (int k = 0; k < n_items; ++k) ms = fmaxf(ms, sm_ml[k * G + g].x);
        for (int k = 0; k < n_items; ++k) {
            const float2 ml = sm_ml[k * G + g];
            const float f = fast_exp2(ml.x - ms);
            l += ml.y * f;
            acc = fmaf(sm_o[k * (G * D) + e], f, acc);
        }
        const float r = acc * (n_items == 0 ? 0.f : 1.f / l) * v_scales.of(h);
        if (out_bf16) static_cast<uint16_t*>(out)[row0 * D + e] = f32_to_bf16_rne(r);
        else static_cast<float*>(out)[row0 * D + e] = r;
        if (e % D == 0)
            lse[row0 + g] = n_items == 0 ? -INFINITY : (ms + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
    }
}

}  // namespace ets
