// Log-sum-exp merge of split-K attention partials (Eq. (2) evaluated over
// disjoint position ranges and recombined), shared by the decode combine
// kernel and the fused step's finishing kernel.
#pragma once
#include "common.h"

namespace wushkv {

constexpr int kMaxSplits = 1024;

// Sums and maxima over the lanes of a wave, in every lane, without LDS: DPP
// inside the rows of 16, then the row and half exchanges of v_permlane*_swap
// (a lane shuffle takes an LDS round trip per step).
template <int CTRL>
__device__ __forceinline__ float dpp(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
// x of this lane and of lane ^ 16, ^ 32 (which comes first varies).
struct LanePair {
    float a, b;
};
__device__ __forceinline__ LanePair pair16(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ LanePair pair32(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ float add16(float x) { const LanePair p = pair16(x); return p.a + p.b; }
__device__ __forceinline__ float add32(float x) { const LanePair p = pair32(x); return p.a + p.b; }
// over the 16 lanes of a row (quad butterflies, then rotations)
__device__ __forceinline__ float row_sum16(float x)
{
    x += dpp<0xB1>(x);
    x += dpp<0x4E>(x);
    x += dpp<0x124>(x);
    x += dpp<0x128>(x);
    return x;
}
// The max is four DPP-operand maxima in one assembly block; each is preceded
// by the two wait states a DPP read of a just-written register needs.  The
// inputs are finite or -inf.
__device__ __forceinline__ float row_max16(float x)
{
    float y;
    asm volatile(
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf"
        : "=&v"(y)
        : "v"(x));
    return y;
}
__device__ __forceinline__ float wave_sum(float x) { return add32(add16(row_sum16(x))); }
__device__ __forceinline__ float wave_max(float x)
{
    const LanePair p = pair16(row_max16(x));
    const LanePair q = pair32(fmaxf(p.a, p.b));
    return fmaxf(q.a, q.b);
}

// A row is merged by one wave where there are many rows (they fill the device
// by themselves: 2048 rows of 9 splits take 5.7 us, with four waves a row 7.5),
// by four otherwise (a row's splits are then a shorter chain: 32 rows of 89
// splits 4.6 us, 256 rows of 11 splits 4.5 us).  The fused step and the separate calls go by the same rule,
// so that their outputs are the same bits.
constexpr int kMergeWaves = 4;
__host__ __device__ constexpr bool merge_by_one(int64_t rows) { return rows >= 1024; }

template <int D>
struct MergeLds {
    float o[kMergeWaves][D];
    float m[kMergeWaves], l[kMergeWaves];
};

// One query head: the n_splits partials (o[D] relative to m, m, l) at pp,
// pp + stride, ..  (m in base 2) merge into
//   dst = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s,  M = max_s m_s,
// zero when no split saw a position.  NW waves share the splits (wave w takes
// w, w + NW, ..): lane i loads m and l of the wave's i-th split, the wave
// forms M and the weights in registers, and the rows of o, requested
// together with them, are added up with each weight read from its lane.  The
// merge is a latency chain: one round trip to memory instead of two, and one
// barrier (none for one wave) instead of nine (89 splits: 4.6 instead of 7.4
// us, near a launch's own cost).  With NW = 1 each wave merges
// a row of its own.
template <int D, int NW>
__device__ __forceinline__ void merge_splits(const float *pp, int64_t stride, int32_t n_splits,
                                             float *dst, int tid, MergeLds<D> &lds)
{
    constexpr int kPer = D / 64;     // channels per lane
    constexpr int kFirst = 8;        // rows of o requested at once, and, where
    constexpr int kMore = 16;        // there are more, with them
    const int lane = tid & 63, wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t mine = (n_splits - wave + NW - 1) / NW;  // this wave's splits
    const float *base = pp + wave * stride;
    const int64_t step = NW * stride;
    float M = -INFINITY, l = 0.0f, o[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) o[e] = 0.0f;
    for (int32_t k0 = 0; k0 < mine; k0 += 64) {
        const int32_t n = min(mine - k0, 64);
        float ms = -INFINITY, ls = 0.0f;
        if (lane < n) {
            const float *src = base + (k0 + lane) * step + D;
            ms = src[0];
            ls = src[1];
        }
        // (a row past the end is a repeat of the last)
        auto load_rows = [&](auto &x, int32_t i0) {
#pragma unroll
            for (int i = 0; i < (int)(sizeof(x) / sizeof(x[0])); ++i) {
                const float *src = base + (int64_t)(k0 + min(i0 + i, n - 1)) * step + kPer * lane;
#pragma unroll
                for (int e = 0; e < kPer; ++e) x[i][e] = src[e];
            }
        };
        float x[kFirst][kPer], y[kMore][kPer];
        load_rows(x, 0);
        if (n > kFirst) load_rows(y, kFirst);
        const float m_new = fmaxf(M, wave_max(ms));
        const float f = M == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(M - m_new);
        const float w = ms == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ms - m_new);
        l = fmaf(l, f, wave_sum(w * ls));
#pragma unroll
        for (int e = 0; e < kPer; ++e) o[e] *= f;
        M = m_new;
        auto add_rows = [&](const auto &x, int32_t i0) {
#pragma unroll
            for (int i = 0; i < (int)(sizeof(x) / sizeof(x[0])); ++i) {
                // (lane i0 + i holds weight 0 past the end)
                const float wi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), i0 + i));
#pragma unroll
                for (int e = 0; e < kPer; ++e) o[e] = fmaf(wi, x[i][e], o[e]);
            }
        };
        add_rows(x, 0);
        for (int32_t i0 = kFirst; i0 < n; i0 += kMore) {
            if (i0 > kFirst) load_rows(y, i0);
            add_rows(y, i0);
        }
    }
    if constexpr (NW == 1) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) dst[kPer * lane + e] = l > 0.0f ? o[e] / l : 0.0f;
    } else {
#pragma unroll
        for (int e = 0; e < kPer; ++e) lds.o[wave][kPer * lane + e] = o[e];
        if (lane == 0) {
            lds.m[wave] = M;
            lds.l[wave] = l;
        }
        __syncthreads();
        if (tid >= D) return;
        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < NW; ++v) mx = fmaxf(mx, lds.m[v]);
        float sum = 0.0f, den = 0.0f;
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            const float f = lds.m[v] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(lds.m[v] - mx);
            sum = fmaf(f, lds.o[v][tid], sum);
            den = fmaf(f, lds.l[v], den);
        }
        dst[tid] = den > 0.0f ? sum / den : 0.0f;
    }
}

}  // namespace wushkv
