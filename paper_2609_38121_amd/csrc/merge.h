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
// Inclusive prefix sum over the lanes.
template <int CTRL, int ROWS>
__device__ __forceinline__ int32_t dpp_from(int32_t x)  // 0 where there is no such lane
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ int32_t wave_scan(int32_t x)
{
    x += dpp_from<0x111, 0xF>(x);  // row_shr 1, 2, 4, 8
    x += dpp_from<0x112, 0xF>(x);
    x += dpp_from<0x114, 0xF>(x);
    x += dpp_from<0x118, 0xF>(x);
    x += dpp_from<0x142, 0xA>(x);  // lane 15 of a row to the next row
    x += dpp_from<0x143, 0xC>(x);  // lane 31 to the upper half
    return x;
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

// A row is merged by one wave where there are many rows, by four otherwise.
// Many rows fill the device by themselves, so that one wave each is less work:
// 2048 rows of 4, 10 and 18 splits take 4.1, 4.8 and 5.4 us a launch, with four
// waves a row 4.4, 5.2 and 5.8; 1024 rows of 34 splits 5.4 and 5.9.  With few
// rows the launch's own 4 us is nearly all of it, and a row's splits are a
// shorter chain in four waves, which long contexts feel.  Between 256 and 1536
// rows of at most 18 splits both take 4.0 us, so the line is drawn where the
// work begins to show; it costs 1.5 us at 1024 rows of 66 splits (7.5 us, with
// four waves 6.0; 128 sequences of 262144 tokens).  The fused step and the
// separate calls go by the same rule, so that their outputs are the same bits.
constexpr int kMergeWaves = 4;
__host__ __device__ constexpr bool merge_by_one(int64_t rows) { return rows >= 1024; }

template <int D>
struct MergeLds {
    float o[kMergeWaves][D];
    float m[kMergeWaves], l[kMergeWaves];
};

// Where a row's partials are: query head (h, g) of grid row b, among part's
// [grid row][n_kv][n_splits][G][D + 2].  The window partials are the row's own
// splits from n_page_splits on; so are the page partials, at the splits before,
// unless the attention launch dealt its page runs out by the lengths it found
// (runs, see plan_runs in decode.hip): runs[0] is then not zero and the row's
// page partials are those of the runs[2 + 2 b + 1] page workgroups from number
// runs[2 + 2 b] on, numbered through all the rows.
struct MergeRows {
    const float *part;
    int32_t n_kv, G, n_splits, n_page_splits;
    int32_t b, h, g;
    const int32_t *runs;
};

// One query head: its n partials (o[D] relative to m, m, l; m in base 2) merge
// into
//   dst = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s,  M = max_s m_s,
// zero when no split saw a position.  NW waves share the splits (wave w takes
// w, w + NW, ..): lane i loads m and l of the wave's i-th split, the wave
// forms M and the weights in registers, and the rows of o, requested
// together with them, are added up with each weight read from its lane.  The
// merge is a latency chain: one round trip to memory instead of two, and one
// barrier (none for one wave) instead of nine (89 splits: 4.6 instead of 7.4
// us, near a launch's own cost).  The row's own splits are requested before
// runs[0] is known, and again where the runs were dealt out.  With NW = 1 each
// wave merges a row of its own.
template <int D, int NW>
__device__ __forceinline__ void merge_splits(const MergeRows &r, float *dst, int tid, MergeLds<D> &lds)
{
    constexpr int kPer = D / 64;     // channels per lane
    constexpr int kFirst = 8;        // rows of o requested at once, and, where
    constexpr int kMore = 16;        // there are more, with them
    const int lane = tid & 63, wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t stride = (int64_t)r.G * (D + 2);
    const float *base = r.part + r.g * (D + 2);
    const int32_t own = (r.b * r.n_kv + r.h) * r.n_splits;
    int32_t total = r.n_splits;      // the row's partials
    int32_t first = 0, n_runs = -1;  // dealt out: its page runs
    int32_t slot = own;              // partial of the wave's (k0 + lane)-th split
    int32_t n = 0;                   // the wave's splits of this pass, at most 64
    float ms, ls, x[kFirst][kPer], y[kMore][kPer];
    // (a row past the end is a repeat of the last)
    auto load_rows = [&](auto &v, int32_t i0) {
#pragma unroll
        for (int i = 0; i < (int)(sizeof(v) / sizeof(v[0])); ++i) {
            const int32_t sl = __builtin_amdgcn_readlane(slot, min(i0 + i, n - 1));
            const float *src = base + (int64_t)sl * stride + kPer * lane;
#pragma unroll
            for (int e = 0; e < kPer; ++e) v[i][e] = src[e];
        }
    };
    auto fetch = [&](int32_t k0) {
        n = min((total - wave + NW - 1) / NW - k0, 64);
        const int32_t s = min(wave + NW * (k0 + lane), total - 1);
        slot = own + s;
        if (n_runs >= 0) {
            const int32_t i = first + s;
            slot = s < n_runs ? ((i / r.n_page_splits) * r.n_kv + r.h) * r.n_splits + i % r.n_page_splits
                              : own + r.n_page_splits + (s - n_runs);
        }
        ms = -INFINITY;
        ls = 0.0f;
        if (n <= 0) return;
        if (lane < n) {
            const float *src = base + (int64_t)slot * stride + D;
            ms = src[0];
            ls = src[1];
        }
        load_rows(x, 0);
        if (n > kFirst) load_rows(y, kFirst);
    };
    fetch(0);
    if (r.runs != nullptr && r.runs[0] != 0) {
        first = r.runs[2 + 2 * r.b];
        n_runs = r.runs[2 + 2 * r.b + 1];
        total = n_runs + r.n_splits - r.n_page_splits;
        fetch(0);
    }
    float M = -INFINITY, l = 0.0f, o[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) o[e] = 0.0f;
    for (int32_t k0 = 0; n > 0;) {
        const float m_new = fmaxf(M, wave_max(ms));
        const float f = M == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(M - m_new);
        const float w = ms == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ms - m_new);
        l = fmaf(l, f, wave_sum(w * ls));
#pragma unroll
        for (int e = 0; e < kPer; ++e) o[e] *= f;
        M = m_new;
        // kFirst rows from v[at] on, rows i0 .. of the wave, i0 < n: the lanes
        // i0 .. i0 + kFirst - 1 exist (a lane number is taken modulo 64, and a
        // pass is a whole number of such batches), with weight 0 from n on
        static_assert(64 % kFirst == 0 && kMore % kFirst == 0, "no batch of rows crosses the wave's last lane");
        auto add_rows = [&](const auto &v, int at, int32_t i0) {
#pragma unroll
            for (int i = 0; i < kFirst; ++i) {
                const float wi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), i0 + i));
#pragma unroll
                for (int e = 0; e < kPer; ++e) o[e] = fmaf(wi, v[at + i][e], o[e]);
            }
        };
        add_rows(x, 0, 0);
        for (int32_t i0 = kFirst; i0 < n; i0 += kMore) {
            if (i0 > kFirst) load_rows(y, i0);
#pragma unroll
            for (int at = 0; at < kMore; at += kFirst)
                if (i0 + at < n) add_rows(y, at, i0 + at);
        }
        k0 += 64;
        fetch(k0);
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
