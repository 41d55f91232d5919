// The quantiser shared by the append kernels and the fused decode step:
// kernel arguments of the append path, the per-token clip-range selection
// and parameters of Eq. (7) (and the QuEST projection of Eq. (5)), the
// tile quantiser writing codes and parameters into a page, and the flush of
// a range of positions from the recent ring (Alg. 2 steps 7-11).
#pragma once
#include <type_traits>

#include "common.h"
#include "select.h"

namespace wushkv {

// What an append launch does: quantise the ring positions that are due
// (kModeFlush), append the new tokens (kModeNew: quantise those that are due,
// write the others to the windows), or, for a large append, one half each of
// both: kModeQuant quantises every due position, from the ring or new, and
// kModeWindow then writes the windows.
enum { kModeFlush = 1, kModeNew = 2, kModeQuant = 4, kModeWindow = 8 };

struct AppendArgs {
    uint8_t *pages;
    const int32_t *page_table;
    uint16_t *win_k;
    uint16_t *win_v;
    int32_t *seq_len;
    int32_t *quant_end;
    int32_t *commit;     // [batch] arrivals of this launch's workgroups (zero between calls)
    int32_t arrivals;    // workgroups per sequence that report; 0: this launch does not commit
    int32_t n_kv, s_sink, s_keep, s_flush, win_slots, max_pages, n_pages;
    int32_t lo_k, lo_v;  // quantile positions: lo = floor(kappa (d-1))
    float t_k, t_v;      // and t = kappa (d-1) - lo
    int32_t codec;       // WUSHKV_CODEC_PCLIP (Eq. (7)) or WUSHKV_CODEC_QUEST (Eq. (5))
    int32_t levels;      // 2^b - 1 for b-bit codes (b = 3 codes sit in 4-bit fields)
    double quest_coef;   // QuEST: 2 alpha_b / (2^bits - 1)
    const uint16_t *k_new;
    const uint16_t *v_new;
    const int32_t *n_new;
    int32_t max_new;
    const uint16_t *tk;
    uint16_t *k_tilde_out;
    int32_t mode;
    int32_t sink_tiles;  // ceil(s_sink / 64)
    // headwise RMS normalisation + rotary embedding of the new keys (Alg. 2
    // step 1), applied when rope is not null
    const float *gain;   // [D] or null (one)
    float eps;
    const float *rope;   // [positions][D]: cos(s w_j) | sin(s w_j)
};

// RoPE(Norm(x)) of one key row held by four lanes (the lanes n + 16 j,
// j = 0..3 of a 16-lane column group): lane j holds channels 32 c + 8 j + e
// (c = 0..3, e = 0..7) in x[c][e].  The rotary partner of channel i < D/2
// is i + D/2, chunk c + D/64 of the same lane, so the rotation is local.
// Each step is a separately rounded fp32 operation.  The rotary table's
// entries for this lane (cos in rt[c][0..7], sin in rt[c][8..15] for the
// chunks c < D/64 of position pos) come from load_rope, so that their load
// can be issued with the row's own.
template <int D>
__device__ __forceinline__ void load_rope(const AppendArgs &a, int j, int32_t pos, float (&rt)[D / 64][16])
{
    const float *row = a.rope + (int64_t)pos * D;
#pragma unroll
    for (int c = 0; c < D / 64; ++c) {
        const float *cs = row + 32 * c + 8 * j;
        const float4 c0 = *reinterpret_cast<const float4 *>(cs);
        const float4 c1 = *reinterpret_cast<const float4 *>(cs + 4);
        const float4 s0 = *reinterpret_cast<const float4 *>(cs + D / 2);
        const float4 s1 = *reinterpret_cast<const float4 *>(cs + D / 2 + 4);
        const float v[16] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w,
                             s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
#pragma unroll
        for (int e = 0; e < 16; ++e) rt[c][e] = v[e];
    }
}

template <int D>
__device__ __forceinline__ void norm_rope_row(float (&x)[D / 32][8], int j, const float (&rt)[D / 64][16],
                                              const float *gain, float eps)
{
    constexpr int kC = D / 32;
    float ss = 0.0f;
#pragma unroll
    for (int c = 0; c < kC; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) ss = fmaf(x[c][e], x[c][e], ss);
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    const float r = 1.0f / sqrtf(ss / (float)D + eps);
    // (x r) g, or x r with no gain (a product by 1 is exact)
#pragma unroll
    for (int c = 0; c < kC; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[c][e] = x[c][e] * r;
    if (gain != nullptr) {
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            const float4 g0 = *reinterpret_cast<const float4 *>(gain + 32 * c + 8 * j);
            const float4 g1 = *reinterpret_cast<const float4 *>(gain + 32 * c + 8 * j + 4);
            const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) x[c][e] = x[c][e] * g[e];
        }
    }
#pragma unroll
    for (int c = 0; c < kC / 2; ++c) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float lo = x[c][e], hi = x[c + kC / 2][e];
            x[c][e] = lo * rt[c][e] - hi * rt[c][8 + e];
            x[c + kC / 2][e] = hi * rt[c][e] + lo * rt[c][8 + e];
        }
    }
}

template <int D>
__device__ __forceinline__ void norm_rope_row(float (&x)[D / 32][8], int j, int32_t pos, const AppendArgs &a)
{
    float rt[D / 64][16];
    load_rope<D>(a, j, pos, rt);
    norm_rope_row<D>(x, j, rt, a.gain, a.eps);
}

// Sequence b's counters as they stand before this launch: thread 0 reads
// S, S_quant and the new-token count and hands them to the whole workgroup
// through LDS (sh: three int32 of the caller's), so that every wave works
// with the very values thread 0's arrival is tied to (commit_arrive).  The
// count is clamped to [0, max_nn].  Every thread of the workgroup calls it;
// it contains a barrier.
struct SeqCounters {
    int32_t s_old, q_old, nn;
};
__device__ __forceinline__ SeqCounters read_counters(const AppendArgs &a, int b, int32_t max_nn,
                                                     int32_t *sh, int tid)
{
    if (tid == 0) {
        sh[0] = a.seq_len[b];
        sh[1] = a.quant_end[b];
        sh[2] = a.n_new[b];
    }
    __syncthreads();
    SeqCounters c{sh[0], sh[1], sh[2]};
    c.nn = c.nn < 0 ? 0 : (c.nn > max_nn ? max_nn : c.nn);
    return c;
}

// The same in a launch that reports no arrivals: every wave reads them.
__device__ __forceinline__ SeqCounters plain_counters(const AppendArgs &a, int b, int32_t max_nn)
{
    SeqCounters c{a.seq_len[b], a.quant_end[b], a.n_new[b]};
    c.nn = c.nn < 0 ? 0 : (c.nn > max_nn ? max_nn : c.nn);
    return c;
}

// Sequence b's counters advance from inside the launch that last reads
// them.  Each workgroup reports once, after its reads of seq_len and
// quant_end have returned (the values are tied to the report's operand), to
// the sequence's arrival count (commit_arrive, early in the workgroup's
// work); the workgroup that was last of a.arrivals writes S_new and
// S_quant_new and clears the count for the next call (commit_finish, at its
// end, so that the count's round trip overlaps its work).  Every workgroup
// of the sequence has read the old values before the last one arrives, so
// none can see the new ones: the other waves of a workgroup use thread 0's
// reads (read_counters).  Thread 0 only; a launch with a.arrivals = 0 leaves
// the counters alone (the quantising launch of a large append does, and the
// window launch after it advances them).
__device__ __forceinline__ int32_t commit_arrive(const AppendArgs &a, int b, int32_t s_old, int32_t q_old,
                                                 int32_t nn, int tid)
{
    if (a.arrivals <= 0 || tid != 0) return -1;
    int32_t one = 1;
    asm volatile("" : "+v"(one) : "v"(s_old), "v"(q_old), "v"(nn));
    return __hip_atomic_fetch_add(a.commit + b, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void commit_finish(const AppendArgs &a, int b, int32_t arrived, int32_t s_new,
                                              int32_t q_new, int tid)
{
    if (a.arrivals <= 0 || tid != 0 || arrived != a.arrivals - 1) return;
    a.seq_len[b] = s_new;
    a.quant_end[b] = q_new;
    __hip_atomic_store(a.commit + b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The value of the partner lane (lane ^ 1): the two lanes of a pair share
// one quantisation group, half of its elements each.
__device__ __forceinline__ float pair_swap(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xF,
                                                              0xF, false));
}

// |x| of a bf16 magnitude's pattern; -1 for the place of a NaN.
__device__ __forceinline__ float magnitude(int16_t bits)
{
    return bits < 0 ? -1.0f : bf16_bits_to_f32((uint32_t)bits);
}

// a_lo and a_{lo+1} of the ascending sort of |x| over a bf16 row in LDS,
// for lo = D - K (a_lo is the K-th largest), with the row's min and max.
// The lane pair (2 r, 2 r + 1) shares row r, half of it each; both lanes end
// with the same values.
//
// The vector units bound the append, so the row stays in its 16-bit form:
// each register's half words (even and odd channels) are two lists selected
// side by side by packed networks (select.h), whose top-K lists are merged
// across the lane pair and then across the halves, the last step only as far
// as the two smallest of the top K.  Per element that is 4.3 instructions
// at K = 7 and 6 at K = 12 (one v_med3 per list slot and element before: 9
// and 14).
//
// Extremes: bf16 patterns sort like the fp16 numbers with the same bits, so
// the packed fp16 maximum3 / minimum3 fold two registers per instruction.
// Patterns that are fp16 NaNs (|x| above 2^121, infinities, NaNs) come out as
// one: their rows take a slower path on the floats themselves, where a NaN
// counts for nothing (its magnitude sorts below every other, as -1).
template <int D, int K>
__device__ __forceinline__ void order_stats_topk(const uint16_t *row, int hf, float &a_lo, float &a_hi,
                                                 float &mn, float &mx)
{
    constexpr int kRegs = D / 4;  // registers of half a row, two elements each
    const uint16_t *half = row + hf * (D / 2);
    uint32_t w[kRegs];
#pragma unroll
    for (int c8 = 0; c8 < kRegs / 4; ++c8) {
        const u32x4 v = *reinterpret_cast<const u32x4 *>(half + 8 * c8);
#pragma unroll
        for (int q = 0; q < 4; ++q) w[4 * c8 + q] = v[q];
    }
    auto swap32 = [](auto x) {
        return __builtin_bit_cast(decltype(x), pair_swap(__builtin_bit_cast(float, x)));
    };
    f16x2 top = __builtin_bit_cast(f16x2, w[0]), bot = top;
#pragma unroll
    for (int i = 1; i < kRegs; ++i) {
        top = __builtin_elementwise_maximum(top, __builtin_bit_cast(f16x2, w[i]));
        bot = __builtin_elementwise_minimum(bot, __builtin_bit_cast(f16x2, w[i]));
    }
    top = __builtin_elementwise_maximum(top, swap32(top));
    bot = __builtin_elementwise_minimum(bot, swap32(bot));
    const uint32_t hi = __builtin_bit_cast(uint16_t, __builtin_elementwise_maximum(top[0], top[1]));
    const uint32_t lo = __builtin_bit_cast(uint16_t, __builtin_elementwise_minimum(bot[0], bot[1]));
    mx = bf16_bits_to_f32(hi);
    mn = bf16_bits_to_f32(lo);
    i16x2 x[kRegs];
#pragma unroll
    for (int i = 0; i < kRegs; ++i) x[i] = __builtin_bit_cast(i16x2, w[i] & 0x7FFF7FFFu);
    if (__any((hi & 0x7FFFu) > 0x7C00u)) {
        asm volatile("");  // a branch: this is not to be run and selected from
        mn = INFINITY;
        mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < kRegs; ++i) {
            const float f0 = bf16_bits_to_f32(w[i] & 0xFFFFu), f1 = bf16_bits_to_f32(w[i] >> 16);
            mn = fminf(fminf(mn, f0), f1);
            mx = fmaxf(fmaxf(mx, f0), f1);
#pragma unroll
            for (int e = 0; e < 2; ++e) x[i][e] = x[i][e] > 0x7F80 ? (int16_t)-1 : x[i][e];
        }
        mn = fminf(mn, pair_swap(mn));
        mx = fmaxf(mx, pair_swap(mx));
    }
    i16x2 t[K], c[K], o[K];
    top_k<K>(x, t);
#pragma unroll
    for (int i = 0; i < K; ++i) o[i] = swap32(t[i]);
    top_of_two(t, o, c);
    bitonic_sort(c);
#pragma unroll
    for (int i = 0; i < K; ++i) o[i] = i16x2{c[i][1], c[i][0]};
    top_of_two(c, o, t);
    bitonic_sort(t);
    a_lo = magnitude(t[K - 1][0]);
    a_hi = K > 1 ? magnitude(t[K > 1 ? K - 2 : 0][0]) : a_lo;
}

// Same order statistics by counting ranks: any lo, O(D^2) work.  Used when
// kappa is small enough that the top-k list would not fit in registers.
// Each lane of the pair ranks the elements of its half against the whole
// row; an order statistic is found in the half (or halves, for equal values)
// that holds it.
template <int D>
__device__ __forceinline__ void order_stats_rank(const uint16_t *row, int hf, int lo, float &a_lo,
                                              float &a_hi, float &mn, float &mx)
{
    mn = INFINITY;
    mx = -INFINITY;
    a_lo = -1.0f;
    a_hi = -1.0f;
    for (int e = hf * (D / 2); e < (hf + 1) * (D / 2); ++e) {
        float xe = bf16_bits_to_f32(row[e]);
        mn = fminf(mn, xe);
        mx = fmaxf(mx, xe);
        float ae = fabsf(xe);
        int less = 0, le = 0;
        for (int f = 0; f < D; ++f) {
            float af = fabsf(bf16_bits_to_f32(row[f]));
            less += (af < ae);
            le += (af <= ae);
        }
        // |x_e| occupies ascending ranks [less, le)
        if (less <= lo && lo < le) a_lo = ae;
        if (less <= lo + 1 && lo + 1 < le) a_hi = ae;
    }
    a_lo = fmaxf(a_lo, pair_swap(a_lo));
    a_hi = fmaxf(a_hi, pair_swap(a_hi));
    mn = fminf(mn, pair_swap(mn));
    mx = fmaxf(mx, pair_swap(mx));
    if (lo + 1 >= D) a_hi = a_lo;
}

// Eq. (7) parameters from the order statistics.  Every operation is a single
// correctly rounded fp32 operation (the file is built without contraction).
__device__ __forceinline__ void quant_params(float a_lo, float a_hi, float t, bool interp,
                                             float mn, float mx, int levels, uint32_t &s16,
                                             uint32_t &z16, float &z, float &inv)
{
    float q = a_lo;
    if (interp) {
        float diff = a_hi - a_lo;
        float prod = t * diff;
        q = a_lo + prod;
    }
    float x_min = (mn > -q) ? mn : -q;
    float x_max = (mx < q) ? mx : q;
    float delta = (x_max - x_min) / (float)levels;
    s16 = f32_to_f16_bits(delta);
    z16 = f32_to_f16_bits(x_min);
    float s = f16_bits_to_f32(s16);
    z = f16_bits_to_f32(z16);
    inv = (s > 0.0f) ? 1.0f / s : 0.0f;
}

// clamp(rne((x - z) inv), 0, levels) + kCodeBias.  Clamping to [0, levels]
// before the rounding gives the same integer (levels is an integer), and
// adding 2^23 to a value in [0, 2^23) rounds it to an integer in the default
// nearest-even mode, leaving that integer in the low bits of the sum, over
// the bits of 2^23.  The bias stays: words add up biased codes shifted to
// their places (one v_lshl_add_u32 each) and start from minus the sum of the
// shifted biases (code_word_start), modulo 2^32.
constexpr uint32_t kCodeBias = 0x4B000000u;
// word + (code << bit) for a constant bit, in one instruction (left to
// itself the compiler shifts, then adds in threes).
__device__ __forceinline__ void add_code(uint32_t &word, uint32_t code, int bit)
{
    asm("v_lshl_add_u32 %0, %1, %2, %0" : "+v"(word) : "v"(code), "i"(bit));
}
__device__ __forceinline__ uint32_t biased_code_of(float x, float z, float inv, float levels)
{
    const float y = (x - z) * inv;
    const float c = __builtin_amdgcn_fmed3f(y, 0.0f, levels);
    return __float_as_uint(c + 8388608.0f);
}

// Eq. (5) (QuEST) parameters of a group held by a lane pair (this lane's
// half of the channels from hf): the step is 2 alpha_b / (2^bits - 1) times
// the group's RMS, with the sum of squares in fp64 (each square exact, the
// two halves added last; the order does not change the result beyond fp64
// rounding) and the step rounded once to fp32 and then to the fp16 scale.
// The zero is the offset of the lowest bin centre, scale (1/2 - 2^(bits-1)),
// exact in fp32 and rounded to fp16.
// Eq. (5) parameters from the group's sum of squares ss (fp64).
// half = 2^(b-1) for b-bit codes.
template <int D>
__device__ __forceinline__ void quest_finish(double ss, double coef, float half, uint32_t &s16,
                                             uint32_t &z16, float &z, float &inv)
{
    const float step = (float)(coef * sqrt(ss / (double)D));
    s16 = f32_to_f16_bits(step);
    const float s = f16_bits_to_f32(s16);
    z16 = f32_to_f16_bits(s * (0.5f - half));
    z = f16_bits_to_f32(z16);
    inv = (s > 0.0f) ? 1.0f / s : 0.0f;
}

template <int D>
__device__ __forceinline__ void quest_params(const uint16_t *row, int hf, double coef, float h_levels,
                                             uint32_t &s16, uint32_t &z16, float &z, float &inv)
{
    const uint16_t *half = row + hf * (D / 2);
    double ss = 0.0;
#pragma unroll 4
    for (int c8 = 0; c8 < D / 16; ++c8) {
        uint4 v = *reinterpret_cast<const uint4 *>(half + 8 * c8);
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double lo = (double)bf16_bits_to_f32(w[q] & 0xFFFFu);
            const double hi = (double)bf16_bits_to_f32(w[q] >> 16);
            ss = fma(lo, lo, ss);
            ss = fma(hi, hi, ss);
        }
    }
    const uint64_t u = __builtin_bit_cast(uint64_t, ss);
    const uint32_t plo = __builtin_bit_cast(uint32_t, pair_swap(__builtin_bit_cast(float, (uint32_t)u)));
    const uint32_t phi = __builtin_bit_cast(uint32_t, pair_swap(__builtin_bit_cast(float, (uint32_t)(u >> 32))));
    ss += __builtin_bit_cast(double, ((uint64_t)phi << 32) | plo);
    quest_finish<D>(ss, coef, h_levels, s16, z16, z, inv);
}

// clamp(floor(x inv) + h, 0, levels) - h of Eq. (5), h = 2^(bits-1): the
// clamp to [-h, levels - h + 1/2] first, then the floor with the conversion
// to an integer in one instruction.  (A NaN clamps to the lower end, code 0.)
// Words start from h at every code's place, as with kCodeBias.
__device__ __forceinline__ uint32_t biased_quest_code_of(float x, float inv, float h, float levels)
{
    const float y = __builtin_amdgcn_fmed3f(x * inv, -h, levels - h + 0.5f);
    uint32_t c;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(c) : "v"(y));
    return c;
}

// The selection for K = D - lo: the top-K lists for K = KC .. 16 (each its
// own exact length), the rank count beyond.
template <int D, int KC = 1>
__device__ __forceinline__ void order_stats(const uint16_t *row, int hf, int lo, float &a_lo, float &a_hi,
                                            float &mn, float &mx)
{
    if (D - lo == KC) order_stats_topk<D, KC>(row, hf, a_lo, a_hi, mn, mx);
    else if constexpr (KC < 16) order_stats<D, KC + 1>(row, hf, lo, a_lo, a_hi, mn, mx);
    else order_stats_rank<D>(row, hf, lo, a_lo, a_hi, mn, mx);
}

// Value codes (one byte each) are written over the value row they come
// from: the lane holding channels [h D / 2, (h + 1) D / 2) of row t writes
// their codes at bytes h D .. h D + D / 2 - 1 of that row, inside the bytes
// it has already read.
template <int D>
__device__ __forceinline__ uint8_t *vcode_row(uint16_t *vt, int t)
{
    return reinterpret_cast<uint8_t *>(vt + t * (D + 8));
}

// Phase C of a tile: the value-code words of its tokens [t0, t1) (both
// multiples of 8: a word holds eight tokens), from the code bytes that phase
// B left in the value rows (vcode_row).
//
// Four channels a thread: it reads their code bytes of a token as one word,
// gathers the tokens whose codes share byte k of the output words into word k
// (the codes leave the upper bits of their bytes free, and no field of a word
// crosses a byte), and transposes the four words' bytes: 16 reads and 20
// vector instructions for four 2-bit words, where a byte read and a shift-or
// per code took 64.
template <int D, int BITS>
__device__ void whole_value_words(uint16_t *vt, int t0, int t1, uint8_t *pg, int tid)
{
    using L = Layout<D, BITS>;
    constexpr int kRowBytes = 2 * (D + 8);
    uint32_t *vreg = reinterpret_cast<uint32_t *>(pg + L::kRegionBytes);
    constexpr int kU = 2 * L::kNw;  // words of a lane and 32-token slice
    // items: (eight tokens, four channels, u)
    for (int idx = (t0 / 8) * 4 * kU + tid; idx < (t1 / 8) * 4 * kU; idx += 256) {
        const int u = idx % kU, m0 = 4 * ((idx / kU) & 3), j = (idx / (4 * kU)) & 3, kc = idx / (16 * kU);
        const uint8_t *base = vcode_row<D>(vt, 32 * kc + 8 * j);  // token i at + i kRowBytes
        uint32_t g[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < L::kCodesPerWord; ++e) {
            const int o = e >> 3, i = e & 7;
            const int ch = 16 * (u * L::kOpsPerWord + o) + m0;
            const uint32_t codes =
                *reinterpret_cast<const uint32_t *>(base + i * kRowBytes + ch + (ch >= D / 2 ? D / 2 : 0));
            g[L::v_bit(o, i) / 8] |= codes << (L::v_bit(o, i) % 8);
        }
        // bytes (0, 1) and (2, 3) of each pair of words interleaved, then
        // the halves joined: word c is byte c of g[0 .. 3]
        const uint32_t a0 = __builtin_amdgcn_perm(g[1], g[0], 0x05010400u);
        const uint32_t a1 = __builtin_amdgcn_perm(g[1], g[0], 0x07030602u);
        const uint32_t b0 = __builtin_amdgcn_perm(g[3], g[2], 0x05010400u);
        const uint32_t b1 = __builtin_amdgcn_perm(g[3], g[2], 0x07030602u);
        const uint32_t word[4] = {
            __builtin_amdgcn_perm(b0, a0, 0x05040100u), __builtin_amdgcn_perm(b0, a0, 0x07060302u),
            __builtin_amdgcn_perm(b1, a1, 0x05040100u), __builtin_amdgcn_perm(b1, a1, 0x07060302u)};
#pragma unroll
        for (int c = 0; c < 4; ++c) vreg[L::v_word(16 * j + m0 + c, kc * kU + u)] = word[c];
    }
}

// Phase C for any set of positions of the tile: the codes of positions with
// quant(p) merged into what the page holds.
template <int D, int BITS, typename Pred>
__device__ void value_words(uint16_t *vt, int32_t blk_lo, Pred quant, uint8_t *pg, int tid)
{
    using L = Layout<D, BITS>;
    if (pg != nullptr) {
        uint32_t *vreg = reinterpret_cast<uint32_t *>(pg + L::kRegionBytes);
        constexpr int kWords = 64 * L::kWordsPerLane;
        for (int idx = tid; idx < kWords; idx += 256) {
            const int Ln = idx / L::kWordsPerLane, rem = idx % L::kWordsPerLane;
            const int kc = rem / (2 * L::kNw), u = rem % (2 * L::kNw);
            const int widx = L::v_word(Ln, rem);
            const int j = Ln >> 4, m = Ln & 15;
            uint32_t mask = 0, bits = 0;
#pragma unroll
            for (int e = 0; e < L::kCodesPerWord; ++e) {
                const int o = e >> 3, i = e & 7;
                const int t = 32 * kc + 8 * j + i;
                const int32_t p = blk_lo + t;
                if (quant(p)) {
                    const int ch = 16 * (u * L::kOpsPerWord + o) + m;
                    const int bit = L::v_bit(o, i);
                    mask |= ((1u << BITS) - 1u) << bit;
                    bits |= (uint32_t)vcode_row<D>(vt, t)[ch + (ch >= D / 2 ? D / 2 : 0)] << bit;
                }
            }
            if (mask == 0u) continue;
            if (mask != 0xFFFFFFFFu) bits |= vreg[widx] & ~mask;
            vreg[widx] = bits;
        }
    }
}

// Phases B and C of a tile of up to 64 positions starting at blk_lo, all in
// one page (pg, or null when the page is outside the pool): quantise every
// position p with quant(p) from its bf16 rows in kt / vt (row p - blk_lo),
// write its parameters and key words, then assemble the value words, merging
// words only partly covered with what the page holds.  all_quant: the
// caller's statement that quant(p) holds for every p of [blk_lo, blk_lo +
// 64) (the common case of a prefill); the value words are then assembled
// without per-code checks or merges.  Every thread of the workgroup must
// call it (it synchronises).
template <int D, int BITS, typename Pred>
__device__ void quantise_tile(const AppendArgs &a, const uint16_t *kt, uint16_t *vt,
                              int32_t blk_lo, Pred quant, bool all_quant, uint8_t *pg, int tid)
{
    using L = Layout<D, BITS>;
    constexpr int kPitch = D + 8;
    const bool full = all_quant && pg != nullptr;
    // ---- phase B: quantise.  Lanes 2 r and 2 r + 1 share group r (rows
    // 0-63 keys, 64-127 values), one half of its channels each, so that all
    // four waves take part.
    {
        const int grp = tid >> 1, hf = tid & 1;
        const bool is_v = grp >= kPage;
        const int r = grp & (kPage - 1);
        const int32_t p = blk_lo + r;
        if (quant(p) && pg != nullptr) {  // the same for both lanes of the pair
            const uint16_t *row = (is_v ? vt : kt) + r * kPitch;
            uint32_t s16, z16;
            float z, inv;
            const int kLevels = a.levels;             // 2^b - 1 (b = 3 in 4-bit fields)
            const float kMid = (float)((kLevels + 1) / 2);  // 2^(b-1)
            const bool quest = a.codec == WUSHKV_CODEC_QUEST;
            if (quest) {
                quest_params<D>(row, hf, a.quest_coef, kMid, s16, z16, z, inv);
            } else {
                const int qlo = is_v ? a.lo_v : a.lo_k;
                const float qt = is_v ? a.t_v : a.t_k;
                float a_lo, a_hi, mn, mx;
                order_stats<D>(row, hf, qlo, a_lo, a_hi, mn, mx);
                quant_params(a_lo, a_hi, qt, qlo + 1 < D, mn, mx, kLevels, s16, z16, z, inv);
            }
            if (hf == 0)
                *reinterpret_cast<uint32_t *>(pg + L::kParamOffset + 4 * r + (is_v ? 4 * kPage : 0)) =
                    s16 | (z16 << 16);
            constexpr int kHalf = D / 2;
            const int c0 = hf * kHalf;  // first channel of this lane's half
            // the code loops, instantiated once per codec's code formula
            auto write_codes = [&](uint32_t code_bias, auto code_fn) {
                if (!is_v) {
                    // key words of this token: lane group jj = ch / 32 holds
                    // BITS words per token (see Layout::k_pos); this half covers
                    // groups hf D / 64 .. (hf + 1) D / 64 - 1
                    uint32_t kw[D / 64][BITS];
#pragma unroll
                    for (int jl = 0; jl < D / 64; ++jl)
#pragma unroll
                        for (int w = 0; w < BITS; ++w) {
                            uint32_t ones = 0u;  // a one at each code's place
#pragma unroll
                            for (int e = 0; e < 32 / BITS; ++e) {
                                int word, bit;
                                L::k_pos(0, e, word, bit);
                                ones += 1u << bit;
                            }
                            kw[jl][w] = 0u - code_bias * ones;
                        }
#pragma unroll
                    for (int c8 = 0; c8 < kHalf / 8; ++c8) {
                        uint4 v = *reinterpret_cast<const uint4 *>(row + c0 + 8 * c8);
                        uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            uint32_t hb = (i & 1) ? (wv[i >> 1] >> 16) : (wv[i >> 1] & 0xFFFFu);
                            uint32_t code = code_fn(bf16_bits_to_f32(hb));
                            const int cl = 8 * c8 + i;  // channel c0 + cl
                            int word, bit;
                            L::k_pos(r, c0 + cl, word, bit);
                            add_code(kw[cl >> 5][(cl & 31) / (32 / BITS)], code, bit);
                        }
                    }
                    uint32_t *kreg = reinterpret_cast<uint32_t *>(pg);
#pragma unroll
                    for (int jl = 0; jl < D / 64; ++jl)
#pragma unroll
                        for (int w = 0; w < BITS; ++w)
                            kreg[L::k_word(16 * (hf * (D / 64) + jl) + (r >> 2), BITS * (r & 3) + w)] = kw[jl][w];
                } else {
#pragma unroll
                    for (int c8 = 0; c8 < kHalf / 8; ++c8) {
                        uint4 v = *reinterpret_cast<const uint4 *>(row + c0 + 8 * c8);
                        uint32_t wv[4] = {v.x, v.y, v.z, v.w};
                        uint32_t lo4 = 0u - code_bias * 0x01010101u, hi4 = lo4;
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            uint32_t hb = (i & 1) ? (wv[i >> 1] >> 16) : (wv[i >> 1] & 0xFFFFu);
                            uint32_t code = code_fn(bf16_bits_to_f32(hb));
                            add_code(i < 4 ? lo4 : hi4, code, 8 * (i & 3));
                        }
                        // over bytes of this lane's half of the row that it has read
                        *reinterpret_cast<uint2 *>(vcode_row<D>(vt, r) + hf * D + 8 * c8) = make_uint2(lo4, hi4);
                    }
                }
            };
            const float kLv = (float)kLevels;
            if (quest) {
                // Eq. (5): clamp(floor(x inv) + 2^(bits-1))
                write_codes(0u - (uint32_t)((kLevels + 1) / 2), [&](float x) { return biased_quest_code_of(x, inv, kMid, kLv); });
            } else {
                // Eq. (7): clamp(rne((x - z) inv))
                write_codes(kCodeBias, [&](float x) { return biased_code_of(x, z, inv, kLv); });
            }
        }
    }
    __syncthreads();

    if (full) whole_value_words<D, BITS>(vt, 0, kPage, pg, tid);
    else value_words<D, BITS>(vt, blk_lo, quant, pg, tid);
}

// ------------------------------------------------ few positions, wide groups

// Lane exchanges inside each row of 16 lanes (DPP): partner lane ^ 1, ^ 2
// (quad permutations), 7 - lane within 8 and 15 - lane within 16 (the half
// mirror and the mirror).  Applied in that order they combine all 16 lanes,
// as a butterfly does.
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kCtrl, 0xF, 0xF, false);
}
template <int kStep>
__device__ __forceinline__ uint32_t row16_swap(uint32_t x)
{
    constexpr int kCtrl = kStep == 0 ? 0xB1 : kStep == 1 ? 0x4E : kStep == 2 ? 0x141 : 0x140;
    return dpp_u32<kCtrl>(x);
}
template <int kStep>
__device__ __forceinline__ float row16_swap(float x)
{
    return __builtin_bit_cast(float, row16_swap<kStep>(__builtin_bit_cast(uint32_t, x)));
}

// The descending top min(K, 2 N) of a lane's list t[0 .. N - 1] and its
// partner's at exchange step kStep.
template <int kStep, int K, int N>
__device__ __forceinline__ void merge_lanes(const i16x2 (&t)[N], i16x2 (&c)[K < 2 * N ? K : 2 * N])
{
    i16x2 o[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
        o[i] = __builtin_bit_cast(i16x2, row16_swap<kStep>(__builtin_bit_cast(uint32_t, t[i])));
    if constexpr (K <= N) {
        static_assert(K == N, "lists hold at most K");
        top_of_two(t, o, c);
        bitonic_sort(c);
    } else {
        // all of both lists: a descending one, then an ascending one
        i16x2 all[2 * N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            all[i] = t[i];
            all[N + i] = o[N - 1 - i];
        }
        bitonic_sort(all);
#pragma unroll
        for (int i = 0; i < (K < 2 * N ? K : 2 * N); ++i) c[i] = all[i];
    }
}

// The order statistics of order_stats_topk over a group held by 16 lanes,
// two elements to each of a lane's kRegs registers: the half words' lists are
// sorted in the lane, merged over the four exchange steps (every lane ends
// with the top K of its half words' lists), then across the halves.  (As
// median insertions of the partner's list at each step: 730 dependent
// instructions at K = 12, 8 channels a lane; these networks: 260.)
template <int K, int kRegs>
__device__ __forceinline__ void few_order_stats(const uint32_t (&w)[kRegs], float &a_lo, float &a_hi,
                                                float &mn, float &mx)
{
    mn = INFINITY;
    mx = -INFINITY;
    i16x2 x[kRegs];
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
        const float f0 = bf16_bits_to_f32(w[i] & 0xFFFFu), f1 = bf16_bits_to_f32(w[i] >> 16);
        mn = fminf(fminf(mn, f0), f1);
        mx = fmaxf(fmaxf(mx, f0), f1);
        x[i] = __builtin_bit_cast(i16x2, w[i] & 0x7FFF7FFFu);
#pragma unroll
        for (int e = 0; e < 2; ++e) x[i][e] = x[i][e] > 0x7F80 ? (int16_t)-1 : x[i][e];  // (a NaN)
    }
    auto extremes = [&](auto st) {
        constexpr int kStep = decltype(st)::value;
        mn = fminf(mn, row16_swap<kStep>(mn));
        mx = fmaxf(mx, row16_swap<kStep>(mx));
    };
    extremes(std::integral_constant<int, 0>{});
    extremes(std::integral_constant<int, 1>{});
    extremes(std::integral_constant<int, 2>{});
    extremes(std::integral_constant<int, 3>{});
    constexpr int k0 = K < kRegs ? K : kRegs, k1 = K < 2 * k0 ? K : 2 * k0, k2 = K < 2 * k1 ? K : 2 * k1,
                  k3 = K < 2 * k2 ? K : 2 * k2, k4 = K < 2 * k3 ? K : 2 * k3;
    static_assert(k4 == K, "16 lanes hold at least K of each half");
    sort_blocks<0, kRegs>(x);
    i16x2 t0[k0], t1[k1], t2[k2], t3[k3], t[K], o[K], c[K];
#pragma unroll
    for (int i = 0; i < k0; ++i) t0[i] = x[i];
    merge_lanes<0, K>(t0, t1);
    merge_lanes<1, K>(t1, t2);
    merge_lanes<2, K>(t2, t3);
    merge_lanes<3, K>(t3, t);
#pragma unroll
    for (int i = 0; i < K; ++i) o[i] = i16x2{t[i][1], t[i][0]};
    top_of_two(t, o, c);
    bitonic_sort(c);
    a_lo = magnitude(c[K - 1][0]);
    a_hi = K > 1 ? magnitude(c[K > 1 ? K - 2 : 0][0]) : a_lo;
}

template <int kRegs, int KC = 1>
__device__ __forceinline__ void few_order_stats_of(int K, const uint32_t (&w)[kRegs], float &a_lo, float &a_hi,
                                                   float &mn, float &mx)
{
    if (K == KC) few_order_stats<KC>(w, a_lo, a_hi, mn, mx);
    else if constexpr (KC < 16) few_order_stats_of<kRegs, KC + 1>(K, w, a_lo, a_hi, mn, mx);
}

// Phases B and C for a short range of positions [lo, hi) of the tile at
// blk_lo (one page, pg, or null outside the pool), eight at a time with 16
// lanes per quantisation group: group g = tid / 16 is the key row (g < 8) or
// the value row (g >= 8) of position lo + g % 8 (then lo + 8 + g % 8, ..),
// lane s = tid % 16 holds its channels kPer s .. kPer s + kPer - 1.  The
// parameters, codes and words are those quantise_tile writes (the selection
// keeps the same multiset; the QuEST sum of squares is exact in fp64 for bf16
// inputs of the usual range, so its order does not matter).  Needs D - lo_k
// and D - lo_v <= 16 for Eq. (7).  Every thread of the workgroup calls it.
template <int D, int BITS>
__device__ void quantise_few(const AppendArgs &a, uint16_t *kt, uint16_t *vt, int32_t blk_lo,
                             int32_t lo, int32_t hi, uint8_t *pg, int tid)
{
    using L = Layout<D, BITS>;
    constexpr int kPitch = D + 8;
    constexpr int kPer = D / 16;                 // channels per lane: 8 or 4
    const int kLevels = a.levels;                // 2^b - 1 (b = 3 in 4-bit fields)
    const float kHalf = (float)((kLevels + 1) / 2);  // 2^(b-1)
    constexpr int kPerWord = 32 / BITS;          // key codes per word
    constexpr int kLanesPerWord = kPerWord / kPer;  // 1, 2 or 4
    const int g = tid >> 4, sl = tid & 15;
    const bool is_v = g >= 8;
    const int r0 = lo - blk_lo, r1 = hi - blk_lo;
    for (int r = r0 + (g & 7); r < r1 && pg != nullptr; r += 8) {  // uniform over the group's 16 lanes
        uint16_t *row = (is_v ? vt : kt) + r * kPitch;
        const int ch0 = kPer * sl;
        uint32_t w[kPer / 2];
        if constexpr (kPer == 8) {
            const uint4 v = *reinterpret_cast<const uint4 *>(row + ch0);
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        } else {
            const uint2 v = *reinterpret_cast<const uint2 *>(row + ch0);
            w[0] = v.x; w[1] = v.y;
        }
        float x[kPer];
#pragma unroll
        for (int e = 0; e < kPer; ++e) x[e] = bf16_bits_to_f32((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu));
        uint32_t s16, z16;
        float z, inv;
        const bool quest = a.codec == WUSHKV_CODEC_QUEST;
        if (quest) {
            double ss = 0.0;
#pragma unroll
            for (int e = 0; e < kPer; ++e) ss = fma((double)x[e], (double)x[e], ss);
            auto add = [&](auto st) {
                constexpr int kStep = decltype(st)::value;
                const uint64_t u = __builtin_bit_cast(uint64_t, ss);
                const uint64_t o = ((uint64_t)row16_swap<kStep>((uint32_t)(u >> 32)) << 32) |
                                   row16_swap<kStep>((uint32_t)u);
                ss += __builtin_bit_cast(double, o);
            };
            add(std::integral_constant<int, 0>{});
            add(std::integral_constant<int, 1>{});
            add(std::integral_constant<int, 2>{});
            add(std::integral_constant<int, 3>{});
            quest_finish<D>(ss, a.quest_coef, kHalf, s16, z16, z, inv);
        } else {
            const int qlo = is_v ? a.lo_v : a.lo_k;
            const float qt = is_v ? a.t_v : a.t_k;
            float a_lo, a_hi, mn, mx;
            few_order_stats_of(D - qlo, w, a_lo, a_hi, mn, mx);
            quant_params(a_lo, a_hi, qt, qlo + 1 < D, mn, mx, kLevels, s16, z16, z, inv);
        }
        if (sl == 0)
            *reinterpret_cast<uint32_t *>(pg + L::kParamOffset + 4 * r + (is_v ? 4 * kPage : 0)) =
                s16 | (z16 << 16);
        uint32_t code[kPer];
        const float kLv = (float)kLevels;
#pragma unroll
        for (int e = 0; e < kPer; ++e)
            code[e] = quest ? biased_quest_code_of(x[e], inv, kHalf, kLv) + (uint32_t)((kLevels + 1) / 2)
                            : biased_code_of(x[e], z, inv, kLv) - kCodeBias;
        if (!is_v) {
            // this lane's channels lie in one key word: word w of 32-channel
            // chunk jc; the lanes sharing the word OR their bits together
            uint32_t bits = 0;
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                int word, bit;
                L::k_pos(r, ch0 + e, word, bit);
                bits |= code[e] << bit;
            }
            if constexpr (kLanesPerWord >= 2) bits |= row16_swap<0>(bits);
            if constexpr (kLanesPerWord >= 4) bits |= row16_swap<1>(bits);
            if (sl % kLanesPerWord == 0) {
                const int jc = ch0 >> 5, w = (ch0 & 31) / kPerWord;
                reinterpret_cast<uint32_t *>(pg)[L::k_word(16 * jc + (r >> 2), BITS * (r & 3) + w)] = bits;
            }
        } else {
            // code bytes over the row, where phase C reads them (the whole
            // row was read by this wave's one load above)
            uint8_t *dst = vcode_row<D>(vt, r) + ch0 + (ch0 >= D / 2 ? D / 2 : 0);
            if constexpr (kPer == 8) {
                *reinterpret_cast<uint2 *>(dst) =
                    make_uint2(code[0] | code[1] << 8 | code[2] << 16 | code[3] << 24,
                               code[4] | code[5] << 8 | code[6] << 16 | code[7] << 24);
            } else {
                *reinterpret_cast<uint32_t *>(dst) = code[0] | code[1] << 8 | code[2] << 16 | code[3] << 24;
            }
        }
    }
    __syncthreads();
    if (pg != nullptr && ((r0 | r1) & 7) == 0) whole_value_words<D, BITS>(vt, r0, r1, pg, tid);
    else value_words<D, BITS>(vt, blk_lo, [&](int32_t p) { return p >= lo && p < hi; }, pg, tid);
}

// Quantise positions [start, q_new) of (sequence b, kv head h) into their
// pages, one 64-position block at a time (Alg. 2 steps 7-11).  A position
// before s_ring comes from the windows' ring (keys row-major, values
// channel-major); one at or after it is a new token of this call, its key
// already transformed in kn and its value in vn (LDS, pitch D + 8).  kt and
// vt are 64-row LDS tiles, sh one LDS word.  Every thread of the 256-thread
// workgroup calls it.  kNewRows false: every position comes from the ring
// (s_ring, kn and vn unused).
template <int D, int BITS, bool kNewRows>
__device__ void flush_range(const AppendArgs &a, int b, int h, int32_t start, int32_t q_new,
                            int32_t s_ring, const uint16_t *kn, const uint16_t *vn, uint16_t *kt,
                            uint16_t *vt, int32_t *sh, int tid)
{
    using L = Layout<D, BITS>;
    constexpr int kPitch = D + 8;
    constexpr int kVec = D / 8;
    const int32_t ring = a.win_slots - a.s_sink;
    const int64_t head_win = ((int64_t)b * a.n_kv + h) * a.win_slots;
    for (int32_t blk = a.s_sink + (start - a.s_sink) / kPage * kPage; blk < q_new; blk += kPage) {
        const int32_t lo = max(blk, start), hi = min(blk + kPage, q_new);
        for (int idx = tid; idx < (hi - lo) * kVec; idx += 256) {
            const int cv = idx % kVec;
            const int32_t p = lo + idx / kVec;
            const int r = p - blk;
            uint4 kv, vv;
            if (kNewRows && p >= s_ring) {
                kv = *reinterpret_cast<const uint4 *>(kn + (p - s_ring) * kPitch + 8 * cv);
                vv = *reinterpret_cast<const uint4 *>(vn + (p - s_ring) * kPitch + 8 * cv);
            } else {
                const int32_t slot = ring_slot(p, a.s_sink, ring);
                kv = *reinterpret_cast<const uint4 *>(a.win_k + (head_win + slot) * D + 8 * cv);
                const uint16_t *vsrc = a.win_v + (head_win * D) + slot;  // channel-major
                uint16_t e[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) e[q] = vsrc[(int64_t)(8 * cv + q) * a.win_slots];
                vv.x = e[0] | ((uint32_t)e[1] << 16);
                vv.y = e[2] | ((uint32_t)e[3] << 16);
                vv.z = e[4] | ((uint32_t)e[5] << 16);
                vv.w = e[6] | ((uint32_t)e[7] << 16);
            }
            *reinterpret_cast<uint4 *>(kt + r * kPitch + 8 * cv) = kv;
            *reinterpret_cast<uint4 *>(vt + r * kPitch + 8 * cv) = vv;
        }
        if (tid == 0) {
            const int32_t lp = (blk - a.s_sink) / kPage;
            int32_t phys = -1;
            if (lp < a.max_pages) {
                phys = a.page_table[(int64_t)b * a.max_pages + lp];
                if (phys < 0 || phys >= a.n_pages) phys = -1;
            }
            sh[0] = phys;
        }
        __syncthreads();
        const int32_t page = sh[0];
        uint8_t *pg = page >= 0 ? a.pages + ((int64_t)page * a.n_kv + h) * L::kPageBytes : nullptr;
        // a short range (the flush of a decode step or of a 16-token chunk):
        // 16 lanes per group (of 16 rows the lane-pair tile would keep a
        // quarter of its lanes busy, for as long as all 64 take)
        const bool few = hi - lo <= 16 &&
                         (a.codec == WUSHKV_CODEC_QUEST || (D - a.lo_k <= 16 && D - a.lo_v <= 16));
        if (few)
            quantise_few<D, BITS>(a, kt, vt, blk, lo, hi, pg, tid);
        else
            quantise_tile<D, BITS>(a, kt, vt, blk, [&](int32_t p) { return p >= lo && p < hi; },
                                   lo <= blk && blk + kPage <= hi, pg, tid);
        __syncthreads();
    }
}

}  // namespace wushkv
