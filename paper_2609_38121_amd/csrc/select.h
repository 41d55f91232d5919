// Exact selection by min / max networks, for the order statistics of Eq.
// (7): sorting networks (Batcher's odd-even mergesort) for blocks, and
// bitonic sorters that keep the top K of two sorted lists.
//
// The lists hold the bit patterns of |x| for bf16 x: as integers these sort
// like the magnitudes.  The packed form (i16x2) works on two independent lists at a
// time, one per half word, with one packed instruction per minimum and
// maximum; a comparator then costs one instruction per element, as a
// median-of-three insertion step does, but a network needs far fewer of them
// (128 elements, K = 12: 6 per element instead of 14).  All indices are
// compile-time constants, so the lists stay in registers and comparators
// whose results nobody reads are dropped by the compiler.
#pragma once
#include "common.h"

namespace wushkv {

typedef __attribute__((ext_vector_type(2))) int16_t i16x2;

// Signed 16-bit order on both halves (magnitudes are below 2^15).
__device__ __forceinline__ i16x2 sel_max(i16x2 a, i16x2 b) { return __builtin_elementwise_max(a, b); }
__device__ __forceinline__ i16x2 sel_min(i16x2 a, i16x2 b) { return __builtin_elementwise_min(a, b); }

// x[i] the larger, x[j] the smaller.
template <typename T>
__device__ __forceinline__ void comparator(T &a, T &b)
{
    const T hi = sel_max(a, b), lo = sel_min(a, b);
    a = hi;
    b = lo;
}

__host__ __device__ constexpr int pow2_at_least(int k)
{
    int p = 1;
    while (p < k) p *= 2;
    return p;
}

// Batcher's odd-even merge of the sorted halves of x[lo .. lo + n - 1],
// taken every r-th element, and the mergesort built on it; descending.
template <int LO, int N, int R, typename T, int M>
__device__ __forceinline__ void odd_even_merge(T (&x)[M])
{
    constexpr int kStep = 2 * R;
    if constexpr (kStep < N) {
        odd_even_merge<LO, N, kStep>(x);
        odd_even_merge<LO + R, N, kStep>(x);
#pragma unroll
        for (int i = LO + R; i + R < LO + N; i += kStep) comparator(x[i], x[i + R]);
    } else {
        comparator(x[LO], x[LO + R]);
    }
}
template <int LO, int N, typename T, int M>
__device__ __forceinline__ void sort_block(T (&x)[M])
{
    if constexpr (N > 1) {
        sort_block<LO, N / 2>(x);
        sort_block<LO + N / 2, N / 2>(x);
        odd_even_merge<LO, N, 1>(x);
    }
}

// Every block of B elements sorted.
template <int LO, int B, typename T, int M>
__device__ __forceinline__ void sort_blocks(T (&x)[M])
{
    if constexpr (LO < M) {
        sort_block<LO, B>(x);
        sort_blocks<LO + B, B>(x);
    }
}

// Sorts (descending) the bitonic list c[0 .. K - 1]: the bitonic sorter of
// the next power of two, whose missing elements stand before c as larger
// than all (a comparator with one of them changes nothing).
template <int K, typename T>
__device__ __forceinline__ void bitonic_sort(T (&c)[K])
{
    constexpr int kP = pow2_at_least(K), kPad = kP - K;
#pragma unroll
    for (int dist = kP / 2; dist >= 1; dist /= 2)
#pragma unroll
        for (int i = 0; i < kP; ++i)
            if ((i & dist) == 0 && i >= kPad) comparator(c[i - kPad], c[i + dist - kPad]);
}

// The top K of two descending lists of K (b read backwards): a descending
// list against an ascending one, each larger value of a pair is in the top K
// of both and each smaller one is not.  The result is bitonic.
template <int K, typename T>
__device__ __forceinline__ void top_of_two(const T (&a)[K], const T (&b)[K], T (&c)[K])
{
#pragma unroll
    for (int i = 0; i < K; ++i) c[i] = sel_max(a[i], b[K - 1 - i]);
}

// The descending top K of x[0 .. N - 1] (N a multiple of the block of
// pow2_at_least(K) elements): blocks sorted, their top K merged.
template <int K, int N, typename T>
__device__ __forceinline__ void top_k(T (&x)[N], T (&t)[K])
{
    constexpr int kB = pow2_at_least(K) < N ? pow2_at_least(K) : N;
    static_assert(N % kB == 0 && kB >= K, "whole blocks of at least K");
    sort_blocks<0, kB>(x);
    T blk[N / kB][K];
#pragma unroll
    for (int b = 0; b < N / kB; ++b)
#pragma unroll
        for (int i = 0; i < K; ++i) blk[b][i] = x[kB * b + i];
#pragma unroll
    for (int w = N / kB / 2; w >= 1; w /= 2)
#pragma unroll
        for (int b = 0; b < w; ++b) {
            T c[K];
            top_of_two(blk[b], blk[b + w], c);
            bitonic_sort(c);
#pragma unroll
            for (int i = 0; i < K; ++i) blk[b][i] = c[i];
        }
#pragma unroll
    for (int i = 0; i < K; ++i) t[i] = blk[0][i];
}

}  // namespace wushkv
