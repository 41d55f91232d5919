// wushkv_wush_transform: the WUSH transform of Eq. (1) for a batch of
// (Gram matrix M, Hessian H) pairs, one d x d transform per pair (Sec. 3;
// per key or value head in Eq. (4) and Alg. 1).
//
//   L L^T = H_d = H + gamma tr(H)/d I            Cholesky
//   U Lam U^T = L^T M_d L,  M_d = M + gamma tr(M)/d I
//   c = ((1 + gamma) tr(M))^(1/2) tr(Lam^(1/2))^(-1/2)
//   T = c Had Lam^(-1/4) U^T L^T,   T^{-1} = c^{-1} M_d (L U) Lam^(-3/4) Had
//
// (the second form of T^{-1} follows from L^{-T} U = M_d L U Lam^{-1}).
//
// One workgroup per pair, two on a compute unit, around one LDS frame of
// d + 1 columns of d entries (fp32):
//   1. H_d in the lower triangle of columns 0 .. d - 1, M_d transposed in the
//      upper triangle of columns 1 .. d; both Cholesky factors, L and R
//      (M_d = R R^T), at once, one barrier per column;
//   2. B = R^T L, so that B^T B = L^T M_d L;
//   3. one-sided (Hestenes) Jacobi on the columns of B: plane rotations that
//      make them mutually orthogonal, applied to the columns of L as well.  At
//      convergence the B columns have squared norms Lam and the L columns are
//      L U: the eigendecomposition without forming L^T M_d L, and with the
//      eigenvalues' relative accuracy of a one-sided method.  The d/2 disjoint
//      pairs of a round (a round-robin tournament) rotate in parallel, each by
//      1024/d threads (512 per workgroup).  B is in the frame; L, whose rows
//      need nothing of a round but its rotations, is in registers, a row to
//      512/d threads, and moves through them as the tournament turns;
//   4. the eigenpairs in ascending order, each eigenvector's sign fixed so
//      that the largest-magnitude entry of L u_k is positive (the paper
//      fixes neither; Had mixes them, so T depends on both);
//   5. T by a fast Walsh-Hadamard transform of the rows Lam^(-1/4) (L U)^T,
//      and T^{-1} from the product M_d (L U) and a second transform (M_d waits
//      in T^{-1}'s own memory: a pair's inputs are read whole before its
//      outputs are first written).
// The rounds bound it: a chain of LDS reads, dot products, the rotation and
// writes between two barriers, which the second workgroup fills.  With L in
// the frame too there is room for one workgroup, and twice the LDS traffic of
// a round: 512 pairs of d = 128 took 4.61 ms, now 2.96 (the same
// operations on the same numbers in the same order).
#include <cmath>
#include <type_traits>

#include "common.h"

namespace wushkv {

constexpr int kWushMaxSweeps = 40;
// Threads of a workgroup: eight waves, two per SIMD, and two workgroups per
// compute unit, so that one wave's LDS and barrier waits overlap the others'
// arithmetic.
constexpr int kWushThreads = 512;
constexpr int kWushWaves = kWushThreads / 64;

// Sum of one value per wave (in red[wave]) in a fixed order.
__device__ __forceinline__ float wave_total(const float *red)
{
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < kWushWaves; ++w) t += red[w];
    return t;
}

// The frame: column stride 16-byte aligned, four banks apart for neighbouring
// columns.
template <int D>
struct WushLds {
    static constexpr int kP = D + 4;
    static constexpr int kFloats = (D + 1) * kP;
};

// Lane exchange within aligned groups of N lanes (N a power of two <= 64):
// the sum over the group, the same value in every lane of the group (each
// step adds the same two partial sums in every lane, so all lanes agree bit
// for bit).  Groups of up to 16 lanes sum by DPP inside the lanes' row:
// quad permutations, then the half-row and the row mirrors, which pair each
// quad (each half row) with the other one of its group.
template <int CTRL>
__device__ __forceinline__ float wush_dpp(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF,
                                                                  0xF, false));
}
template <int N>
__device__ __forceinline__ float group_sum(float x)
{
    if constexpr (N <= 16) {
        if constexpr (N >= 2) x += wush_dpp<0xB1>(x);   // quad_perm [1, 0, 3, 2]
        if constexpr (N >= 4) x += wush_dpp<0x4E>(x);   // quad_perm [2, 3, 0, 1]
        if constexpr (N >= 8) x += wush_dpp<0x141>(x);  // row_half_mirror
        if constexpr (N >= 16) x += wush_dpp<0x140>(x); // row_mirror
        return x;
    } else {
#pragma unroll
        for (int off = 1; off < N; off <<= 1) x += __shfl_xor(x, off);
        return x;
    }
}

// Trace of the row-major matrix A.
template <int D>
__device__ float trace_of(const float *A, int tid, float *red)
{
    float t = 0.0f;
    for (int i = tid; i < D; i += kWushThreads) t += A[i * D + i];
    t = group_sum<64>(t);
    __syncthreads();  // red may still be read
    if ((tid & 63) == 0) red[tid >> 6] = t;
    __syncthreads();
    return wave_total(red);
}

// Both in-place Cholesky factorisations.  H_d's entry (i, k), i >= k, is
// X[k P + i] and M_d's X[(i + 1) P + k].  Step j subtracts l_i l_k from the
// trailing lower triangles, l = column j over the root of its pivot, one
// barrier a step: the columns themselves are scaled at the end (piv_l, piv_r:
// the pivots).  Returns false (in every thread) on a pivot that is not
// positive.
template <int D>
__device__ bool cholesky_both(float *X, int tid, float *piv_l, float *piv_r)
{
    constexpr int P = WushLds<D>::kP;
    constexpr int kTy = kWushThreads / D;
    const int tx = tid % D, ty = tid / D;
    auto inverse_root = [](float piv) { return piv > 0.0f ? 1.0f / sqrtf(piv) : 0.0f; };
    bool ok = true;
    for (int j = 0; j < D; ++j) {
        const float ph = X[j * P + j], pm = X[(j + 1) * P + j];
        ok = ok && ph > 0.0f && pm > 0.0f;
        const float ih = inverse_root(ph), im = inverse_root(pm);
        if (tid == 0) {
            piv_l[j] = ph;
            piv_r[j] = pm;
        }
        if (tx > j) {
            // H: row tx of the columns e <= tx; M: entry tx of the rows e >= tx
            const float lh = X[j * P + tx] * ih;
            const float lm = X[(tx + 1) * P + j] * im;
            for (int e = j + 1 + ty; e < D; e += kTy) {
                const float oh = X[j * P + e] * ih;
                const float om = X[(e + 1) * P + j] * im;
                if (e <= tx) X[e * P + tx] -= lh * oh;
                if (e >= tx) X[(e + 1) * P + tx] -= lm * om;
            }
        }
        __syncthreads();
    }
    for (int e = tid; e < D * D; e += kWushThreads) {
        const int c = e / D, r = e % D;  // entry r of column c, and of column c + 1
        if (r > c) X[c * P + r] *= inverse_root(piv_l[c]);
        if (r < c) X[(c + 1) * P + r] *= inverse_root(piv_r[r]);
        if (r == c) {
            X[c * P + r] = sqrtf(piv_l[c]);
            X[(c + 1) * P + r] = sqrtf(piv_r[c]);
        }
    }
    __syncthreads();
    return ok;
}

// Unnormalised Walsh-Hadamard transform (Sylvester order) of every column's
// first D entries: x_r <- sum_r' (-1)^popcount(r & r') x_r'.  Sixteen
// consecutive entries in registers, then the D / 16 entries 16 apart.
template <int D>
__device__ void fwht_columns(float *X, int tid)
{
    constexpr int P = WushLds<D>::kP;
    constexpr int kN = D / 16;
    auto transform = [](auto &v, auto n) {
        constexpr int N = decltype(n)::value;
#pragma unroll
        for (int h = 1; h < N; h <<= 1)
#pragma unroll
            for (int i = 0; i < N; ++i)
                if ((i & h) == 0) {
                    const float a = v[i], b = v[i + h];
                    v[i] = a + b;
                    v[i + h] = a - b;
                }
    };
    for (int e = tid; e < D * kN; e += kWushThreads) {
        f32x4 *c = reinterpret_cast<f32x4 *>(X + (e / kN) * P + 16 * (e % kN));
        float v[16];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * q + i] = c[q][i];
        transform(v, std::integral_constant<int, 16>{});
#pragma unroll
        for (int q = 0; q < 4; ++q) c[q] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    }
    __syncthreads();
    for (int e = tid; e < D * 16; e += kWushThreads) {
        float *c = X + (e / 16) * P + e % 16;
        float v[kN];
#pragma unroll
        for (int i = 0; i < kN; ++i) v[i] = c[16 * i];
        transform(v, std::integral_constant<int, kN>{});
#pragma unroll
        for (int i = 0; i < kN; ++i) c[16 * i] = v[i];
    }
    __syncthreads();
}

// A row of L in the registers of 512/d threads, by tournament position: thread
// t holds positions kQ t + x (lo[x]) and, their partners, d - 1 - (kQ t + x)
// (hi[x]).
template <int D>
struct RowOfL {
    static constexpr int kT = kWushThreads / D;  // threads per row
    static constexpr int kQ = D / 2 / kT;        // pairs per thread
    float lo[kQ], hi[kQ];
    template <int CTRL>
    static __device__ __forceinline__ float lane_dpp(float x)
    {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF,
                                                                      false));
    }
    // the rotations of a round (cs, sn of pair m at rot[m]), then the turn to
    // the next round's positions: position 0 stays, position m takes the
    // column of m + 1 and the last one that of position 1
    __device__ __forceinline__ void rotate_and_turn(const float2 *rot, int t)
    {
        // ascending, each pair's results into the places the pair before it
        // has left: u goes down one place, v up one once its place is read
        float u0 = 0.0f, u1 = 0.0f, carry = 0.0f;
#pragma unroll
        for (int x = 0; x < kQ; x += 2) {
            const f32x4 r = *reinterpret_cast<const f32x4 *>(rot + kQ * t + x);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int m = x + e;
                const float cs = r[2 * e], sn = r[2 * e + 1];
                const float u = fmaf(cs, lo[m], -sn * hi[m]);
                const float v = fmaf(sn, lo[m], cs * hi[m]);
                if (m == 0) u0 = u;
                else if (m == 1) u1 = u;
                else lo[m - 1] = u;
                if (m > 0) hi[m] = carry;
                carry = v;
            }
        }
        const float next = lane_dpp<0x101>(u0);     // of thread t + 1
        const float prev = lane_dpp<0x111>(carry);  // of thread t - 1
        lo[0] = t == 0 ? u0 : u1;
        lo[kQ - 1] = t == kT - 1 ? carry : next;
        hi[0] = t == 0 ? u1 : prev;
    }
};

template <int D>
__global__ void __launch_bounds__(kWushThreads, 4) wush_kernel(const float *m_all, const float *h_all, float gamma,
                                                      float *t_all, float *tinv_all, int32_t *sweeps_out)
{
    constexpr int P = WushLds<D>::kP;
    constexpr int kPairs = D / 2;
    constexpr int kTpp = kWushThreads / kPairs;  // threads per pair: 8 (d 128) or 16 (d 64)
    constexpr int kRows = D / kTpp;              // rows of B per thread
    constexpr float kTol = 4.0f * (D == 128 ? 11.3137085f : 8.0f) * 5.9604645e-8f;
    // the products' register tiles: kTa x kTb outputs a thread
    constexpr int kTa = D * D / (4 * kWushThreads);  // 8 (d 128) or 2 (d 64)
    constexpr int kTb = 4;
    __shared__ __attribute__((aligned(16))) float X[WushLds<D>::kFloats];
    __shared__ __attribute__((aligned(16))) float2 rot[2][kPairs];  // (cs, sn) of a round's pairs
    __shared__ float lam[D], scl[D];
    __shared__ int perm[D];
    __shared__ float red[kWushWaves];
    const int tid = threadIdx.x;
    const int64_t pair = blockIdx.x;
    const float *M = m_all + pair * D * D;
    const float *H = h_all + pair * D * D;
    float *T = t_all + pair * D * D;
    float *Ti = tinv_all != nullptr ? tinv_all + pair * D * D : nullptr;

    // ---- 1. the damped matrices (lower triangles read) and their factors
    const float trH = trace_of<D>(H, tid, red), trM = trace_of<D>(M, tid, red);
    const float dampH = gamma * trH / (float)D, dampM = gamma * trM / (float)D;
    for (int e = tid; e < D * D; e += kWushThreads) {
        const int i = e / D, k = e % D;  // row-major reads, coalesced
        if (i >= k) {
            X[k * P + i] = H[e] + (i == k ? dampH : 0.0f);
            X[(i + 1) * P + k] = M[e] + (i == k ? dampM : 0.0f);
        }
    }
    __syncthreads();  // (every input of the pair has been read)
    if (Ti != nullptr) {
        for (int e = tid; e < D * D; e += kWushThreads) {
            const int i = e / D, k = e % D;
            Ti[e] = i >= k ? X[(i + 1) * P + k] : X[(k + 1) * P + i];  // M_d
        }
        __syncthreads();
    }
    if (!cholesky_both<D>(X, tid, lam, scl)) {
        for (int e = tid; e < D * D; e += kWushThreads) {
            T[e] = NAN;
            if (Ti != nullptr) Ti[e] = NAN;
        }
        if (sweeps_out != nullptr && tid == 0) sweeps_out[pair] = -1;
        return;
    }

    // ---- 2. B = R^T L: B[b][a] = sum_i R[i][b] L[i][a], i >= max(a, b)
    const int ta = (tid % (D / kTa)) * kTa, tb = (tid / (D / kTa)) * kTb;  // the thread's tile
    float acc[kTa][kTb];
    auto clear = [&]() {
#pragma unroll
        for (int x = 0; x < kTa; ++x)
#pragma unroll
            for (int y = 0; y < kTb; ++y) acc[x][y] = 0.0f;
    };
    clear();
    for (int i0 = (ta > tb ? ta : tb) & ~3; i0 < D; i0 += 4) {
        f32x4 l[kTa];
#pragma unroll
        for (int x = 0; x < kTa; ++x) {
            l[x] = *reinterpret_cast<const f32x4 *>(X + (ta + x) * P + i0);
#pragma unroll
            for (int q = 0; q < 4; ++q) l[x][q] = i0 + q >= ta + x ? l[x][q] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            f32x4 r = *reinterpret_cast<const f32x4 *>(X + (i0 + q + 1) * P + tb);
#pragma unroll
            for (int y = 0; y < kTb; ++y) r[y] = tb + y <= i0 + q ? r[y] : 0.0f;
#pragma unroll
            for (int x = 0; x < kTa; ++x)
#pragma unroll
                for (int y = 0; y < kTb; ++y) acc[x][y] = fmaf(r[y], l[x][q], acc[x][y]);
        }
    }
    // the rows of L, before B takes the frame
    RowOfL<D> row;
    const int ri = tid / RowOfL<D>::kT, rt = tid % RowOfL<D>::kT;
#pragma unroll
    for (int x = 0; x < RowOfL<D>::kQ; ++x) {
        const int k = RowOfL<D>::kQ * rt + x, k2 = D - 1 - k;
        row.lo[x] = ri >= k ? X[k * P + ri] : 0.0f;
        row.hi[x] = ri >= k2 ? X[k2 * P + ri] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < kTa; ++x)
        *reinterpret_cast<f32x4 *>(X + (ta + x) * P + tb) = f32x4{acc[x][0], acc[x][1], acc[x][2], acc[x][3]};
    __syncthreads();

    // ---- 3. one-sided Jacobi on the columns of B, and of L
    const int pm = tid / kTpp, part = tid % kTpp;
    int sweeps = 0;
    for (; sweeps < kWushMaxSweeps; ++sweeps) {
        int rotated = 0;
        for (int round = 0; round < D - 1; ++round) {
            // round-robin: position 0 stays, positions 1 .. D-1 turn by one
            // per round; pair m meets positions m and D - 1 - m
            auto at = [&](int pos) {
                const int x = pos - 1 + round;  // (below 2 (D - 1))
                return pos == 0 ? 0 : 1 + (x >= D - 1 ? x - (D - 1) : x);
            };
            const int p = at(pm), q = at(D - 1 - pm);
            // this thread's rows of the two columns stay in registers from
            // the dot products to the rotation: the 4-row pieces
            // 4 (kTpp k + part) .. + 3, one 16-byte access each
            float *cp = X + p * P + 4 * part, *cq = X + q * P + 4 * part;
            f32x4 xb[kRows / 4], yb[kRows / 4];
            float al = 0.0f, be = 0.0f, ga = 0.0f;
#pragma unroll
            for (int k = 0; k < kRows / 4; ++k) {
                xb[k] = *reinterpret_cast<const f32x4 *>(cp + 4 * kTpp * k);
                yb[k] = *reinterpret_cast<const f32x4 *>(cq + 4 * kTpp * k);
            }
#pragma unroll
            for (int k = 0; k < kRows / 4; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    al = fmaf(xb[k][i], xb[k][i], al);
                    be = fmaf(yb[k][i], yb[k][i], be);
                    ga = fmaf(xb[k][i], yb[k][i], ga);
                }
            al = group_sum<kTpp>(al);
            be = group_sum<kTpp>(be);
            ga = group_sum<kTpp>(ga);
            // rotate while the columns' cosine exceeds what rounding leaves
            // behind (a few units of 2^-24 sqrt(d))
            float cs = 1.0f, sn = 0.0f;
            if (fabsf(ga) > kTol * sqrtf(al * be) && ga != 0.0f) {
                const float zeta = (be - al) / (2.0f * ga);
                const float t = copysignf(1.0f, zeta) / (fabsf(zeta) + sqrtf(1.0f + zeta * zeta));
                cs = 1.0f / sqrtf(1.0f + t * t);
                sn = cs * t;
#pragma unroll
                for (int k = 0; k < kRows / 4; ++k) {
                    f32x4 u, v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        u[i] = fmaf(cs, xb[k][i], -sn * yb[k][i]);
                        v[i] = fmaf(sn, xb[k][i], cs * yb[k][i]);
                    }
                    *reinterpret_cast<f32x4 *>(cp + 4 * kTpp * k) = u;
                    *reinterpret_cast<f32x4 *>(cq + 4 * kTpp * k) = v;
                }
                rotated = 1;
            }
            if (part == 0) rot[round & 1][pm] = make_float2(cs, sn);
            __syncthreads();
            row.rotate_and_turn(rot[round & 1], rt);
        }
        // (as many rounds as turns bring every column back: position m holds
        // column m)
        if (!__syncthreads_or(rotated)) break;
    }

    // ---- 4. eigenvalues, their order, the eigenvector signs, c
    for (int k = tid; k < D; k += kWushThreads) {
        const float *ck = X + k * P;
        float s = 0.0f;
        for (int i = 0; i < D; ++i) s = fmaf(ck[i], ck[i], s);
        lam[k] = s;
    }
    // (every slot of perm holds a valid column even if non-finite norms
    // left ranks tied)
    for (int r = tid; r < D; r += kWushThreads) perm[r] = r;
    __syncthreads();
    // the frame now holds L U: entry i of column k at X[k P + i]
#pragma unroll
    for (int x = 0; x < RowOfL<D>::kQ; ++x) {
        const int k = RowOfL<D>::kQ * rt + x;
        X[k * P + ri] = row.lo[x];
        X[(D - 1 - k) * P + ri] = row.hi[x];
    }
    for (int k = tid; k < D; k += kWushThreads) {
        int rank = 0;
        const float lk = lam[k];
        for (int j = 0; j < D; ++j) rank += (lam[j] < lk) || (lam[j] == lk && j < k);
        perm[rank] = k;
    }
    float rs = 0.0f;
    for (int k = tid; k < D; k += kWushThreads) rs += sqrtf(lam[k]);
    rs = group_sum<64>(rs);
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = rs;
    // sign of u_k: the largest-magnitude entry of L u_k (the first of equal
    // ones) made positive
    for (int k = tid / 16; k < D; k += kWushThreads / 16) {
        float best = -1.0f;
        int at = 0;
        for (int i = tid % 16; i < D; i += 16) {
            const float a = fabsf(X[k * P + i]);
            if (a > best) {
                best = a;
                at = i;
            }
        }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const float ob = __shfl_xor(best, off);
            const int oa = __shfl_xor(at, off);
            if (ob > best || (ob == best && oa < at)) {
                best = ob;
                at = oa;
            }
        }
        if (tid % 16 == 0) scl[k] = X[k * P + at] < 0.0f ? -1.0f : 1.0f;
    }
    __syncthreads();
    const float sum_sqrt = wave_total(red);
    const float c = sqrtf((1.0f + gamma) * trM) / sqrtf(sum_sqrt);
    const float had = 1.0f / sqrtf((float)D);

    // ---- 5b, its product: Z = M_d (L U), columns in order and scaled, held
    // in registers while T goes through the frame
    if (Ti != nullptr) {
        clear();
        int kr[kTb];
#pragma unroll
        for (int y = 0; y < kTb; ++y) kr[y] = perm[tb + y];
        for (int j0 = 0; j0 < D; j0 += 4) {
            f32x4 w[kTb];
#pragma unroll
            for (int y = 0; y < kTb; ++y) w[y] = *reinterpret_cast<const f32x4 *>(X + kr[y] * P + j0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float mv[kTa];  // M_d[i][j], symmetric
#pragma unroll
                for (int x = 0; x < kTa; ++x) mv[x] = Ti[(j0 + q) * D + ta + x];
#pragma unroll
                for (int x = 0; x < kTa; ++x)
#pragma unroll
                    for (int y = 0; y < kTb; ++y) acc[x][y] = fmaf(mv[x], w[y][q], acc[x][y]);
            }
        }
#pragma unroll
        for (int y = 0; y < kTb; ++y) {
            const float s = scl[kr[y]] * powf(lam[kr[y]], -0.75f) / c;
#pragma unroll
            for (int x = 0; x < kTa; ++x) acc[x][y] *= s;
        }
    }

    // ---- 5a. T: column j of the frame gets y_r[j] = s_k lam_k^(-1/4)
    // (L u_k)[j], k = perm[r]; the transform along r gives row r of Had Y
    {
        constexpr int kPer = D * D / kWushThreads;
        const int r = tid % D, k = perm[r];
        const float s = scl[k] * powf(lam[k], -0.25f);
        float y[kPer];
#pragma unroll
        for (int n = 0; n < kPer; ++n) y[n] = s * X[k * P + tid / D + (kWushThreads / D) * n];
        __syncthreads();
#pragma unroll
        for (int n = 0; n < kPer; ++n) X[(tid / D + (kWushThreads / D) * n) * P + r] = y[n];
        __syncthreads();
    }
    fwht_columns<D>(X, tid);
    for (int e = tid; e < D * D; e += kWushThreads) {
        const int i = e / D, j = e % D;  // row-major write, coalesced
        T[e] = (c * had) * X[j * P + i];
    }
    if (sweeps_out != nullptr && tid == 0) sweeps_out[pair] = sweeps;
    if (Ti == nullptr) return;
    __syncthreads();

    // ---- 5b. T^{-1} = c^-1 M_d (L U) Lam^(-3/4) Had: row i of Z into column
    // i of the frame, then the transform along each row
#pragma unroll
    for (int x = 0; x < kTa; ++x)
#pragma unroll
        for (int y = 0; y < kTb; ++y) X[(ta + x) * P + tb + y] = acc[x][y];  // Z[i][r]
    __syncthreads();
    fwht_columns<D>(X, tid);
    for (int e = tid; e < D * D; e += kWushThreads) {
        const int i = e / D, r = e % D;
        Ti[e] = had * X[i * P + r];
    }
}

}  // namespace wushkv

using namespace wushkv;

extern "C" int wushkv_wush_transform(const float *m, const float *h, int32_t count, int32_t d,
                                     float gamma, float *t_out, float *t_inv_out,
                                     int32_t *sweeps_out, wushkv_stream_t stream)
{
    if (count < 0 || !(gamma >= 0.0f) || gamma == INFINITY) return WUSHKV_EINVAL;
    if (d != 64 && d != 128) return WUSHKV_EUNSUPPORTED;
    if (count == 0) return WUSHKV_OK;
    if (!m || !h || !t_out) return WUSHKV_EINVAL;
    if (((uintptr_t)m | (uintptr_t)h | (uintptr_t)t_out | (uintptr_t)t_inv_out |
         (uintptr_t)sweeps_out) & 15u)
        return WUSHKV_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const dim3 grid((unsigned)count);
    if (d == 128)
        launch("wush_kernel", wush_kernel<128>, grid, dim3(kWushThreads), s, m, h, gamma, t_out, t_inv_out, sweeps_out);
    else
        launch("wush_kernel", wush_kernel<64>, grid, dim3(kWushThreads), s, m, h, gamma, t_out, t_inv_out, sweeps_out);
    if (hipGetLastError() != hipSuccess) return WUSHKV_ELAUNCH;
    return WUSHKV_OK;
}
