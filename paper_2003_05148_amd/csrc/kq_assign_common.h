// Device code shared by the two assignment kernels (kq_assign.hip: every codebook of at most
// 1024 entries; kq_assign_large.hip: any codebook).
#pragma once

#include "kq_internal.h"

namespace kq {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowFloats = 12;      // fp32 codebook rows in LDS: 9 values, padded to 48 bytes
constexpr float kTrustQ = 1e37f;    // Q' at or above this: rescored over the whole codebook
constexpr float kMaxFloat = 3.402823466e38f;

__device__ __forceinline__ float sqdist9(const float* x, const float* c) {
    float acc = 0.0f;
#pragma unroll
    for (int d = 0; d < kDim; ++d) {
        const float t = x[d] - c[d];
        acc = __fmaf_rn(t, t, acc);
    }
    return acc;
}

__device__ __forceinline__ float min2(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, -3.402823466e38f); }
// the smallest of three finite values (v_min3_f32 without the compiler's NaN canonicalisation:
// the operands are never NaN)
__device__ __forceinline__ float min3f(float a, float b, float c) {
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// slot minima: one v_min3 per two scores; the first pair of a segment starts them, capped at
// the largest finite float so that packing keeps a number
template <bool FIRST>
__device__ __forceinline__ void fold_pair(float (&best)[16], const f32x16 (&acc)[2]) {
#pragma unroll
    for (int q = 0; q < 16; ++q)
        best[q] = __builtin_fminf(__builtin_fminf(acc[0][q], acc[1][q]), FIRST ? kMaxFloat : best[q]);
}

// (d, j) becomes the lexicographic minimum of the pair and its partner's (o_d, o_j); a
// partner holding the same pair leaves it unchanged, so both lanes end with the same pair
__device__ __forceinline__ void argmin_take(float& d, int& j, float od, int oj) {
    const bool take = od < d || (od == d && oj < j);
    d = take ? od : d;
    j = take ? oj : j;
}
template <int CTL>
__device__ __forceinline__ void argmin_dpp(float& d, int& j) {
    const float od = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(d), CTL, 0xF, 0xF, true));
    const int oj = __builtin_amdgcn_mov_dpp(j, CTL, 0xF, 0xF, true);
    argmin_take(d, j, od, oj);
}
// the wave's lexicographic minimum of the lanes' (distance, index) pairs, in every lane:
// partners 32 and 16 lanes away by the half and row swaps, then DPP moves inside a row
// (the rotation by four meets a lane that holds the same pair as the lane 4 away)
__device__ __forceinline__ void wave_argmin(float& d, int& j) {
    {
        const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(d), __float_as_uint(d), false, false);
        const auto b = __builtin_amdgcn_permlane32_swap((unsigned)j, (unsigned)j, false, false);
        d = __uint_as_float(a[0]);
        j = (int)b[0];
        argmin_take(d, j, __uint_as_float(a[1]), (int)b[1]);
    }
    {
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(d), __float_as_uint(d), false, false);
        const auto b = __builtin_amdgcn_permlane16_swap((unsigned)j, (unsigned)j, false, false);
        d = __uint_as_float(a[0]);
        j = (int)b[0];
        argmin_take(d, j, __uint_as_float(a[1]), (int)b[1]);
    }
    argmin_dpp<0x128>(d, j);  // row_ror:8
    argmin_dpp<0x124>(d, j);  // row_ror:4
    argmin_dpp<0x4E>(d, j);   // quad_perm [2,3,0,1]
    argmin_dpp<0xB1>(d, j);   // quad_perm [1,0,3,2]
}

// this lane's kernel of unit u of the layer (kernel 64 u + lane); a valid row past the end
__device__ __forceinline__ void load_kernel(const DevLayer& L, int u, int lane, float (&x)[kDim]) {
    const int i = u * kWave + lane;
    const int ic = i < L.n ? i : L.n - 1;
#pragma unroll
    for (int d = 0; d < kDim; ++d) x[d] = L.X[(size_t)ic * kDim + d];
}

// one codebook row: from its 48-byte LDS copy, or from memory (36 bytes, 4-byte aligned)
__device__ __forceinline__ void lds_row(float (&c)[kDim], const f32x4* s_c, int j) {
    const f32x4 r0 = s_c[j * 3 + 0], r1 = s_c[j * 3 + 1];
    const float c8 = reinterpret_cast<const float*>(s_c)[j * kRowFloats + 8];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        c[d] = r0[d];
        c[4 + d] = r1[d];
    }
    c[8] = c8;
}
__device__ __forceinline__ void mem_row(float (&c)[kDim], const float* __restrict__ C, int j) {
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    const float* const r = C + (size_t)j * kDim;
    const f32x4u r0 = *reinterpret_cast<const f32x4u*>(r), r1 = *reinterpret_cast<const f32x4u*>(r + 4);
    const float c8 = r[8];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        c[d] = r0[d];
        c[4 + d] = r1[d];
    }
    c[8] = c8;
}

// One workgroup's run: a share of one layer's units (the layer's workgroups split them evenly).
// The table of first workgroups is read once, and the layer's fields in one batch after it:
// every dependent load of the arguments is a memory round trip before any work.
struct AssignRun {
    int layer;   // the layer
    int wg;      // this workgroup among the layer's
    int ub, ue;  // units [ub, ue)
};
__device__ __forceinline__ AssignRun assign_run(const StackParams& p, int& n, int& k, const float*& C) {
    int lb = 0, g0 = 0, g1 = (int)gridDim.x;
#pragma unroll
    for (int l = 1; l < KQ_MAX_STACK; ++l) lb += (int)blockIdx.x >= p.wg_begin[l] ? 1 : 0;
#pragma unroll
    for (int l = 0; l < KQ_MAX_STACK; ++l) {  // past the last layer the table holds 0x7fffffff
        g0 = l == lb ? p.wg_begin[l] : g0;
        g1 = l == lb + 1 ? min(p.wg_begin[l], (int)gridDim.x) : g1;
    }
    const int gl = g1 - g0;
    const DevLayer& L = p.L[lb];
    n = L.n;
    k = L.k;
    C = L.C;
    const int U = L.nunits, j = (int)blockIdx.x - g0, nxmax = L.nxmax, derive = p.derive_shift;
    const float* const Xl = L.X;
    const unsigned* const xmax = L.xmax;
    asm volatile("" ::"s"(n), "s"(k), "s"(U), "s"(C), "s"(Xl), "s"(xmax), "s"(nxmax), "s"(derive));
    const int q = U / gl, r = U - q * gl;  // workgroup j: q units, one more for the first r
    AssignRun run;
    run.layer = lb;
    run.wg = j;
    run.ub = j * q + min(j, r);
    run.ue = run.ub + q + (j < r ? 1 : 0);
    return run;
}

// exact fp32 rescoring of N kernels (xf, the same in every lane) over a whole codebook: each
// lane scans entries lane, lane + 64, ... in increasing order (strict <: the lowest index among
// equal distances), kU rows in flight, then the lanes' (distance, index) pairs meet in their
// lexicographic minimum
template <int N, typename Row>
__device__ __forceinline__ void scan_all(const float (&xf)[N][kDim], int k, int lane, float (&fd)[N], int (&fj)[N], Row&& row) {
    constexpr int kU = 4;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        fd[e] = __builtin_inff();
        fj[e] = 0x7fffffff;
    }
    for (int j0 = lane; j0 < k; j0 += kU * kWave) {
        float c[kU][kDim];
#pragma unroll
        for (int u = 0; u < kU; ++u) row(c[u], min(j0 + u * kWave, k - 1));  // a valid row past the end
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int jj = j0 + u * kWave;
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const float d = sqdist9(xf[e], c[u]);
                const bool take = jj < k && d < fd[e];
                fj[e] = take ? jj : fj[e];
                fd[e] = take ? d : fd[e];
            }
        }
    }
#pragma unroll
    for (int e = 0; e < N; ++e) wave_argmin(fd[e], fj[e]);
}

// The lanes of fl (their kernels x) rescored over the whole codebook, kMany at a time (the rows are read
// once for them) while there are that many, then one by one; done(lane's distance, index) in each of them.
// Where the screening cannot tell near ties apart (kernels of few dimensions, around a common offset, copies
// of one entry), most kernels come here.  131,072 kernels, k = 4096, one by one and by four: of rank 2 610
// and 283 us, around ten times their deviation 858 and 346, half of them zero with as many zero entries 542
// and 247; none such 64 both.
constexpr int kMany = 4;
template <typename Row, typename Done>
__device__ __forceinline__ void rescan(unsigned long long fl, const float (&x)[kDim], int k, int lane, Row&& row, Done&& done) {
    auto some = [&](auto count) {
        constexpr int N = decltype(count)::value;
        int f[N];
        float xf[N][kDim], fd[N];  // lane f's kernel, the same in every lane (f is uniform)
        int fj[N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
            f[e] = __ffsll((long long)fl) - 1;
            fl &= fl - 1;
#pragma unroll
            for (int d = 0; d < kDim; ++d) xf[e][d] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[d]), f[e]));
        }
        scan_all<N>(xf, k, lane, fd, fj, row);
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (lane == f[e]) done(fd[e], fj[e] == 0x7fffffff ? 0 : fj[e]);  // every distance NaN or +inf: entry 0
    };
    while (__popcll(fl) >= kMany) some(std::integral_constant<int, kMany>{});
    while (fl) some(std::integral_constant<int, 1>{});
}

}  // namespace kq
