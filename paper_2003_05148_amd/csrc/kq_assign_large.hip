// Assignment against codebooks of any size (Sec. 3.1, Eq. 1), used whenever a launch holds a
// codebook of more than 1024 entries (kAssignMaxK).  The result is the one of kq_assign.hip, bit
// for bit: the argmin of the fp32 squared distances, ties to the lowest index.
//
// The screening takes one fp16 product, K = 16, instead of the three bf16 cross terms, K = 32, of the
// small-codebook kernel, keeps the three best groups instead of two, and rescores a second group
// where one is not enough.  The product loop alone, with folding and real operands: 187 ns per pair of
// 32-entry tiles, 64 kernels and SIMD with K = 32, 112 ns with K = 16.
//
// What bounds it: the issue of vector instructions (folding the scores, the three best, the fp32
// rescoring).  By counters, on the VGG-16 stack with k = 60 .. 1088 (79 us a launch), the ResNet-18 stack
// with k = 609 .. 7679 (315 us) and 1,048,576 kernels at k = 4096 (248 us): VALU busy 88, 75 and 79 % of a
// SIMD's cycles, MFMA 18, 32 and 29 %, two thirds of these with a VALU instruction issued at the same
// time; the address units 17, 32 and 50 % (the gathered rows of codebooks above 1920 entries).  The clock
// is 1.8 to 2.0 GHz under this load.
//
// Screening.  Scaled by powers of two, ys = x 2^b and cs = c 2^a with max |c_jd| 2^a in [2^12,
// 2^13) over the codebook but its far entries (kFarExp; they are scored as padding) and b = a, or less
// where max |x_d| exceeds max |c_jd| (then |ys_d| < 2^13 too), the score s_j = |c_j|^2 - 2 x . c_j
// becomes, times 2^(a+b),
//     sum_{d < 9} w_jd ys_d + n_j u,   w_j = -2 cs_j,  n_j = |cs_j|^2 2^-14,  u = 2^(14 + b - a).
// w and ys are rounded to fp16, n_j u is split into three products n_h u + n_m 2^-11 u + n_l 2^-22 u of
// fp16 values (n_h = fp16(n_j), n_m = fp16(2^11 (n_j - n_h)), and so on): 12 of the 16 terms of one
// v_mfma_f32_32x32x16_f16 per 32 x 32 tile of (entries, kernels), products exact, sums in fp32.
// In the D layout a lane holds one kernel (column) and 16 of its 32 rows.  A segment is
// 256 or 512 entries (8 or 16 tiles); a group is the 8 or 16 entries of one row ("slot") of it.  Each lane keeps
// the minimum score of each slot over the segment, one v_min3 per two scores; then the three
// smallest are found by a tournament and merged into the kernel's summary: the three smallest
// group minima over all segments so far, and the groups of the first two.
//
// Exactness.  Let u0 = 2^-24, P_j = 2 |x| |c_j| + |c_j|^2 <= (|x| + |c_j|)^2, A = 2^-14 2^-a and
// B = 2^-14 2^-b (the smallest normal fp16 in units of c and of x: a value below it may be lost
// whole).  In units of s_j a screened score is off by at most
//     (2^-10 + 2^-22) 2 |x| |c_j|  (both roundings to fp16, 2^-11 each)
//   + 1.01 (6 B |c_j| + 3 A |x|) + 2^(-22 - 2a)  (fp16 values that may be flushed: the last below 2^-14
//     in n_l; where b is so far below a that a u flushes, |c_j|^2 is below 2^-29 |x|^2)
//   + 104 u0 P_j  (33: the sums of 13 terms, truncated or rounded; 9: the fp32 norm; 62: the slot
//     number in the 5 lowest mantissa bits of a slot minimum).
// The first group is rescored in the plain fp32 form; d* is its smallest distance, at the lowest
// index; M2 is the smallest minimum of all other groups.  With r = |x| + (1 + 2^-9) sqrt(d*) +
// 2^-61, an entry outside the group either has |c_j| > r, and then lies farther than (1 + 2^-9)
// sqrt(d*), so that its fp32 distance (relative error <= 12 u0) exceeds d*; or its bound holds
// with r for |c_j|, and its fp32 distance exceeds d* once M2 + |x|^2 - d* is larger than the bound
// plus 18 u0 (|x| + r)^2 (the fp32 |x|^2, the distance's rounding and the guard's own).  The guard
// asks for more than
//     theta = 1.05 (2^-9 |x| r' + 2^-17 (|x| + r')^2 + 6 B r' + 3 A |x| + 2^(-21 - 2a)) + 2^-100,
// r' = |x| + 1.01 sqrt(d*) + 2^-60, and for r' below the length of every far entry (an entry that is not
// finite never wins).  Where it fails (1 to 7 % of the kernels), the second group is
// rescored too, d* is the smaller distance of both, and the guard is asked of M3, the smallest
// minimum of all groups but these two.  Where that fails too (about one kernel in a thousand),
// and wherever (|x| + r')^2 >= 1e37 or a value is not finite, the kernel is rescored over the
// whole codebook.  Padding entries only lower a minimum: they cost a rescan, never a result.
#include <hip/hip_ext.h>

#include "kq_assign_common.h"

namespace kq {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kSegMax = 512;                 // entries of the longer segments
constexpr int kOperandLds = 32;              // bytes of operands per staged entry
constexpr int kEntryLds = kOperandLds + 4 * kRowFloats;
// One workgroup per CU.  Codebooks of up to kRowsMaxK entries are staged whole with their fp32
// rows, of up to kResidentMaxK without (their rows are gathered from memory); larger ones stream
// through LDS in chunks of whole segments.
constexpr int kLargeLds = 152 * 1024;
constexpr int kResidentMaxK = kLargeLds / kOperandLds / 64 * 64;        // 4864
constexpr int kRowsMaxK = kLargeLds / kEntryLds / 64 * 64;              // 1920
constexpr int kStreamChunk = kLargeLds / kOperandLds / kSegMax * kSegMax;  // 4608
constexpr int kShortSegK = 2048;  // segments of 256 entries for launches up to this codebook size
// entries more than 2^kFarExp above the middle of the waves' largest exponents are far: they keep the
// scale from the others, and no kernel nearer to zero than they are takes them
constexpr int kFarExp = 12;
// scaled: |cs_jd| < 2^13 gives |cs_j|^2 < 6.04e8; below kNearNorm an entry's operands are finite fp16 values
constexpr float kNearNorm = 7e8f, kFarLength = 26457.0f;  // kFarLength^2 < kNearNorm
constexpr int kStreamUnits = 8;  // units whose summaries a wave keeps while a codebook streams

__device__ __forceinline__ float max2(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, __builtin_inff()); }
__device__ __forceinline__ float max3f(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float absmax3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ unsigned pack16(float a, float b) {  // (a, b) rounded to fp16, a in the low half
    const f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, f16x2));
}
// 2^(12 - e) and 2^(e - 12) for the biased exponent E = e + 127, 13 <= E <= 254
__device__ __forceinline__ float scale_of(int E) { return __uint_as_float((unsigned)(266 - E) << 23); }
__device__ __forceinline__ float inverse_of(int E) { return __uint_as_float((unsigned)(E - 12) << 23); }

// a value of at least the smallest normal fp16 in magnitude, rounded to fp16; a smaller one is zero
__device__ __forceinline__ float half_of(float v) { return fabsf(v) < 0x1p-14f ? 0.0f : (float)(_Float16)v; }

// entries [c0, c0 + cn) into LDS: fp16 operands [w_0 .. w_8, n_h, n_m, n_l, 0 ..] at s_a, in the
// A layout [tile][lane][8 x fp16], and (ROWS) the fp32 rows at s_c; entries past the codebook and far
// ones are padding, with a score above any trusted one
template <bool ROWS>
__device__ __forceinline__ void stage16(const float* __restrict__ C, int k, int c0, int cn, float sc, u32x4* s_a,
                                        f32x4* s_c, int tid, const float* own = nullptr) {
    for (int jl = tid; jl < cn; jl += kAssignWaves * kWave) {
        const int j = c0 + jl;
        float c[kDim], w[kDim], n0, n1, n2, nn = __builtin_inff();
        if (j < k) {
#pragma unroll
            for (int d = 0; d < kDim; ++d) c[d] = (own && jl == tid) ? own[d] : C[(size_t)j * kDim + d];
            nn = 0.0f;
#pragma unroll
            for (int d = 0; d < kDim; ++d) {
                const float s = c[d] * sc;
                nn = __fmaf_rn(s, s, nn);
                w[d] = -2.0f * s;
            }
        } else {
#pragma unroll
            for (int d = 0; d < kDim; ++d) c[d] = __builtin_inff();
        }
        if (nn < kNearNorm) {  // (not a NaN's)
            nn *= 0x1p-14f;
            n0 = half_of(nn);
            const float t1 = (nn - n0) * 0x1p11f;  // exact
            n1 = half_of(t1);
            n2 = half_of((t1 - n1) * 0x1p11f);
        } else {
#pragma unroll
            for (int d = 0; d < kDim; ++d) w[d] = 0.0f;
            n0 = n1 = n2 = 65504.0f;
        }
        const u32x4 lo = {pack16(w[0], w[1]), pack16(w[2], w[3]), pack16(w[4], w[5]), pack16(w[6], w[7])};
        const u32x4 hi = {pack16(w[8], n0), pack16(n1, n2), 0u, 0u};
        const int at = (jl >> 5) * kWave + (jl & 31);
        s_a[at] = lo;
        s_a[at + 32] = hi;
        if (ROWS) {
            const f32x4 r0 = {c[0], c[1], c[2], c[3]}, r1 = {c[4], c[5], c[6], c[7]}, r2 = {c[8], 0.f, 0.f, 0.f};
            s_c[jl * 3 + 0] = r0;
            s_c[jl * 3 + 1] = r1;
            s_c[jl * 3 + 2] = r2;
        }
    }
}

// B operands of a unit's two kernel tiles (the kernels of lanes 0..31 and 32..63): lane (col,
// half) holds terms 8 half .. + 7 of the column's kernel
__device__ __forceinline__ void make_b16(u32x4 (&bop)[2], const float (&x)[kDim], float sx, float u) {
    const unsigned D[4] = {pack16(x[0] * sx, x[1] * sx), pack16(x[2] * sx, x[3] * sx), pack16(x[4] * sx, x[5] * sx),
                           pack16(x[6] * sx, x[7] * sx)};
    const unsigned E[4] = {pack16(x[8] * sx, u), pack16(u * 0x1p-11f, u * 0x1p-22f), 0u, 0u};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const auto sw = __builtin_amdgcn_permlane32_swap(D[e], E[e], false, false);
        bop[0][e] = sw[0];
        bop[1][e] = sw[1];
    }
}

// scores of codebook tiles 2p and 2p + 1 (A operands a) against one kernel tile (B operand b)
__device__ __forceinline__ void score16(f32x16 (&acc)[2], const u32x4 (&a)[2], const u32x4& b) {
    const f32x16 zero = {0.0f};
#pragma unroll
    for (int u = 0; u < 2; ++u)
        acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a[u]),
                                                        __builtin_bit_cast(f16x8, b), zero, 0, 0, 0);
}
__device__ __forceinline__ void lds_a16(u32x4 (&a)[2], const u32x4* s_a, int p, int lane) {
    a[0] = s_a[2 * p * kWave + lane];
    a[1] = s_a[(2 * p + 1) * kWave + lane];
}

// One pair of codebook tiles against both kernel tiles, software-pipelined: p holds tile 0's
// scores against this pair, a the pair's operands.  Tile 1's MFMAs run while tile 0's scores are
// folded, the next pair's tile-0 MFMAs (when there is a next pair) while tile 1's are: MFMA and
// VALU work overlap where they are independent.
template <bool FIRST, bool MORE>
__device__ __forceinline__ void scan_pair16(float (&best)[2][16], f32x16 (&p)[2], u32x4 (&a)[2], const u32x4 (&bop)[2],
                                            const u32x4* s_a, int t, int lane) {
    f32x16 q[2];
    score16(q, a, bop[1]);
    if (MORE) lds_a16(a, s_a, t + 1, lane);  // (the operands just used are free)
    fold_pair<FIRST>(best[0], p);
    if (MORE) score16(p, a, bop[0]);
    fold_pair<FIRST>(best[1], q);
}

// the three smallest of two ascending triples, ascending: the i-th is the least of max(a_s, b_t)
// over s + t = i (a_0 = b_0 = -inf)
__device__ __forceinline__ void merge3(float& a1, float& a2, float& a3, float b1, float b2, float b3) {
    const float m1 = min2(a1, b1);
    const float m2 = min3f(max2(a1, b1), a2, b2);
    a3 = min2(min3f(a3, b3, max2(a2, b1)), max2(a1, b2));
    a1 = m1;
    a2 = m2;
}

// The three smallest slot minima of this lane's kernel, ascending; the 5 low mantissa bits hold
// q + 16 half of the slot, row 8 (q / 4) + 4 half + q % 4 of its tiles.
__device__ __forceinline__ void top3_slots(const float (&best)[2][16], float& s1, float& s2, float& s3, unsigned hb) {
    float m[2][3];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        float pq[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) pq[q] = __uint_as_float((__float_as_uint(best[r][q]) & ~31u) | (unsigned)q);
        float t[5][3];
#pragma unroll
        for (int e = 0; e < 5; ++e) {
            t[e][0] = min3f(pq[3 * e], pq[3 * e + 1], pq[3 * e + 2]);
            t[e][1] = __builtin_amdgcn_fmed3f(pq[3 * e], pq[3 * e + 1], pq[3 * e + 2]);
            t[e][2] = max3f(pq[3 * e], pq[3 * e + 1], pq[3 * e + 2]);
        }
        merge3(t[0][0], t[0][1], t[0][2], t[1][0], t[1][1], t[1][2]);
        merge3(t[2][0], t[2][1], t[2][2], t[3][0], t[3][1], t[3][2]);
        {  // one more value into a triple
            float& a1 = t[4][0];
            float& a2 = t[4][1];
            float& a3 = t[4][2];
            a3 = __builtin_amdgcn_fmed3f(a2, a3, pq[15]);
            a2 = __builtin_amdgcn_fmed3f(a1, a2, pq[15]);
            a1 = min2(a1, pq[15]);
        }
        merge3(t[0][0], t[0][1], t[0][2], t[2][0], t[2][1], t[2][2]);
        merge3(t[0][0], t[0][1], t[0][2], t[4][0], t[4][1], t[4][2]);
#pragma unroll
        for (int e = 0; e < 3; ++e) m[r][e] = __uint_as_float(__float_as_uint(t[0][e]) | hb);
    }
    // own kernel: lanes < 32 tile 0, lanes >= 32 tile 1; first from the lower half's rows
    float lo[3], hi[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(m[0][e]), __float_as_uint(m[1][e]), false, false);
        lo[e] = __uint_as_float(x[0]);
        hi[e] = __uint_as_float(x[1]);
    }
    merge3(lo[0], lo[1], lo[2], hi[0], hi[1], hi[2]);
    s1 = lo[0];
    s2 = lo[1];
    s3 = lo[2];
}

// A kernel's summary: the three smallest group minima (their slots in the low mantissa bits) and
// the segments of the first two (g1 | g2 << 16)
struct Screen3 {
    float m1, m2, m3;
    unsigned seg;
};
__device__ __forceinline__ Screen3 screen_start() { return Screen3{kMaxFloat, kMaxFloat, kMaxFloat, 0u}; }

// the summary s with another one of other segments (a segment's: its three smallest, g1 = g2)
__device__ __forceinline__ void merge_screen(Screen3& s, float o1, float o2, float o3, unsigned og1, unsigned og2) {
    const bool c1 = o1 < s.m1, c2 = o2 < s.m1, c3 = o1 < s.m2;
    const unsigned g1 = s.seg & 0xffffu, g2 = s.seg >> 16;
    // the second: after a new first, the old first or the other's second; else the old second or
    // the other's first
    const unsigned h2 = c1 ? (c2 ? og2 : g1) : (c3 ? og1 : g2);
    s.seg = (c1 ? og1 : g1) | (h2 << 16);
    merge3(s.m1, s.m2, s.m3, o1, o2, o3);
}

// the staged segments from segment g0 on (npair pairs of tiles, kSegPairs to a segment) screened
// against a unit's kernels
template <int kSegPairs>
__device__ __forceinline__ void scan16(Screen3& s, const u32x4 (&bop)[2], const u32x4* s_a, int g0, int npair, int lane) {
    asm volatile("" : "+v"(lane));  // the operands are read here, not kept from one unit to the next
    const unsigned hb = lane >= 32 ? 16u : 0u;
    float best[2][16], s1, s2, s3;
    int t = 0;
    if (kSegPairs <= npair) {  // segments of full length
        u32x4 a[2];
        lds_a16(a, s_a, 0, lane);
        f32x16 p[2];
        score16(p, a, bop[0]);
#pragma unroll 1
        for (; t + 2 * kSegPairs <= npair; t += kSegPairs) {  // with another one after it
            scan_pair16<true, true>(best, p, a, bop, s_a, t, lane);
#pragma unroll
            for (int u = 1; u < kSegPairs; ++u) scan_pair16<false, true>(best, p, a, bop, s_a, t + u, lane);
            top3_slots(best, s1, s2, s3, hb);
            merge_screen(s, s1, s2, s3, g0 + t / kSegPairs, g0 + t / kSegPairs);
        }
        scan_pair16<true, true>(best, p, a, bop, s_a, t, lane);
#pragma unroll
        for (int u = 1; u + 1 < kSegPairs; ++u) scan_pair16<false, true>(best, p, a, bop, s_a, t + u, lane);
        scan_pair16<false, false>(best, p, a, bop, s_a, t + kSegPairs - 1, lane);
        top3_slots(best, s1, s2, s3, hb);
        merge_screen(s, s1, s2, s3, g0 + t / kSegPairs, g0 + t / kSegPairs);
        t += kSegPairs;
    }
    if (t < npair) {  // a last, shorter one
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int q = 0; q < 16; ++q) best[r][q] = kMaxFloat;
#pragma unroll 1
        for (int v = t; v < npair; ++v) {
            u32x4 a[2];
            lds_a16(a, s_a, v, lane);
            f32x16 p[2], q[2];
            score16(p, a, bop[0]);
            score16(q, a, bop[1]);
            fold_pair<false>(best[0], p);
            fold_pair<false>(best[1], q);
        }
        top3_slots(best, s1, s2, s3, hb);
        merge_screen(s, s1, s2, s3, g0 + t / kSegPairs, g0 + t / kSegPairs);
    }
}

template <int kSegPairs>
__global__ __launch_bounds__(kAssignWaves * kWave, 1) void assign_large_kernel(const StackParams p) {
    constexpr int kSegTiles = 2 * kSegPairs;  // entries of a group
    constexpr int kSeg = 64 * kSegPairs;      // entries of a segment
    static_assert(kSegMax % kSeg == 0, "chunks hold whole segments");
    // operands of the staged entries, then (codebooks of at most kRowsMaxK entries) their fp32 rows
    __shared__ u32x4 s_a[kLargeLds / 16];
    __shared__ int s_next;       // the next unit to hand out
    __shared__ int s_max[kAssignWaves];  // the largest exponent of each wave's entries

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    int n, k;
    const float* C0;
    const AssignRun run = assign_run(p, n, k, C0);
    const float* __restrict__ C = C0;
    const DevLayer& L = p.L[run.layer];
    const int ub = run.ub, u_end = run.ue;
    if (ub >= u_end) return;

    const int kpad = (k + 63) & ~63;
    const bool resident = kpad <= kResidentMaxK;  // the whole codebook's operands stay in LDS
    const bool rows = kpad <= kRowsMaxK;          // and its fp32 rows too
    f32x4* const s_c = reinterpret_cast<f32x4*>(s_a + kpad * (kOperandLds / 16));

    // the codebook's scale: fp16 operands need it before any entry is staged
    if (tid == 0) s_next = ub + kAssignWaves;
    float xo[kDim];  // this lane's kernel
    load_kernel(L, ub + wave, lane, xo);
    float c0[kDim];  // entry tid, kept for the staging
    {
        unsigned m = 0u;
#pragma unroll
        for (int d = 0; d < kDim; ++d) c0[d] = tid < k ? C[(size_t)tid * kDim + d] : 0.0f;
        const unsigned* __restrict__ Cu = reinterpret_cast<const unsigned*>(C);
#pragma unroll 8
        for (int e = kAssignWaves * kWave * kDim + tid; e < k * kDim; e += kAssignWaves * kWave)
            m = max(m, Cu[e] & 0x7fffffffu);
#pragma unroll
        for (int d = 0; d < kDim; ++d) m = max(m, __float_as_uint(c0[d]) & 0x7fffffffu);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, off));
        if (lane == 0) s_max[wave] = (int)(m >> 23);
    }
    __syncthreads();
    int Ec, Emax = 0, Emin = 255;  // of the waves whose entries are not all zero
    {
        const int E = lane < kAssignWaves ? s_max[lane] : 0;
#pragma unroll
        for (int w = 0; w < kAssignWaves; ++w) {
            const int o = __builtin_amdgcn_readlane(E, w);
            Emax = max(Emax, o);
            Emin = min(Emin, o > 0 ? o : 255);
        }
        Ec = Emax;
        if (Emax > Emin + kFarExp) {  // the middle one, and what lies within reach above it
            int rank = 0, n = 0;
            for (int w = 0; w < kAssignWaves; ++w) {
                const int o = __builtin_amdgcn_readlane(E, w);
                rank += o > 0 && (o < E || (o == E && w < lane)) ? 1 : 0;
                n += o > 0 ? 1 : 0;
            }
            const unsigned long long mid = __ballot(E > 0 && rank == n / 2);  // one lane
            Ec = min(Emax, __builtin_amdgcn_readlane(E, __ffsll((long long)mid) - 1) + kFarExp);
        }
        Ec = min(max(Ec, 13), 254);
    }
    const float sc = scale_of(Ec), isc = inverse_of(Ec);
    // the guard's terms of the codebook alone: 3 A, 2^(-21 - 2a), and how far from zero far entries begin
    const float gA = 3.0f * 0x1p-14f * isc, gN = 0x1p-21f * isc * isc;
    const float gL = Emax > Ec ? 0.99f * kFarLength * isc : __builtin_inff();

    if (rows)
        stage16<true>(C, k, 0, kpad, sc, s_a, s_c, tid, c0);
    else if (resident)
        stage16<false>(C, k, 0, kpad, sc, s_a, nullptr, tid, c0);

    // this lane's kernel: its scale (biased exponent) and the weight u of the norm terms
    auto kernel_exp = [&](const float (&x)[kDim]) {
        const float m = absmax3(absmax3(x[0], x[1], x[2]), absmax3(x[3], x[4], x[5]), absmax3(x[6], x[7], x[8]));
        return min(max((int)(__float_as_uint(m) >> 23), Ec), 254);
    };
    auto operands = [&](u32x4 (&bop)[2], const float (&x)[kDim]) {
        const int E = kernel_exp(x);
        make_b16(bop, x, scale_of(E), __uint_as_float((unsigned)max(141 - (E - Ec), 0) << 23));
    };

    // unit lu (kernel x of this lane) ends: groups rescored in fp32, the guard, the kernels that it
    // could not settle, the outputs
    auto settle = [&](int lu, const float (&x)[kDim], const Screen3& s) {
        const int i = lu * kWave + lane;
        const bool valid = i < n;
        const float isx = inverse_of(kernel_exp(x));
        float xn2 = 0.0f;
#pragma unroll
        for (int d = 0; d < kDim; ++d) xn2 = __fmaf_rn(x[d], x[d], xn2);
        const float X1 = __builtin_amdgcn_sqrtf(xn2);
        float rd = __builtin_inff();
        int rj = 0x7fffffff;
        // the entries of the group of minimum m in segment g, in increasing index order
        auto rescore = [&](float m, unsigned g, bool ties) {
            const unsigned b = __float_as_uint(m);
            const int e0 = (int)g * kSeg + (int)(8u * ((b >> 2) & 3u) + (b & 3u) + ((b & 16u) ? 4u : 0u));
            float bd = __builtin_inff();
            int bt = -1;
            auto each = [&](int tq, const float (&c)[kDim]) {
                const float d = sqdist9(x, c);
                const bool take = e0 + 32 * tq < k && d < bd;
                bd = take ? d : bd;
                bt = take ? tq : bt;
            };
            if (rows) {
#pragma unroll 4
                for (int tq = 0; tq < kSegTiles; ++tq) {
                    float c[kDim];
                    lds_row(c, s_c, min(e0 + 32 * tq, kpad - 1));
                    each(tq, c);
                }
            } else {
                constexpr int kB = 8;  // rows in flight
#pragma unroll 1
                for (int t0 = 0; t0 < kSegTiles; t0 += kB) {
                    float c[kB][kDim];
#pragma unroll
                    for (int q = 0; q < kB; ++q) mem_row(c[q], C, min(e0 + 32 * (t0 + q), k - 1));
#pragma unroll
                    for (int q = 0; q < kB; ++q) each(t0 + q, c[q]);
                }
            }
            const int bj = e0 + 32 * bt;
            const bool better = bt >= 0 && (bd < rd || (ties && bd == rd && bj < rj));
            rd = better ? bd : rd;
            rj = better ? bj : rj;
        };
        // whether no entry outside the rescored groups can win, m the smallest minimum outside
        auto guard = [&](float m) {
            const float r = X1 + 1.01f * __builtin_amdgcn_sqrtf(rd) + 0x1p-60f;
            const float q = X1 + r, q2 = q * q;
            const float theta = 1.05f * (0x1p-9f * X1 * r + 0x1p-17f * q2 + 6.0f * 0x1p-14f * isx * r + gA * X1 + gN) + 0x1p-100f;
            return valid && q2 < kTrustQ && r < gL && m * isc * isx - (rd - xn2) > theta && rj < k;
        };
        rescore(s.m1, s.seg & 0xffffu, false);
        bool sure = guard(s.m2);
        if (valid && !sure) {  // the second group too
            rescore(s.m2, s.seg >> 16, true);
            sure = guard(s.m3);
        }
        float dist = 0.0f;
        if (sure) {
            dist = rd;
            if (L.idx) L.idx[i] = rj;  // (a fit's rounds before the last may keep no indices)
            if (L.best_d) L.best_d[i] = rd;
        }
        // the kernels the guard could not settle, over the whole codebook
        const unsigned long long fl = __ballot(valid && !sure);
        auto done = [&](float fd, int fj) {
            if (L.idx) L.idx[i] = fj;
            if (L.best_d) L.best_d[i] = fd;
            dist = fd;
        };
        if (rows)
            rescan(fl, x, k, lane, [&](float (&c)[kDim], int jj) { lds_row(c, s_c, jj); }, done);
        else
            rescan(fl, x, k, lane, [&](float (&c)[kDim], int jj) { mem_row(c, C, jj); }, done);
        if (L.part) {
            const double v = wave_sum_f64(valid ? (double)dist : 0.0);
            if (lane == 0) L.part[lu] = v;
        }
    };

    // A run of few units leaves waves idle: several waves then share a unit, each screens every
    // parts-th segment, and the unit's first wave merges their summaries (in LDS, past the staged
    // entries) and settles it.
    const int nseg = (kpad + kSeg - 1) / kSeg;
    int parts = min(kAssignWaves / (u_end - ub), nseg);
    const int staged = kpad * (rows ? kEntryLds : kOperandLds);
    if (!resident || staged + kAssignWaves * kWave * 16 > kLargeLds) parts = 1;
    if (parts > 1) {
        u32x4* const s_x = s_a + (staged + 15) / 16;
        __syncthreads();
        const int uw = wave / parts, part = wave - uw * parts, lu = ub + uw;  // uniform over the wave
        Screen3 s = screen_start();
        if (lu < u_end) {
            load_kernel(L, lu, lane, xo);
            u32x4 bop[2];
            operands(bop, xo);
#pragma unroll 1
            for (int g = part; g < nseg; g += parts)
                scan16<kSegPairs>(s, bop, s_a + g * (kSeg / 32) * kWave, g, min(kSegPairs, (kpad - g * kSeg) >> 6), lane);
            s_x[wave * kWave + lane] = u32x4{__float_as_uint(s.m1), __float_as_uint(s.m2), __float_as_uint(s.m3), s.seg};
        }
        __syncthreads();
        if (lu < u_end && part == 0) {
            for (int q = 1; q < parts; ++q) {
                const u32x4 o = s_x[(wave + q) * kWave + lane];
                merge_screen(s, __uint_as_float(o[0]), __uint_as_float(o[1]), __uint_as_float(o[2]), o[3] & 0xffffu, o[3] >> 16);
            }
            settle(lu, xo, s);
        }
    } else if (resident) {
        // Each wave starts with unit ub + wave and then takes the next unit from an LDS counter,
        // so that a wave its SIMD serves less often takes fewer units; the loop has no barrier.
        __syncthreads();
        int cur = __builtin_amdgcn_readfirstlane(ub + wave);
#pragma unroll 1
        while (cur < u_end) {
            // the next unit's kernel, prefetched while this one is scored (after its last unit this
            // unit's rows again; none is used)
            int g = 0;
            if (lane == 0) g = atomicAdd(&s_next, 1);
            const int nxt = __builtin_amdgcn_readfirstlane(g);
            float xn[kDim];
            load_kernel(L, nxt < u_end ? nxt : cur, lane, xn);
            u32x4 bop[2];
            operands(bop, xo);
            Screen3 s = screen_start();
            scan16<kSegPairs>(s, bop, s_a, 0, kpad >> 6, lane);
            settle(cur, xo, s);
#pragma unroll
            for (int d = 0; d < kDim; ++d) xo[d] = xn[d];
            cur = nxt;
        }
    } else {
        // The codebook streams through LDS in nearly equal chunks of whole segments.  A wave keeps
        // the summaries of up to kStreamUnits units in registers, so a chunk is staged once per
        // kStreamUnits * kAssignWaves units; wave w takes units w, w + kAssignWaves, ... of the
        // block.  The summaries rotate, so every register index is a constant.
        const int nch = (kpad + kStreamChunk - 1) / kStreamChunk;
        const int chunk = ((kpad + nch - 1) / nch + kSeg - 1) / kSeg * kSeg;
#pragma unroll 1
        for (int u0 = ub; u0 < u_end; u0 += kStreamUnits * kAssignWaves) {
            Screen3 st[kStreamUnits];
#pragma unroll
            for (int v = 0; v < kStreamUnits; ++v) st[v] = screen_start();
#pragma unroll 1
            for (int c0 = 0; c0 < kpad; c0 += chunk) {
                const int cn = min(chunk, kpad - c0);
                __syncthreads();  // every wave is done with the previous contents
                stage16<false>(C, k, c0, cn, sc, s_a, nullptr, tid);
                __syncthreads();
                const bool last = c0 + chunk >= kpad;
#pragma unroll 1
                for (int v = 0; v < kStreamUnits; ++v) {
                    const int lu = u0 + wave + v * kAssignWaves;  // uniform over the wave
                    Screen3 s = st[0];
#pragma unroll
                    for (int w = 0; w + 1 < kStreamUnits; ++w) st[w] = st[w + 1];
                    if (lu < u_end) {
                        load_kernel(L, lu, lane, xo);
                        u32x4 bop[2];
                        operands(bop, xo);
                        scan16<kSegPairs>(s, bop, s_a, c0 / kSeg, cn >> 6, lane);
                        if (last) settle(lu, xo, s);
                    }
                    st[kStreamUnits - 1] = s;
                }
            }
        }
    }
}

hipError_t launch_assign_large(const StackParams& p, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
    int kmax = 0;
    for (int l = 0; l < p.nlayers; ++l) kmax = p.L[l].k > kmax ? p.L[l].k : kmax;
    const bool shorter = kmax <= kShortSegK;
    const dim3 g(p.assign_grid), b(kAssignWaves * kWave);
    if (start || stop) {  // the events take the kernel's own start and end times
        if (shorter)
            hipExtLaunchKernelGGL(assign_large_kernel<4>, g, b, 0, s, start, stop, 0, p);
        else
            hipExtLaunchKernelGGL(assign_large_kernel<8>, g, b, 0, s, start, stop, 0, p);
    } else if (shorter) {
        hipLaunchKernelGGL(assign_large_kernel<4>, g, b, 0, s, p);
    } else {
        hipLaunchKernelGGL(assign_large_kernel<8>, g, b, 0, s, p);
    }
    return hipGetLastError();
}

}  // namespace kq
