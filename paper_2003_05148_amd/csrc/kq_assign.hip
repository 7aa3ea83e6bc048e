// Assignment step of kernel-level quantization (Sec. 3.1, Eq. 1) for gfx950.
//
// idx[i] = argmin_j d(x_i, c_j) with d the fp32 squared distance evaluated term by
// term in dimension order (t = x - c, acc = fma(t, t, acc)), ties to the lowest j.
//
// Screening on the matrix cores.  Up to the constant |x|^2, d(x, c_j) is the score
//     s_j = |c_j|^2 - 2 x . c_j = sum_{d < 10} w_jd y_d,  w_j = (-2 c_j, |c_j|^2), y = (x, 1).
// Every fp32 value v is split exactly into v = v_h + v_m + v_l with v_h = bf16(v) and
// v_m = bf16(v - v_h) (round to nearest), and the three cross terms w_h y_h + w_h y_m +
// w_m y_h form a K = 30 (padded to 32) bf16 contraction: two v_mfma_f32_32x32x16_bf16
// per 32 x 32 tile of (codebook entries, kernels), products exact and sums in fp32.  In
// the 32x32 D layout lane l holds column (kernel) l % 32 and 16 of its rows (entries);
// the 32 rows of a kernel are its "slots", slot r holding entries r, r + 32, r + 64, ...
// Each lane keeps the minimum score of each slot, one v_min3 per two scores.
//
// Exactness.  Write u = 2^-24 and P_j = 2 |x| |c_j| + |c_j|^2 <= (|x| + |c_j|)^2.  A
// screened score differs from s_j by at most 823 u P_j (dropped cross terms
// 3 * 2^-16 (1 + 2^-7), at most 33 fp32 roundings in the MFMA sums, 9 u in the fp32
// norm), and a slot minimum that carries its slot number in its 4 lowest mantissa bits
// moves by at most 30 u of its magnitude.  The entries of the slot with the smallest
// minimum are rescored in the plain fp32 form: d* is their smallest distance, taken at
// the lowest index; M2 is the smallest minimum of the other slots, so every entry j
// outside the slot has a screened score >= M2.  With R = 2 |x| + (1 + 2^-9) sqrt(d*) +
// 2^-61 and Q = R^2, such an entry either has |c_j| > R - |x|, and then lies farther
// than (1 + 2^-9) sqrt(d*) from x, so that its fp32 distance (every term positive,
// relative error <= 12 u) exceeds d*; or has P_j <= Q, and then its fp32 distance is at
// least (1 - 12 u) (M2 + |x|^2 - 823 u Q), which exceeds d* once
// M2 + |x|^2 - d* > 870 u Q (packing, the fp32 |x|^2, the distance's rounding and the
// guard's own two roundings included).  The guard asks for more than
// theta = 2^-14 Q' + 2^-100 with Q' = 1.03 (2 sqrt(fl |x|^2) + sqrt(d*) + 2^-60)^2 >= Q
// (1024 u Q; the hardware square roots' errors sit far inside the factor 1.03, and
// 2^-100 covers underflow).  A kernel that passes ends with the slot's fp32 argmin;
// the others are rescored over the whole codebook in the exact fp32 form by their
// wave.  The output is therefore the plain fp32 argmin, bit for bit.  Q' < 1e37 is also
// asked for: every entry with P_j <= Q then has finite partial sums, while a screened
// score of a farther entry may overflow to +inf or NaN, which the slot minima skip.
//
// Grid.  Kernels are cut into units of 64 (one kernel per lane of a wave).  The grid of
// at most kAssignGridMax workgroups is split per layer by cost (assign_partition): layer l
// gets ceil(U_l / floor(t / w_l)) workgroups, w_l the cost of one of its units and t the
// smallest cost per workgroup for which the total fits, and its U_l units are spread
// evenly over them, so a workgroup works within one layer.  This file's kernel serves the
// launches whose codebooks all have at most kAssignMaxK entries (kq_assign_large.hip the others): the
// codebook is split and staged once in LDS, in the MFMA A-operand order [tile][k-step][lane][8 x
// bf16] (one conflict-free ds_read_b128 per MFMA operand) and as fp32 rows for the slot
// rescoring, and the unit loop has no barrier.  Each lane splits its own kernel; the B operands
// of the two 32-kernel tiles of a wave are exchanged between the lane halves with
// v_permlane32_swap.  The next unit's kernels are loaded while the current ones are scored.
// After the scoring each wave settles its own 64 kernels (no workgroup barrier) and, when asked,
// writes an fp64 distortion partial; a second kernel sums the partials in a fixed order.
#include <hip/hip_ext.h>

#include "kq_assign_common.h"

namespace kq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr float kPadScore = 1e38f;  // score of padding entries: finite and above any trusted score
constexpr int kPairs = kFuseMaxK / 64;  // pairs of 32-entry codebook tiles of 256 entries

// two fp32 values split exactly: v = h + m + l with h = bf16(v), m = bf16(v - h); H and M
// hold (h(a), h(b)) and (m(a), m(b)) packed, a in the low half
__device__ __forceinline__ void split2(float a, float b, unsigned& H, unsigned& M) {
    const f32x2 v = {a, b};
    H = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
    const f32x2 r = {a - __uint_as_float(H << 16), b - __uint_as_float(H & 0xffff0000u)};  // exact
    M = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2));
}

// scores of codebook tiles 2p and 2p + 1 (A operands a) against one kernel tile (B operands b)
__device__ __forceinline__ void score_pair(f32x16 (&acc)[2], const u32x4 (&a)[2][2], const u32x4 (&b)[2]) {
    const f32x16 zero = {0.0f};
#pragma unroll
    for (int u = 0; u < 2; ++u)
        acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[u][0]),
                                                         __builtin_bit_cast(bf16x8, b[0]), zero, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 2; ++u)
        acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[u][1]),
                                                         __builtin_bit_cast(bf16x8, b[1]), acc[u], 0, 0, 0);
}

// A operands (entries) of codebook tiles 2 p and 2 p + 1
__device__ __forceinline__ void lds_a(u32x4 (&a)[2][2], const u32x4* s_a, int p, int lane) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) a[t][kk] = s_a[((2 * p + t) * 2 + kk) * kWave + lane];
}

// B operands of a unit's two kernel tiles from the lanes' own kernels.  Kernel tile r of a wave is
// the kernels of lanes 32 r .. 32 r + 31; lane (col, half) needs, for k-step kk, dwords 8 kk + 4
// half .. + 3 of the column's kernel; dword e packs terms 2e, 2e + 1:
// [y_h pairs 0..4 | y_m pairs 0..4 | y_h pairs 0..4 | 0].
__device__ __forceinline__ void make_b(u32x4 (&bop)[2][2], const float (&x)[kDim]) {
    unsigned H[5], M[5];
#pragma unroll
    for (int q = 0; q < 4; ++q) split2(x[2 * q], x[2 * q + 1], H[q], M[q]);
    split2(x[8], 1.0f, H[4], M[4]);
    unsigned D[16];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        D[q] = H[q];
        D[5 + q] = M[q];
        D[10 + q] = H[q];
    }
    D[15] = 0u;
    // lanes < 32 own tile 0 and lanes >= 32 tile 1: swapping (D[8kk+e], D[8kk+4+e])
    // across the halves leaves tile 0's operand in the first result, tile 1's in the second
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const auto sw = __builtin_amdgcn_permlane32_swap(D[8 * kk + e], D[8 * kk + 4 + e], false, false);
            bop[0][kk][e] = sw[0];
            bop[1][kk][e] = sw[1];
        }
}

// One pair of codebook tiles against both kernel tiles, software-pipelined: p holds tile 0's
// scores against this pair (issued a step earlier), a the pair's A operands.  Tile 1's MFMAs run
// while tile 0's scores are folded, and the next pair's tile-0 MFMAs (when there is a next pair)
// while tile 1's are.  An MFMA and VALU work of the same or another wave of a SIMD overlap when
// they are independent: the plain order (eight MFMAs, then 32 v_min3) measured 142 ns per pair
// and SIMD with three waves, this one 125 ns, MFMAs alone 116 ns.
template <bool FIRST, bool MORE>
__device__ __forceinline__ void scan_pair(float (&best)[2][16], f32x16 (&p)[2], u32x4 (&a)[2][2],
                                          const u32x4 (&bop)[2][2], const u32x4* s_a, int t, int lane) {
    f32x16 q[2];
    score_pair(q, a, bop[1]);
    if (MORE) lds_a(a, s_a, t + 1, lane);  // (the operands just used are free)
    fold_pair<FIRST>(best[0], p);
    if (MORE) score_pair(p, a, bop[0]);
    fold_pair<FIRST>(best[1], q);
}

// Smallest and second smallest slot minimum of this lane's kernel, and the winning slot.  Per
// kernel tile the slot number q (rows 8 (q / 4) + 4 half + q % 4) is packed into the low bits.
// A tournament: the smallest and second smallest of each triple (min3, med3); for groups with
// such pairs (m, s), the set's smallest is the least m and its second smallest the smaller of
// the groups' second-least m and the least s (an s of a group that does not hold the minimum is
// at least that group's m).
__device__ __forceinline__ void top2_slots(const float (&best)[2][16], float& M1, float& M2, int& slot) {
    float m1[2], m2[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        float pq[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) pq[q] = __uint_as_float((__float_as_uint(best[r][q]) & ~15u) | (unsigned)q);
        float tm[5], ts[5];
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            tm[t] = min3f(pq[3 * t], pq[3 * t + 1], pq[3 * t + 2]);
            ts[t] = __builtin_amdgcn_fmed3f(pq[3 * t], pq[3 * t + 1], pq[3 * t + 2]);
        }
        const float ma = min3f(tm[0], tm[1], tm[2]);
        const float sa = min2(__builtin_amdgcn_fmed3f(tm[0], tm[1], tm[2]), min3f(ts[0], ts[1], ts[2]));
        const float mb = min3f(tm[3], tm[4], pq[15]);
        const float sb = min2(__builtin_amdgcn_fmed3f(tm[3], tm[4], pq[15]), min2(ts[3], ts[4]));
        m1[r] = min2(ma, mb);
        m2[r] = __builtin_amdgcn_fmed3f(ma, mb, min2(sa, sb));
    }
    // own kernel: lanes < 32 tile 0, lanes >= 32 tile 1; first from the lower half's rows
    const auto x1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(m1[0]), __float_as_uint(m1[1]), false, false);
    const auto x2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(m2[0]), __float_as_uint(m2[1]), false, false);
    const float lo1 = __uint_as_float(x1[0]), hi1 = __uint_as_float(x1[1]);
    const float lo2 = __uint_as_float(x2[0]), hi2 = __uint_as_float(x2[1]);
    M1 = min2(lo1, hi1);
    M2 = __builtin_amdgcn_fmed3f(lo1, hi1, min2(lo2, hi2));
    const int qs = (int)(__float_as_uint(M1) & 15u);
    slot = 8 * (qs >> 2) + (qs & 3) + (hi1 < lo1 ? 4 : 0);
}

// A kernel's screening summary: the smallest slot minimum, the second smallest, the first's slot
struct Screen {
    float m1, m2;
    int slot;
};

// the staged codebook (npair pairs of tiles; FULL: kPairs) screened against a unit's kernels
template <bool FULL>
__device__ __forceinline__ Screen scan(const u32x4 (&bop)[2][2], const u32x4* s_a, int npair, int lane) {
    float best[2][16];
    if constexpr (FULL) {
        asm volatile("" : "+v"(lane));  // the operands are read here, not kept from one unit to the next
        u32x4 a[2][2];
        lds_a(a, s_a, 0, lane);
        f32x16 p[2];
        score_pair(p, a, bop[0]);
        scan_pair<true, true>(best, p, a, bop, s_a, 0, lane);
#pragma unroll
        for (int u = 1; u + 1 < kPairs; ++u) scan_pair<false, true>(best, p, a, bop, s_a, u, lane);
        scan_pair<false, false>(best, p, a, bop, s_a, kPairs - 1, lane);
    } else {  // one pair after another (the pipelined form as a loop, or unrolled per size, spills)
        u32x4 an[2][2];
        {
            u32x4 a[2][2];
            lds_a(a, s_a, 0, lane);
            lds_a(an, s_a, min(1, npair - 1), lane);  // the next pair's operands
            f32x16 acc[2][2];
#pragma unroll
            for (int r = 0; r < 2; ++r) score_pair(acc[r], a, bop[r]);
#pragma unroll
            for (int r = 0; r < 2; ++r) fold_pair<true>(best[r], acc[r]);
        }
#pragma unroll 1
        for (int tp = 1; tp < npair; ++tp) {
            u32x4 a[2][2];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) a[u][kk] = an[u][kk];
            lds_a(an, s_a, min(tp + 1, npair - 1), lane);  // the next pair's operands
            f32x16 acc[2][2];
#pragma unroll
            for (int r = 0; r < 2; ++r) score_pair(acc[r], a, bop[r]);
#pragma unroll
            for (int r = 0; r < 2; ++r) fold_pair<false>(best[r], acc[r]);
        }
    }
    Screen s;
    top2_slots(best, s.m1, s.m2, s.slot);
    return s;
}

// Fused variant (every codebook of at most kFuseMaxK entries): each lane also adds its
// settled kernel to the workgroup's LDS histogram of exact fixed-point member sums, which
// is stored as the partial of (layer, workgroup) when the workgroup's units are done; the
// update then needs only its finishing launch.
__device__ __forceinline__ void fused_store(const DevLayer& H, const unsigned long long* s_sum, const unsigned* s_cnt,
                                            int tid) {
    __syncthreads();  // every wave has added its kernels
    unsigned long long* out = (unsigned long long*)H.hist + (size_t)(blockIdx.x - H.wfirst) * H.k * 10;
    for (int e = tid; e < H.k * 10; e += kAssignWaves * kWave) {
        const int j = e / 10, d = e - 10 * j;
        out[e] = d == 9 ? (unsigned long long)s_cnt[j] : s_sum[j * kDim + d];
    }
}

// a codebook of k entries into LDS, padded to kpad: A operands [w_h | w_h | w_m] of w = (-2c,
// |c|^2) at s_a and the fp32 rows at s_c; entries past the codebook are padding, screened far
// away and never taken by the rescoring (+inf rows)
__device__ __forceinline__ void stage(const float* __restrict__ C, int k, int kpad, u32x4* s_a, f32x4* s_c, int tid) {
    for (int j = tid; j < kpad; j += kAssignWaves * kWave) {
        float c[kDim], w[10];
        if (j < k) {
#pragma unroll
            for (int d = 0; d < kDim; ++d) c[d] = C[(size_t)j * kDim + d];
            float nn = 0.0f;
#pragma unroll
            for (int d = 0; d < kDim; ++d) {
                nn = __fmaf_rn(c[d], c[d], nn);
                w[d] = -2.0f * c[d];
            }
            w[9] = nn;
        } else {
#pragma unroll
            for (int d = 0; d < kDim; ++d) {
                c[d] = __builtin_inff();
                w[d] = 0.0f;
            }
            w[9] = kPadScore;
        }
        unsigned H[5], M[5], A[16];
#pragma unroll
        for (int q = 0; q < 5; ++q) split2(w[2 * q], w[2 * q + 1], H[q], M[q]);
        // [w_h pairs 0..4 | w_h pairs 0..4 | w_m pairs 0..4 | 0]
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            A[q] = H[q];
            A[5 + q] = H[q];
            A[10 + q] = M[q];
        }
        A[15] = 0u;
        const int tl = j >> 5, row = j & 31;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int e0 = 8 * kk + 4 * h;
                const u32x4 v = {A[e0], A[e0 + 1], A[e0 + 2], A[e0 + 3]};
                s_a[(tl * 2 + kk) * kWave + row + 32 * h] = v;
            }
        const f32x4 r0 = {c[0], c[1], c[2], c[3]}, r1 = {c[4], c[5], c[6], c[7]}, r2 = {c[8], 0.f, 0.f, 0.f};
        s_c[j * 3 + 0] = r0;
        s_c[j * 3 + 1] = r1;
        s_c[j * 3 + 2] = r2;
    }
}

// FULL: every codebook of the launch has kFuseMaxK entries once padded (the pipelined scan; in one
// kernel with the loop over any number of pairs it costs 16 registers and a spill).  It gives 0.3 % of a
// pass of the ResNet-18 stack at k = 256 (1198 and 1195 us, runs of one side 0.1 % apart).
template <bool FUSED, int KMAX, bool FULL>
__global__ __launch_bounds__(kAssignWaves * kWave, 1) void assign_kernel(const StackParams p) {
    static_assert((!FUSED && !FULL) || KMAX == kFuseMaxK, "the sums' histogram holds kFuseMaxK entries");
    constexpr bool kSplit = KMAX > kFuseMaxK;       // waves may share a unit
    __shared__ u32x4 s_x[kSplit ? kAssignWaves * kWave : 1];  // their summaries
    __shared__ u32x4 s_a[KMAX / 32 * 2 * kWave];    // [tile][k-step][lane] A operands
    __shared__ f32x4 s_c[KMAX * kRowFloats / 4];    // fp32 rows of the entries
    __shared__ unsigned long long s_sum[FUSED ? kFuseMaxK * kDim : 1];  // fused: member sums
    __shared__ unsigned s_cnt[FUSED ? kFuseMaxK : 1];                   // fused: member counts
    __shared__ int s_next;                                              // the next unit to hand out
    __shared__ unsigned s_mx;                                           // fused: the layer's largest magnitude

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    int n, k;
    const float* C0;
    const AssignRun run = assign_run(p, n, k, C0);
    const float* __restrict__ C = C0;
    const DevLayer& L = p.L[run.layer];
    const unsigned* const xmax = L.xmax;
    const int nxmax = L.nxmax, derive = p.derive_shift;
    const int ub = run.ub, u_end = run.ue;
    if (ub >= u_end) return;

    const int kpad = (k + 63) & ~63;
    if (kpad > KMAX || (FULL && kpad != kFuseMaxK)) return;  // (the host chooses the kernel accordingly)

    float xo[kDim];  // this lane's kernel
    load_kernel(L, ub + wave, lane, xo);
    // fused: the layer's shift, loaded with the first kernels (a later load would be one more
    // round trip before the first unit)
    const unsigned shift_word = FUSED && !derive ? xmax[nxmax] : 0u;
    stage(C, k, kpad, s_a, s_c, tid);  // its loads and the first kernels' are in flight together
    if (tid == 0) s_next = ub + kAssignWaves;
    if (FUSED) {
        for (int e = tid; e < kFuseMaxK * kDim; e += kAssignWaves * kWave) s_sum[e] = 0ull;
        for (int e = tid; e < kFuseMaxK; e += kAssignWaves * kWave) s_cnt[e] = 0u;
    }
    // fused: the scale of the layer's fixed-point sums, read once (or formed from the block
    // maxima, and then stored by the layer's first workgroup for the launches after)
    double fsc = 0.0;
    if (FUSED) {
        int shift;
        if (derive) {
            shift = derive_shift<kAssignWaves * kWave>(L, &s_mx);
            if (run.wg == 0 && tid == 0) L.xmax[L.nxmax] = (unsigned)shift;
        } else {
            shift = (int)shift_word;
        }
        fsc = fixed_scale(shift);
    }

    // unit lu (kernel x of this lane) ends: the winning slot rescored in fp32, the guard, the
    // kernels that it could not settle, the outputs
    // (part, parts: the winning slot counts only every parts-th pair of tiles, from pair `part` on)
    auto settle = [&](int lu, const float (&x)[kDim], const Screen& s, int part, int parts) {
        const int i = lu * kWave + lane;
        const bool valid = i < n;
        // exact fp32 rescoring of the winning slot's entries, in increasing index order
        float rd = __builtin_inff();
        int bt = -1;  // tile of the best entry so far
        auto rescore = [&](int tq) {  // (padding rows are +inf: never taken)
            float c[kDim];
            lds_row(c, s_c, s.slot + 32 * tq);
            const float d = sqdist9(x, c);
            const bool take = d < rd;
            rd = take ? d : rd;
            bt = take ? tq : bt;
        };
        if (FULL || (!kSplit && kpad == kFuseMaxK)) {  // 256 entries: constant tile numbers
#pragma unroll
            for (int tq = 0; tq < 2 * kPairs; ++tq) rescore(tq);
        } else if (!kSplit || parts == 1) {
#pragma unroll 4
            for (int tq = 0; tq < kpad >> 5; ++tq) rescore(tq);
        } else {  // (the part differs from lane to lane: a pair past the end is taken for the last, again)
            const int npair = kpad >> 6, most = (npair + parts - 1) / parts;
#pragma unroll 2
            for (int i = 0; i < most; ++i) {
                const int v = part + i * parts;
                rescore(2 * (v < npair ? v : part));
                rescore(2 * (v < npair ? v : part) + 1);
            }
        }
        const int rj = bt < 0 ? 0x7fffffff : s.slot + 32 * bt;

        float xn2 = 0.0f;
#pragma unroll
        for (int d = 0; d < kDim; ++d) xn2 = __fmaf_rn(x[d], x[d], xn2);
        // the local bound Q' from |x| and the rescored distance; the hardware square roots
        // will do (their errors are far below the factor 1.03)
        const float rr = 2.0f * __builtin_amdgcn_sqrtf(xn2) + __builtin_amdgcn_sqrtf(rd) + 0x1p-60f;
        const float q2 = rr * rr * 1.03f;
        const float theta = 0x1p-14f * q2 + 0x1p-100f;

        const bool sure = valid && (q2 < kTrustQ) && (s.m2 - (rd - xn2) > theta) && (rj < k);
        float dist = 0.0f;
        int myj = rj;  // the entry this lane's kernel ends with
        if (sure) {
            dist = rd;
            if (L.idx) L.idx[i] = rj;  // (a fit's rounds before the last keep no indices)
            if (L.best_d) L.best_d[i] = rd;
        }

        // exact fp32 rescoring of the kernels the guard could not settle
        rescan(__ballot(valid && !sure), x, k, lane, [&](float (&c)[kDim], int jj) { lds_row(c, s_c, jj); },
               [&](float fd, int fj) {
                   if (L.idx) L.idx[i] = fj;
                   if (L.best_d) L.best_d[i] = fd;
                   dist = fd;
                   myj = fj;
               });

        if (FUSED && valid) {  // the update's exact member sums of this kernel, at the layer's shift
            atomicAdd(&s_cnt[myj], 1u);
#pragma unroll
            for (int d = 0; d < kDim; ++d) atomicAdd(&s_sum[myj * kDim + d], fixed_bits(x[d], fsc));
        }

        if (L.part) {
            const double v = wave_sum_f64(valid ? (double)dist : 0.0);
            if (lane == 0) L.part[lu] = v;
        }
    };

    // A run of few units leaves waves idle: several waves then share a unit, each screens every
    // parts-th pair of tiles, and the unit's first wave merges their summaries (in LDS) and settles
    // it: a group is then the entries of one slot in one wave's pairs.  4096 kernels, k = 600: 8.4
    // -> 7.0 us.
    if constexpr (kSplit) {
        const int npair = kpad >> 6, parts = min(kAssignWaves / (u_end - ub), npair);
        if (parts > 1) {
            __syncthreads();
            const int uw = wave / parts, part = wave - uw * parts, lu = ub + uw;  // uniform over the wave
            Screen s = {kMaxFloat, kMaxFloat, 0};
            if (lu < u_end) {
                load_kernel(L, lu, lane, xo);
                u32x4 bop[2][2];
                make_b(bop, xo);
                float best[2][16];
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int q = 0; q < 16; ++q) best[r][q] = kMaxFloat;
#pragma unroll 1
                for (int v = part; v < npair; v += parts) {
                    u32x4 a[2][2];
                    lds_a(a, s_a, v, lane);
                    f32x16 p0[2], p1[2];
                    score_pair(p0, a, bop[0]);
                    score_pair(p1, a, bop[1]);
                    fold_pair<false>(best[0], p0);
                    fold_pair<false>(best[1], p1);
                }
                top2_slots(best, s.m1, s.m2, s.slot);
                s_x[wave * kWave + lane] = u32x4{__float_as_uint(s.m1), __float_as_uint(s.m2), (unsigned)s.slot, 0u};
            }
            __syncthreads();
            if (lu < u_end && part == 0) {
                int win = 0;
                for (int q = 1; q < parts; ++q) {
                    const u32x4 o = s_x[(wave + q) * kWave + lane];
                    const float o1 = __uint_as_float(o[0]), o2 = __uint_as_float(o[1]);
                    const float mx = __builtin_amdgcn_fmed3f(s.m1, o1, __builtin_inff());  // the larger
                    s.m2 = min3f(s.m2, o2, mx);
                    const bool lt = o1 < s.m1;
                    s.m1 = lt ? o1 : s.m1;
                    s.slot = lt ? (int)o[2] : s.slot;
                    win = lt ? q : win;
                }
                settle(lu, xo, s, win, parts);
            }
            return;
        }
    }
    // Each wave starts with unit ub + wave.  With the small units of up to 256 entries it then takes
    // the next unit from an LDS counter, so that a wave its SIMD serves less often takes fewer
    // units; longer units are dealt out in turn (262,144 kernels at k = 512, 16 units for 12 waves:
    // 16.1 us, with the counter 17.3).  The loop has no barrier.
    constexpr bool kCounter = KMAX <= kFuseMaxK;
    __syncthreads();
    int cur = __builtin_amdgcn_readfirstlane(ub + wave);
#pragma unroll 1
    while (cur < u_end) {
        // the next unit's kernel, prefetched while this one is scored (after its last unit this
        // unit's rows again; none is used)
        int nxt = cur + kAssignWaves;
        if constexpr (kCounter) {
            int g = 0;
            if (lane == 0) g = atomicAdd(&s_next, 1);
            nxt = __builtin_amdgcn_readfirstlane(g);
        }
        float xn[kDim];
        load_kernel(L, nxt < u_end ? nxt : cur, lane, xn);
        u32x4 bop[2][2];
        make_b(bop, xo);
        settle(cur, xo, scan<FULL>(bop, s_a, kpad >> 6, lane), 0, 1);
#pragma unroll
        for (int d = 0; d < kDim; ++d) xo[d] = xn[d];
        cur = nxt;
    }
    if (FUSED) fused_store(L, s_sum, s_cnt, tid);
}

// distortion of each layer: its per-wave partials summed in a fixed order
__global__ __launch_bounds__(kSumThreads) void assign_finish_kernel(const StackParams p) {
    __shared__ double s_w[kSumThreads / kWave];
    const DevLayer& L = p.L[blockIdx.x];
    if (L.dist == nullptr) return;
    const double v = block_fixed_sum<kSumThreads>(L.part, L.nunits, s_w);
    if (threadIdx.x == 0) *L.dist = v;
}


// A unit costs about kUnitCost + kpad entries' time: the scan grows with the codebook, the split,
// the rescoring, the guard and the outputs do not (on the 16-layer ResNet-18 stack a fused launch
// takes 22 us at k = 16 and 34 us at k = 256: 17 us without the start-up, and 12 us for 240
// entries).  With units counted alike, the layers with the largest codebooks ended last: this file's
// kernel, when it still served them, took 150 us per launch on the VGG-16 stack with k = 60 .. 1088
// and with the cost 101 us; on the ResNet-18 stack with k = 609 .. 7679 688 and 568 us.  The same cost
// splits the grid of assign_large_kernel, for which it was not fitted.
constexpr long long kUnitCost = 320;

int assign_partition(const int* units, const int* ks, int nlayers, int* g) {
    long long w[KQ_MAX_STACK], lo = 1, hi = 1;
    for (int l = 0; l < nlayers; ++l) {
        w[l] = kUnitCost + ((ks[l] + 63) & ~63);
        lo = w[l] > lo ? w[l] : lo;
        hi = units[l] * w[l] > hi ? units[l] * w[l] : hi;
    }
    auto count = [&](long long t) {  // workgroups when each takes at most t, t >= every w
        long long c = 0;
        for (int l = 0; l < nlayers; ++l) {
            const long long m = t / w[l];
            c += (units[l] + m - 1) / m;
        }
        return c;
    };
    while (lo < hi) {  // count(hi) = nlayers <= the grid
        const long long mid = (lo + hi) / 2;
        if (count(mid) <= kAssignGridMax)
            hi = mid;
        else
            lo = mid + 1;
    }
    int grid = 0;
    for (int l = 0; l < nlayers; ++l) {
        const long long m = lo / w[l];
        g[l] = (int)((units[l] + m - 1) / m);
        grid += g[l];
    }
    return grid;
}

// Up to kAssignMaxK entries the three bf16 cross terms and one rescored slot are faster than the
// other kernel's single product with a second group (262,144 kernels, k = 512: 17 against 20 us;
// k = 1024: 27 us both; k = 2303: 69 against 49 us).
constexpr int kAssignMaxK = 1024;

hipError_t launch_assign(const StackParams& p, hipStream_t s, bool fused, hipEvent_t start, hipEvent_t stop) {
    int kmax = 0, kmin = KQ_MAX_K;
    for (int l = 0; l < p.nlayers; ++l) {
        kmax = p.L[l].k > kmax ? p.L[l].k : kmax;
        kmin = p.L[l].k < kmin ? p.L[l].k : kmin;
    }
    const bool full = kmin > kFuseMaxK - 64 && kmax <= kFuseMaxK;
    if (fused && kmax > kFuseMaxK) return hipErrorInvalidValue;
    if (kmax > kAssignMaxK) return launch_assign_large(p, s, start, stop);
    const dim3 g(p.assign_grid), b(kAssignWaves * kWave);
    auto launch = [&](auto kernel) {
        if (start || stop)  // the events take the kernel's own start and end times
            hipExtLaunchKernelGGL(kernel, g, b, 0, s, start, stop, 0, p);
        else
            hipLaunchKernelGGL(kernel, g, b, 0, s, p);
        return hipGetLastError();
    };
    if (fused) return full ? launch(assign_kernel<true, kFuseMaxK, true>) : launch(assign_kernel<true, kFuseMaxK, false>);
    bool few = true;  // workgroups of few units: their waves share them
    for (int l = 0; l < p.nlayers; ++l) {
        const int w = (l + 1 < p.nlayers ? p.wg_begin[l + 1] : p.assign_grid) - p.wg_begin[l];
        few &= (p.L[l].nunits + w - 1) / w <= kAssignWaves / 2;
    }
    if (kmax > kFuseMaxK || few) return launch(assign_kernel<false, kAssignMaxK, false>);
    return full ? launch(assign_kernel<false, kFuseMaxK, true>) : launch(assign_kernel<false, kFuseMaxK, false>);
}

hipError_t launch_assign_finish(const StackParams& p, hipStream_t s) {
    hipLaunchKernelGGL(assign_finish_kernel, dim3(p.nlayers), dim3(kSumThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace kq
