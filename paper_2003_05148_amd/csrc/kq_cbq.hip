// Kernel codebook quantization (Sec. 3.2): every scalar of a layer's codebook is
// coded with one of 2^bits fp32 levels found by k-means over those scalars, each
// scalar weighted by the appearance count of its codebook entry.
//
// One workgroup per layer.  The weighted sums are exact: a scalar v = M 2^e (fp32)
// times its integer weight w is the integer w M shifted to a fixed position, split
// into 32-bit digits and added to per-level int64 digit accumulators in LDS
// (ds_add_u64).  Integer addition makes the sums independent of the order of the
// work; the exact sum is then rounded once to fp64 (round to nearest even), divided
// by the exact weight total in fp64 and rounded to fp32.  Grid, codes and level
// updates use only correctly rounded fp64 operations, so the codes and levels are
// a pure function of the codebook and the weights.
#include <type_traits>

#include <string.h>

#include "kq_internal.h"

namespace kq {

constexpr int kCbqThreads = 1024;
constexpr int kCbqMaxLevels = 256;
constexpr int kDigits = 11;  // 32-bit digits: |sum of w v| * 2^149 < 2^328

// smallest q minimising fl64(|v - L_q|), by scanning every level
__device__ __forceinline__ int nearest_level(float v, const float* lev, int nlev) {
    const double vd = (double)v;
    double best = fabs(vd - (double)lev[0]);
    int bq = 0;
    for (int q = 1; q < nlev; ++q) {
        const double d = fabs(vd - (double)lev[q]);
        if (d < best) {
            best = d;
            bq = q;
        }
    }
    return bq;
}

// the same, kept as a loop (for rare rounds, where a fully unrolled scan would only cost registers)
__device__ __forceinline__ int nearest_level_loop(float v, const float* lev, int nlev) {
    const double vd = (double)v;
    double best = fabs(vd - (double)lev[0]);
    int bq = 0;
#pragma unroll 1
    for (int q = 1; q < nlev; ++q) {
        const double d = fabs(vd - (double)lev[q]);
        if (d < best) {
            best = d;
            bq = q;
        }
    }
    return bq;
}

// the same when the levels are sorted (L_0 <= L_1 <= ...): the distances in fp64 do not
// grow towards v from either side, so the answer is the first level >= v or, if not
// farther, the lowest-indexed level whose distance equals that of the last level < v
__device__ __forceinline__ int nearest_sorted(float v, const float* lev, int nlev) {
    int q0 = 0;  // number of levels < v (a prefix, as the levels are sorted)
#pragma unroll
    for (int step = kCbqMaxLevels; step >= 1; step >>= 1)
        if (q0 + step <= nlev && lev[q0 + step - 1] < v) q0 += step;
    const double vd = (double)v;
    int q = q0;
    const double da = q0 < nlev ? fabs(vd - (double)lev[q0]) : __builtin_inf();
    if (q0 > 0) {
        int b = q0 - 1;
        const double db = fabs(vd - (double)lev[b]);
        while (b > 0 && fabs(vd - (double)lev[b - 1]) == db) --b;
        if (db <= da) q = b;
    }
    return q;
}

// add w * v * 2^149 (an exact integer) to the digit accumulators of one level
__device__ __forceinline__ void add_exact(unsigned long long* dig, float v, unsigned w) {
    const unsigned u = __float_as_uint(v);
    const unsigned e = (u >> 23) & 0xffu;
    const unsigned mant = u & 0x7fffffu;
    const unsigned M = e ? (mant | 0x800000u) : mant;
    const int sh = e ? (int)e - 1 : 0;  // v * 2^149 = M * 2^sh
    const unsigned long long P = (unsigned long long)w * M;  // < 2^55
    if (P == 0) return;
    const int d0 = sh >> 5, b = sh & 31;
    const unsigned long long lo = P << b;
    const unsigned long long hi = b ? (P >> (64 - b)) : 0ull;
    long long t0 = (long long)(lo & 0xffffffffull), t1 = (long long)(lo >> 32), t2 = (long long)hi;
    if (u >> 31) {
        t0 = -t0;
        t1 = -t1;
        t2 = -t2;
    }
    atomicAdd(&dig[d0], (unsigned long long)t0);
    atomicAdd(&dig[d0 + 1], (unsigned long long)t1);
    if (t2) atomicAdd(&dig[d0 + 2], (unsigned long long)t2);
}

// the exact integer sum_i dig[i] 2^(32 i), times 2^-149, rounded to nearest-even fp64
// (every loop has a fixed trip count, so the limbs stay in registers)
__device__ double digits_to_double(const unsigned long long* dig) {
    unsigned limb[kDigits + 1];
    long long carry = 0;
#pragma unroll
    for (int i = 0; i < kDigits; ++i) {
        const long long t = (long long)dig[i] + carry;
        limb[i] = (unsigned)(t & 0xffffffffll);
        carry = t >> 32;
    }
    limb[kDigits] = (unsigned)carry;
    const bool neg = carry < 0;
    if (neg) {  // two's complement negate
        unsigned c = 1;
#pragma unroll
        for (int i = 0; i <= kDigits; ++i) {
            const unsigned long long t = (unsigned long long)(~limb[i]) + c;
            limb[i] = (unsigned)t;
            c = (unsigned)(t >> 32);
        }
    }
    int h = -1;  // highest nonzero limb
#pragma unroll
    for (int i = 0; i <= kDigits; ++i) h = limb[i] ? i : h;
    if (h < 0) return 0.0;
    unsigned top = 0, l1 = 0, next = 0;
    bool sticky = false;
#pragma unroll
    for (int i = 0; i <= kDigits; ++i) {
        top = i == h ? limb[i] : top;
        l1 = i == h - 1 ? limb[i] : l1;
        next = i == h - 2 ? limb[i] : next;
        sticky |= (i <= h - 3) && limb[i] != 0u;
    }
    const int lz = __clz(top);
    const unsigned long long hi64 = ((unsigned long long)top << 32) | l1;
    unsigned long long win;
    if (lz) {
        win = (hi64 << lz) | (unsigned long long)(next >> (32 - lz));
        sticky |= (next << lz) != 0u;
    } else {
        win = hi64;
        sticky |= next != 0u;
    }
    unsigned long long mant = win >> 11;
    const unsigned rnd = (unsigned)(win & 0x7ffull);
    if (rnd > 0x400u || (rnd == 0x400u && (sticky || (mant & 1ull)))) ++mant;
    const int pos = 32 * h + 31 - lz;  // bit index of the leading one
    const double r = ldexp((double)mant, pos - 52 - 149);
    return neg ? -r : r;
}

// Nearest level of x among NLEV sorted levels (the answer of nearest_sorted): the number
// of levels below x from every eighth level (registers) and one block of eight (LDS), then
// the exact fp64 comparison of the two neighbours, walking down over equal distances.
template <int NLEV>
__device__ __forceinline__ int nearest_sorted_fast(float x, const float* s_lev, const float (&coarse)[NLEV / 8 + 1]) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    int q0;
    if (NLEV >= 8) {
        int c = 0;
        if (NLEV == 64) {  // sorted: three branch-free halving steps and a check of the last
            const bool h4 = coarse[3] < x;
            const bool h2 = (h4 ? coarse[5] : coarse[1]) < x;
            const bool h1 = (h4 ? (h2 ? coarse[6] : coarse[4]) : (h2 ? coarse[2] : coarse[0])) < x;
            c = (h4 ? 4 : 0) + (h2 ? 2 : 0) + (h1 ? 1 : 0);
            c += (c == 7 && coarse[7] < x) ? 1 : 0;
        } else {
#pragma unroll
            for (int i = 0; i < NLEV / 8; ++i) c += coarse[i] < x ? 1 : 0;
        }
        if (c == NLEV / 8) {
            q0 = NLEV;  // the last level is below x, and with it every level
        } else {
            // the block's last level is coarse[c], not below x: halving steps over the other seven
            const f32x4 a = reinterpret_cast<const f32x4*>(s_lev)[2 * c];
            const f32x4 b = reinterpret_cast<const f32x4*>(s_lev)[2 * c + 1];
            const bool f4 = a[3] < x;
            const bool f2 = (f4 ? b[1] : a[1]) < x;
            const bool f1 = (f4 ? (f2 ? b[2] : b[0]) : (f2 ? a[2] : a[0])) < x;
            q0 = 8 * c + (f4 ? 4 : 0) + (f2 ? 2 : 0) + (f1 ? 1 : 0);
        }
    } else {
        q0 = 0;
#pragma unroll
        for (int i = 0; i < NLEV; ++i) q0 += s_lev[i] < x ? 1 : 0;
    }
    const double vd = (double)x;
    int q = q0;
    const double da = q0 < NLEV ? fabs(vd - (double)s_lev[q0]) : __builtin_inf();
    if (q0 > 0) {
        int bq = q0 - 1;
        const double db = fabs(vd - (double)s_lev[bq]);
        while (bq > 0 && fabs(vd - (double)s_lev[bq - 1]) == db) --bq;
        if (db <= da) q = bq;
    }
    return q;
}

// Code thresholds.  With sorted levels whose distinct neighbours are at least 2^-50 M apart (M
// the largest magnitude of the data, so of the levels too) the code of v (nearest level, lowest
// index on ties, distances rounded to fp64) never decreases as v grows, for any v in the data
// range.  Let fl be the rounding, which is monotone, v < v', and suppose code(v) = q and
// code(v') = q' < q (so L_q' < L_q).  fl|v - L_q| < fl|v - L_q'| (a tie would take q'), so v, and
// with it v', lies above the middle of the two.  If v' <= L_q, then fl(L_q - v') <= fl(L_q - v) <
// fl(v - L_q') <= fl(v' - L_q'): q' cannot win at v'.  If v' > L_q, the two distances differ by
// L_q - L_q' >= 2^-50 M, at least two units in the last place of numbers up to 2 M: their
// roundings keep the order, and again q' cannot win.  So code(v) = the number of q < nlev - 1
// with t_q <= v, where t_q is the smallest fp32 value whose code exceeds q (+inf if none).  By the
// same margin no level but a neighbour of v can tie with it, so nearest_sorted finds the code.
// t_q is found by bisection over the fp32 values in their order, evaluating code() with
// nearest_sorted; afterwards each scalar needs only fp32 comparisons.
__device__ __forceinline__ unsigned ordered_key(float f) {
    const unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(unsigned k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// Searched within the data range [vmin, vmax] only.  The boundary lies next to the midpoint of levels q and q + 1, so the search starts there:
// it steps away from the midpoint by 1, 2, 4, ... keys until the code crosses q, then
// bisects the last step.  Every probe keeps code(lo) <= q < code(hi), and the code does not
// decrease with the value, so the answer is the same as bisecting [vmin, vmax] from the
// start; the midpoint only saves probes (about 5 instead of 32).
__device__ float code_threshold(int q, const float* lev, int nlev, float vmin, float vmax) {
    unsigned lo = ordered_key(vmin), hi = ordered_key(vmax);
    auto above = [&](unsigned key) { return nearest_sorted(key_value(key), lev, nlev) > q; };
    if (!above(hi)) return __builtin_inff();
    if (above(lo)) return key_value(lo);
    if (q + 1 < nlev) {
        const unsigned g = ordered_key((float)(0.5 * ((double)lev[q] + (double)lev[q + 1])));
        if (g > lo && g < hi) {
            if (above(g)) {  // the boundary is at g or below: step down from g
                hi = g;
                for (unsigned st = 1u; hi - lo > st; st *= 2u) {
                    if (!above(hi - st)) {
                        lo = hi - st;
                        break;
                    }
                    hi -= st;
                }
            } else {  // above g: step up from g
                lo = g;
                for (unsigned st = 1u; hi - lo > st; st *= 2u) {
                    if (above(lo + st)) {
                        hi = lo + st;
                        break;
                    }
                    lo += st;
                }
            }
        }
    }
    while (hi - lo > 1u) {  // code(lo) <= q < code(hi)
        const unsigned mid = lo + (hi - lo) / 2u;
        if (above(mid))
            hi = mid;
        else
            lo = mid;
    }
    return key_value(hi);
}

// (level_threshold, below, finds most thresholds without a search)
//
// fp32 values v, L with |v|, |L| <= M differ exactly in fp64 when neither is a nonzero
// value below 2^(e(M) - 29) (e = floor(log2)): their exponents then differ by at most 29,
// so v - L needs at most 53 bits.  Returns that floor (0 when M is subnormal or zero).
__device__ __forceinline__ float exact_floor(float M) {
    const int be = (int)((__float_as_uint(M) >> 23) & 255u);
    return be == 0 ? 0.0f : __builtin_ldexpf(1.0f, be - 127 - 29);
}

__device__ __forceinline__ float fp32_above(double y);

// code_threshold without its search where every fp64 distance involved is exact: levels q and
// q + 1 differ, they and the two fp32 values around their midpoint are zero or at least
// exact_floor of the largest magnitude.  The code then changes exactly above the midpoint (which
// fp64 holds exactly); within the data range only.
__device__ __forceinline__ float level_threshold(int q, const float* lev, int nlev, float vmin, float vmax) {
    const float a = lev[q], b = lev[q + 1], fl = exact_floor(fmaxf(fabsf(vmin), fabsf(vmax)));
    if (a != b) {
        const float t = fp32_above(0.5 * ((double)a + (double)b));
        const bool fine = (a == 0.0f || fabsf(a) >= fl) && (b == 0.0f || fabsf(b) >= fl) && fabsf(t) >= 2.0f * fl && fl > 0.0f;
        if (fine) return t > vmax ? __builtin_inff() : fmaxf(t, vmin);
    }
    return code_threshold(q, lev, nlev, vmin, vmax);
}

// code of x from NLEV - 1 sorted thresholds (s_thr[NLEV - 1] = +inf): every eighth from
// registers, then one block of eight from LDS
template <int NLEV>
__device__ __forceinline__ int code_from_thresholds(float x, const float* s_thr, const float (&coarse)[NLEV / 8 + 1]) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    if (NLEV < 8) {
        int q = 0;
#pragma unroll
        for (int i = 0; i < NLEV - 1; ++i) q += s_thr[i] <= x ? 1 : 0;
        return q;
    }
    int c = 0;
    if (NLEV == 64) {
        // the thresholds do not decrease, so the count of the eight coarse ones at or below
        // x takes three halving steps (selects, no branches) and a last check of the eighth
        const bool h4 = coarse[3] <= x;
        const bool h2 = (h4 ? coarse[5] : coarse[1]) <= x;
        const bool h1 = (h4 ? (h2 ? coarse[6] : coarse[4]) : (h2 ? coarse[2] : coarse[0])) <= x;
        c = (h4 ? 4 : 0) + (h2 ? 2 : 0) + (h1 ? 1 : 0);
        c += (c == 7 && coarse[7] <= x) ? 1 : 0;
    } else {
#pragma unroll
        for (int i = 0; i < NLEV / 8; ++i) c += coarse[i] <= x ? 1 : 0;  // coarse[NLEV / 8 - 1] = +inf
    }
    const f32x4 a = reinterpret_cast<const f32x4*>(s_thr)[2 * c];
    const f32x4 b = reinterpret_cast<const f32x4*>(s_thr)[2 * c + 1];
    // the block's eighth threshold is coarse[c] > x: three halving steps over the other seven
    const bool f4 = a[3] <= x;
    const bool f2 = (f4 ? b[1] : a[1]) <= x;
    const bool f1 = (f4 ? (f2 ? b[2] : b[0]) : (f2 ? a[2] : a[0])) <= x;
    return 8 * c + (f4 ? 4 : 0) + (f2 ? 2 : 0) + (f1 ? 1 : 0);
}

// ---- codebooks of at most kCbqExactMax scalars whose values all meet the exactness condition
// (finite, no nonzero magnitude below 2^(e(M) - 29), M the largest magnitude): the rounds
// in integers.  Every value is then a multiple of 2^-S with S = 52 - e(M) (149 when M is
// subnormal), so w v 2^S is an integer below 2^84 in magnitude, held as a 2^42 + b with
// 0 <= b < 2^42; a level keeps the sums A of the a and B of the b of its members (below
// 2^56 for 16384 scalars) and W of their weights in three 64-bit LDS accumulators.  Its new
// value is the exact integer A 2^42 + B rounded once to fp64, times 2^-S, over W in fp64,
// rounded to fp32: the value the digit sums give, bit for bit.  When a round's levels are
// sorted and none is a nonzero value below 2^(e(M) - 29) either, every fp64 distance is
// exact, the nearest level of v (lowest index on ties) changes from q to q + 1 exactly
// above the midpoint of L_q and L_{q+1} (exact in fp64), and the code of v is the number of
// thresholds t_q <= v, t_q the smallest fp32 value above that midpoint (t_q = t_{q+1} when
// L_q = L_{q+1}, whose upper level never wins).  Other rounds search the levels as
// cbq_kernel does.  The scalars, their weights and codes live in LDS; one wave computes the
// levels and thresholds; in a threshold round every scalar checks that it still lies in its
// code's interval [t_{c-1}, t_c), and the few that left it are queued and searched by dense
// lanes, which move their (a, b, w) between the two levels' sums (three barriers a round).
// The 16384 scalars' values, codes and queue, with a weight per entry, fill the LDS (148 KB; up to
// 8192 scalars a weight per scalar).  By the digit path, through memory past 8192 scalars, a launch
// with codebooks of 9792 or 10,827 scalars took 340 to 364 us (limit 4096 scalars), now 104; whole passes:
// VGG-16 stack with k = 60 .. 1088 3.29 ms, now 3.06; ResNet-18 stack with k = 609 .. 7679 11.67, now 11.41.
constexpr int kCbqExactMax = 16384;                         // scalars of a codebook
constexpr int kCbqExactStep = 4096;                         // scalars whose intervals are checked at a time
constexpr int kCbqFastLevels = 64;                          // six bits

// an int128 rounded to nearest-even fp64
__device__ __forceinline__ double i128_to_double(__int128 x) {
    const bool neg = x < 0;
    const unsigned __int128 u = neg ? (unsigned __int128)(-x) : (unsigned __int128)x;
    const unsigned long long hi = (unsigned long long)(u >> 64), lo = (unsigned long long)u;
    double r;
    if (hi == 0) {
        r = (double)lo;  // correctly rounded conversion of 64 bits
    } else {
        const int lz = __clzll((long long)hi);  // 0..63
        const unsigned long long top = lz ? (hi << lz) | (lo >> (64 - lz)) : hi;
        const bool sticky = (lz ? (lo << lz) : lo) != 0ull;
        unsigned long long mant = top >> 11;
        const unsigned rnd = (unsigned)(top & 0x7ffull);
        if (rnd > 0x400u || (rnd == 0x400u && (sticky || (mant & 1ull)))) ++mant;
        r = ldexp((double)mant, 64 + 63 - lz - 52);
    }
    return neg ? -r : r;
}

// the smallest fp32 value above y (y finite, within fp32 range)
__device__ __forceinline__ float fp32_above(double y) {
    const float f = (float)y;  // nearest; a larger fp32 below y cannot exist
    if ((double)f > y) return f;
    const unsigned u = __float_as_uint(f);
    if (u == 0x80000000u || u == 0u) return __uint_as_float(1u);  // above a zero: the smallest subnormal
    return __uint_as_float((u & 0x80000000u) ? u - 1u : u + 1u);
}

// WD: scalars per staged weight (1, or kDim: one weight per entry)
template <int WD>
__device__ void cbq_exact_rounds(const CbqParams& p, const CbqLayer& L, int m, float lo, float hi, float M, float* s_x,
                                 unsigned* s_wt, uint8_t* s_cd, unsigned short* s_q) {
    __shared__ __attribute__((aligned(16))) float s_flev[kCbqFastLevels];
    __shared__ __attribute__((aligned(16))) float s_thr[kCbqFastLevels];
    __shared__ __attribute__((aligned(16))) float s_coarse[kCbqFastLevels / 8];  // every eighth of s_flev or s_thr
    __shared__ unsigned long long s_A[kCbqFastLevels], s_B[kCbqFastLevels], s_W[kCbqFastLevels];
    __shared__ int s_mode;
    __shared__ int s_chg[2];
    __shared__ unsigned s_qn;  // scalars queued this round
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int beM = (int)((__float_as_uint(M) >> 23) & 255u);
    const int S = beM == 0 ? 149 : 179 - beM;
    const float fl = exact_floor(M);

    // the scalars, their weights (those <= 0 add nothing) and, later, their codes in LDS
    for (int r = tid; r < m; r += kCbqThreads) {
        s_x[r] = L.C[r];
        if (WD > 1) continue;
        const int w = L.w ? L.w[r / kDim] : 1;
        s_wt[r] = w > 0 ? (unsigned)w : 0u;
    }
    if (WD > 1)
        for (int r = tid; r < m / WD; r += kCbqThreads) {
            const int w = L.w ? L.w[r] : 1;
            s_wt[r] = w > 0 ? (unsigned)w : 0u;
        }
    // w v 2^S as a 2^42 + b: v 2^S from the bits (the integer mantissa shifted into place,
    // 0 <= shift <= 29 for every value that meets the condition), times w in 128 bits
    auto contrib = [&](float xv, unsigned w, long long& a, unsigned long long& b) {
        const unsigned bits = __float_as_uint(xv);
        const int be = (int)((bits >> 23) & 255u);
        const unsigned long long mant = (unsigned long long)((bits & 0x7fffffu) | (be ? 0x800000u : 0u));
        const long long vs = mant ? (long long)(mant << ((be ? be : 1) - 150 + S)) : 0ll;
        const __int128 X = (__int128)((bits >> 31) ? -vs : vs) * (__int128)w;
        a = (long long)(X >> 42);
        b = (unsigned long long)X & ((1ull << 42) - 1ull);
    };
    // scalar r moves into level q (and, unless `first`, out of level c)
    auto move = [&](int r, int c, int q, bool first) {
        const unsigned w = s_wt[r / WD];
        if (!w) return;
        long long a;
        unsigned long long b;
        contrib(s_x[r], w, a, b);
        if (!first) {
            atomicAdd(&s_A[c], (unsigned long long)(-a));
            atomicAdd(&s_B[c], (unsigned long long)(-(long long)b));
            atomicAdd(&s_W[c], (unsigned long long)(-(long long)w));
        }
        atomicAdd(&s_A[q], (unsigned long long)a);
        atomicAdd(&s_B[q], b);
        atomicAdd(&s_W[q], (unsigned long long)w);
    };
    if (tid < kCbqFastLevels) {
        s_A[tid] = s_B[tid] = s_W[tid] = 0ull;
        const double delta = ((double)hi - (double)lo) / (double)(kCbqFastLevels - 1);
        s_flev[tid] = (float)__dadd_rn((double)lo, __dmul_rn((double)tid, delta));
    }
    if (tid < 2) s_chg[tid] = 0;

    // level q from its sums (unchanged when empty or without `update`): N = A 2^42 + B with
    // B's carries moved into A; while |A| <= 2^53 both parts are exact doubles and one fp64
    // addition rounds N correctly
    auto level_of = [&](int q, bool update) {
        float Lq = s_flev[q];
        const unsigned long long W = s_W[q];
        if (update && W > 0ull) {
            const unsigned long long B = s_B[q];
            const long long A = (long long)s_A[q] + (long long)(B >> 42);
            const unsigned long long Bl = B & ((1ull << 42) - 1ull);
            double N;
            if (A <= (1ll << 53) && A >= -(1ll << 53))
                N = __builtin_ldexp((double)A, 42) + (double)Bl;
            else
                N = i128_to_double(((__int128)A << 42) + (__int128)Bl);
            Lq = (float)(ldexp(N, -S) / (double)W);
        }
        return Lq;
    };
    // wave 0: the levels (from the sums, when `update`), whether they are sorted and exact,
    // and then the thresholds; s_mode = 2 (thresholds), 1 (sorted levels) or 0 (unsorted)
    auto levels = [&](bool update) {
        const int q = lane;
        const float Lq = level_of(q, update);
        s_flev[q] = Lq;
        const float Ln = __shfl_down(Lq, 1);  // the level above (lane 63: its own)
        const bool srt = __all(q == kCbqFastLevels - 1 || Lq <= Ln);
        const bool ex = __all(Lq == 0.0f || fabsf(Lq) >= fl);
        float t = __builtin_inff();
        int src = -1;  // a duplicate takes the threshold of the next level up
        if (q < kCbqFastLevels - 1) {
            if (Lq == Ln)
                src = q + 1;
            else
                t = fp32_above(0.5 * ((double)Lq + (double)Ln));
        }
        if (__any(src >= 0)) {
#pragma unroll
            for (int st = 0; st < 6; ++st) {  // pointer jumping over runs of equal levels
                const float ts = __shfl(t, src < 0 ? q : src);
                const int ss = __shfl(src, src < 0 ? q : src);
                if (src >= 0) {
                    t = ts;
                    src = ss;
                }
            }
        }
        const int mode = srt ? (ex ? 2 : 1) : 0;
        s_thr[q] = t;
        if ((q & 7) == 7) s_coarse[q >> 3] = mode == 2 ? t : Lq;
        if (q == 0) {
            s_mode = mode;
            s_qn = 0u;
        }
    };
    __syncthreads();  // scalars and grid in place
    if (wave == 0) levels(false);
    __syncthreads();

    auto load_coarse = [&](float (&coarse)[kCbqFastLevels / 8 + 1]) {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        const f32x4 c0 = reinterpret_cast<const f32x4*>(s_coarse)[0], c1 = reinterpret_cast<const f32x4*>(s_coarse)[1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            coarse[i] = c0[i];
            coarse[4 + i] = c1[i];
        }
        coarse[kCbqFastLevels / 8] = 0.0f;
    };
    // code of x against the current levels (the mode decides how)
    auto search = [&](float x, int mode, const float (&coarse)[kCbqFastLevels / 8 + 1]) {
        return mode == 2 ? code_from_thresholds<kCbqFastLevels>(x, s_thr, coarse)
                         : (mode == 1 ? nearest_sorted_fast<kCbqFastLevels>(x, s_flev, coarse)
                                      : nearest_level_loop(x, s_flev, kCbqFastLevels));
    };

    {  // the first codes, and with them the sums
        const int mode = __builtin_amdgcn_readfirstlane(s_mode);
        float coarse[kCbqFastLevels / 8 + 1];
        load_coarse(coarse);
        for (int r = tid; r < m; r += kCbqThreads) {
            const int q = search(s_x[r], mode, coarse);
            s_cd[r] = (uint8_t)q;
            move(r, 0, q, true);
        }
    }
    __syncthreads();

    for (int it = 0; it < p.iters; ++it) {
        if (wave == 0) {
            levels(true);
            if (lane == 0) s_chg[it & 1] = 0;  // last read before the previous round's first barrier
        }
        __syncthreads();
        const int mode = __builtin_amdgcn_readfirstlane(s_mode);
        int chg = 0;
        if (mode == 2) {
            // code c stays while t_{c-1} <= v < t_c; the scalars that left their interval are
            // queued and searched by dense lanes (a few per round: no wave runs the search for
            // one lane)
            // (a thread's next four scalars: every code read first, then every bound)
            constexpr int kPer = kCbqExactStep / kCbqThreads;
            for (int r0 = tid; r0 < m; r0 += kCbqExactStep) {
                int c[kPer];
                float x[kPer], tl[kPer], th[kPer];
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const int r = r0 + u * kCbqThreads;
                    c[u] = r < m ? s_cd[r] : 0;
                    x[u] = r < m ? s_x[r] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    tl[u] = s_thr[c[u] > 0 ? c[u] - 1 : 0];
                    th[u] = s_thr[c[u]];
                }
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const int r = r0 + u * kCbqThreads;
                    if (r < m && !((c[u] == 0 || tl[u] <= x[u]) && x[u] < th[u]))
                        s_q[atomicAdd(&s_qn, 1u)] = (unsigned short)r;
                }
            }
            __syncthreads();
            const int n = (int)s_qn;
            if (tid < n) {
                float coarse[kCbqFastLevels / 8 + 1];
                load_coarse(coarse);
                for (int e = tid; e < n; e += kCbqThreads) {
                    const int r = s_q[e];
                    const int c = s_cd[r];
                    const int q = code_from_thresholds<kCbqFastLevels>(s_x[r], s_thr, coarse);  // differs from c
                    move(r, c, q, false);
                    s_cd[r] = (uint8_t)q;
                }
                chg = 1;
            }
        } else {
            float coarse[kCbqFastLevels / 8 + 1];
            load_coarse(coarse);
            for (int r = tid; r < m; r += kCbqThreads) {
                const int c = s_cd[r];
                const int q = search(s_x[r], mode, coarse);
                if (q != c) {
                    move(r, c, q, false);
                    s_cd[r] = (uint8_t)q;
                    chg = 1;
                }
            }
        }
        if (chg) s_chg[it & 1] = 1;
        __syncthreads();
        if (!s_chg[it & 1]) break;
    }

    if (tid < kCbqFastLevels) L.levels[tid] = s_flev[tid];
    for (int r = tid; r < m; r += kCbqThreads) {
        const int c = s_cd[r];
        L.codes[r] = (uint8_t)c;
        if (L.C_hat) L.C_hat[r] = s_flev[c];
    }
}

// Codebooks that the exact rounds do not serve: thread tid handles scalars r = tid, tid + 1024,
// ...  With LDS (codebooks of at most
// kCbqLdsScalars scalars) the scalars, their weights and codes are copied into LDS once;
// otherwise every pass reads them from memory.  The level sums are kept up to date
// incrementally: after the first full accumulation only scalars whose code changes move
// their (exact) contribution between two levels, which leaves the same integers as
// summing from scratch.
constexpr int kCbqLdsScalars = 8192;

// FAST64: 64 levels (6 bits, the paper's width), searched with nearest_sorted_fast
template <bool LDS, bool FAST64>
__global__ __launch_bounds__(kCbqThreads) void cbq_kernel(const CbqParams p) {
    __shared__ __attribute__((aligned(16))) float s_lev[kCbqMaxLevels];
    __shared__ unsigned long long s_dig[kCbqMaxLevels * kDigits];
    __shared__ unsigned long long s_w[kCbqMaxLevels];
    __shared__ float s_lo[kCbqThreads / kWave], s_hi[kCbqThreads / kWave], s_sm[kCbqThreads / kWave];
    __shared__ int s_changed;
    __shared__ int s_unsorted;
    __shared__ float s_v[LDS ? kCbqLdsScalars : 1];
    __shared__ int s_wt[LDS ? kCbqLdsScalars : 1];
    __shared__ uint8_t s_code[LDS ? kCbqLdsScalars : 1];
    // the exact rounds of codebooks past kCbqLdsScalars (weights per entry)
    constexpr bool BIG = !LDS && FAST64;
    __shared__ float s_bv[BIG ? kCbqExactMax : 1];
    __shared__ unsigned s_bw[BIG ? kCbqExactMax / kDim + 1 : 1];
    __shared__ uint8_t s_bc[BIG ? kCbqExactMax : 1];
    __shared__ unsigned short s_bq[BIG ? kCbqExactMax : 1];

    const CbqLayer& L = p.L[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = L.k * kDim;
    const int nlev = 1 << p.bits;
    const bool wk = p.mode == KQ_CBQ_WKMEANS;
    const float* __restrict__ v = L.C;
    uint8_t* __restrict__ codes = L.codes;
    auto val = [&](int r) { return LDS ? s_v[r] : v[r]; };
    auto wgt = [&](int r) { return LDS ? s_wt[r] : (L.w ? L.w[r / kDim] : 1); };
    auto code = [&](int r) { return LDS ? (int)s_code[r] : (int)codes[r]; };
    auto set_code = [&](int r, int q) {
        if (LDS)
            s_code[r] = (uint8_t)q;
        else
            codes[r] = (uint8_t)q;
    };

    // grid on [min, max]; for the integer rounds also the smallest nonzero magnitude and
    // whether a value is not finite
    float lo = __builtin_inff(), hi = -__builtin_inff(), sm = __builtin_inff();
    bool nonfinite = false;
    for (int r = tid; r < m; r += kCbqThreads) {
        const float x = v[r];
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
        if (x != 0.0f) sm = fminf(sm, fabsf(x));
        nonfinite |= !(fabsf(x) <= 3.402823466e38f);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off));
        hi = fmaxf(hi, __shfl_xor(hi, off));
        sm = fminf(sm, __shfl_xor(sm, off));
    }
    nonfinite = __any(nonfinite);
    if (lane == 0) {
        s_lo[wave] = lo;
        s_hi[wave] = hi;
        s_sm[wave] = nonfinite ? -1.0f : sm;
    }
    if (tid == 0) s_unsorted = 0;
    __syncthreads();
    lo = s_lo[0];
    hi = s_hi[0];
    sm = s_sm[0];
    for (int w = 1; w < kCbqThreads / kWave; ++w) {
        lo = fminf(lo, s_lo[w]);
        hi = fmaxf(hi, s_hi[w]);
        sm = s_sm[w] < 0.0f || sm < 0.0f ? -1.0f : fminf(sm, s_sm[w]);
    }
    if (FAST64 && wk && m <= (LDS ? kCbqLdsScalars : kCbqExactMax) && sm >= 0.0f) {
        const float M = fmaxf(fabsf(lo), fabsf(hi));
        if (!(sm < exact_floor(M))) {  // every value meets the exactness condition
            if constexpr (LDS) {
                static_assert(sizeof(s_dig) >= kCbqLdsScalars * sizeof(unsigned short), "the queue of changes");
                cbq_exact_rounds<1>(p, L, m, lo, hi, M, s_v, reinterpret_cast<unsigned*>(s_wt), s_code,
                                    reinterpret_cast<unsigned short*>(s_dig));
                return;
            } else if constexpr (BIG) {
                cbq_exact_rounds<kDim>(p, L, m, lo, hi, M, s_bv, s_bw, s_bc, s_bq);
                return;
            }
        }
    }
    if (LDS) {
        for (int r = tid; r < m; r += kCbqThreads) {
            s_v[r] = v[r];
            s_wt[r] = L.w ? L.w[r / kDim] : 1;
        }
    }
    for (int e = tid; e < nlev * kDigits; e += kCbqThreads) s_dig[e] = 0ull;
    for (int e = tid; e < nlev; e += kCbqThreads) s_w[e] = 0ull;
    if (tid < nlev) {
        const double delta = ((double)hi - (double)lo) / (double)(nlev - 1);
        s_lev[tid] = (float)__dadd_rn((double)lo, __dmul_rn((double)tid, delta));
    }
    __syncthreads();
    if (tid + 1 < nlev && !(s_lev[tid] <= s_lev[tid + 1])) s_unsorted = 1;
    __syncthreads();
    bool sorted = s_unsorted == 0;
    float coarse[64 / 8 + 1];  // every eighth level, for the 64-level search
    auto load_coarse = [&]() {
#pragma unroll
        for (int i = 0; i < 64 / 8; ++i) coarse[i] = FAST64 ? s_lev[8 * i + 7] : 0.0f;
        coarse[64 / 8] = 0.0f;
    };
    auto nearest = [&](float x) {
        if (!sorted) return nearest_level(x, s_lev, nlev);
        return FAST64 ? nearest_sorted_fast<64>(x, s_lev, coarse) : nearest_sorted(x, s_lev, nlev);
    };
    load_coarse();

    // initial codes, and with them the level sums
    for (int r = tid; r < m; r += kCbqThreads) {
        const float x = val(r);
        const int q = nearest(x);
        set_code(r, q);
        const int w = wgt(r);
        if (wk && w > 0) {
            add_exact(s_dig + q * kDigits, x, (unsigned)w);
            atomicAdd(&s_w[q], (unsigned long long)w);
        }
    }
    __syncthreads();

    if (wk) {
        for (int it = 0; it < p.iters; ++it) {
            if (tid == 0) {
                s_changed = 0;
                s_unsorted = 0;
            }
            if (tid < nlev && s_w[tid] > 0ull) {
                const double N = digits_to_double(s_dig + tid * kDigits);
                s_lev[tid] = (float)(N / (double)s_w[tid]);
            }
            __syncthreads();
            if (tid + 1 < nlev && !(s_lev[tid] <= s_lev[tid + 1])) s_unsorted = 1;
            __syncthreads();
            sorted = s_unsorted == 0;
            load_coarse();
            int changed = 0;
            for (int r = tid; r < m; r += kCbqThreads) {
                const float x = val(r);
                const int q = nearest(x);
                const int c = code(r);
                if (q != c) {
                    const int w = wgt(r);
                    if (w > 0) {  // move the exact contribution from level c to level q
                        add_exact(s_dig + c * kDigits, -x, (unsigned)w);
                        add_exact(s_dig + q * kDigits, x, (unsigned)w);
                        atomicAdd(&s_w[c], (unsigned long long)(-(long long)w));
                        atomicAdd(&s_w[q], (unsigned long long)w);
                    }
                    set_code(r, q);
                    changed = 1;
                }
            }
            if (changed) s_changed = 1;
            __syncthreads();
            const int any = s_changed;
            __syncthreads();
            if (!any) break;
        }
    }

    if (tid < nlev) L.levels[tid] = s_lev[tid];
    for (int r = tid; r < m; r += kCbqThreads) {
        const int c = code(r);
        if (LDS) codes[r] = (uint8_t)c;
        if (L.C_hat) L.C_hat[r] = s_lev[c];
    }
}

// ---- large scalar sets (the fully-connected layers, end of Sec. 3.2) ---------------------
// The same method on one flat vector of m scalars, every weight 1, spread over a
// persistent grid.  Per round:
//   fc_assign_kernel  every workgroup codes its scalars against the current levels (LDS)
//                     and adds, in LDS, the exact contributions it moves: in the first
//                     pass every scalar's, later only those of scalars whose code changed
//                     (subtracted from the old level, added to the new); it stores the
//                     per-level digits and counts as its partial and whether it changed
//                     any code;
//   fc_sum_kernel     one workgroup per level adds the partials (stored per level, one per
//                     coding workgroup) to the level's running
//                     exact sum and forms the candidate level fp32(round64(sum) / count);
//   fc_state_kernel   one workgroup: a round that changed no code ends the run (every
//                     later launch returns at once); otherwise the candidates become the
//                     levels while fewer than `iters` updates were made.
// Integer sums make the levels, and with them the codes, independent of the grid and the
// order of the work: the result is the single-workgroup quantizer's, bit for bit.
// A launch serves up to KQ_MAX_STACK sets (blockIdx.y): one large one, or the large codebooks of
// a stack, whose rounds would each leave the chip idle (ten codebooks of 20,727 to 69,111 scalars
// one after another: 3 launches of 3 to 7 us for each round of each, 5.3 ms; together 0.6 ms).
constexpr int kFcCols = kDigits + 1;  // digits, then the count
// scalars from which codes come from thresholds: below, the per-round boundary search costs
// more than the exact search it saves (measured per round: about even at 2^21 scalars,
// 35 instead of 42 us at 3 * 2^20)
constexpr long long kFcThresholdMin = 3ll << 20;
// whether rounds may take their codes from thresholds: unweighted sets only (weighted
// codebooks stay far below that size), by the size rule unless a flag forces a way; the
// device's choice and the host's launch of the threshold kernel use the same rule
__host__ __device__ __forceinline__ bool fc_thr_wanted(const FcParams& p) {
    return p.w == nullptr && (p.thr_mode == 2 || (p.thr_mode == 0 && p.m >= kFcThresholdMin));
}

__device__ __forceinline__ bool fc_done(const FcParams& p) { return p.state[0] != 0; }

// the launch's sets; a set uses the first G workgroups of its row of the grid.  (A single set
// has an argument block of its own: 3 KB of arguments cost each launch 0.3 us more.)
template <int NS>
struct FcStack {
    FcParams L[NS];
};
template <int NS>
__device__ __forceinline__ const FcParams& fc_set(const FcStack<NS>& st) {
    return st.L[NS == 1 ? 0 : blockIdx.y];
}
// the set's workgroups, in a launch whose grid has them along x (a single set's are the grid)
template <int NS>
__device__ __forceinline__ int fc_blocks(const FcStack<NS>& st) {
    return NS == 1 ? (int)gridDim.x : fc_set(st).G;
}

// per workgroup: min and max of its scalars
template <int NS>
__global__ __launch_bounds__(kFcThreads) void fc_minmax_kernel(const FcStack<NS> st) {
    const FcParams& p = fc_set(st);
    const int nblk = fc_blocks(st);
    if (NS > 1 && (int)blockIdx.x >= nblk) return;
    __shared__ float s_lo[kFcThreads / kWave], s_hi[kFcThreads / kWave];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float lo = __builtin_inff(), hi = -__builtin_inff();
    auto take = [&](float x) {
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
    };
    long long r0 = 0;  // scalars from here on: one at a time
    if ((reinterpret_cast<uintptr_t>(p.v) & 15u) == 0) {  // float4 groups, four per thread in flight
        constexpr int kPer = 4;
        const long long ng = p.m >> 2;
        const float4* __restrict__ v4 = reinterpret_cast<const float4*>(p.v);
        for (long long g0 = (long long)blockIdx.x * kFcThreads * kPer + tid; g0 < ng;
             g0 += (long long)nblk * kFcThreads * kPer) {
            float4 xv[kPer];
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const long long g = g0 + (long long)j * kFcThreads;
                xv[j] = g < ng ? v4[g] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (g0 + (long long)j * kFcThreads < ng) {
                    take(xv[j].x);
                    take(xv[j].y);
                    take(xv[j].z);
                    take(xv[j].w);
                }
        }
        r0 = 4 * ng;
    }
    for (long long r = r0 + (long long)blockIdx.x * kFcThreads + tid; r < p.m; r += (long long)nblk * kFcThreads)
        take(p.v[r]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off));
        hi = fmaxf(hi, __shfl_xor(hi, off));
    }
    if (lane == 0) {
        s_lo[wave] = lo;
        s_hi[wave] = hi;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kFcThreads / kWave; ++w) {
            lo = fminf(lo, s_lo[w]);
            hi = fmaxf(hi, s_hi[w]);
        }
        p.minmax[2 * blockIdx.x] = lo;
        p.minmax[2 * blockIdx.x + 1] = hi;
    }
}

// the bucket of x: (x - lo) * sc clamped to [0, kFcBuckets - 1] (NaN to 0), truncated.  Each
// step is monotone, so x <= y gives bucket(x) <= bucket(y); the table and the coding launch
// compute it with the same operations on the same lo and sc.
__device__ __forceinline__ int fc_bucket(float x, float lo, float sc) {
    const float t = (x - lo) * sc;
    return (int)fminf(fmaxf(t, 0.0f), (float)(kFcBuckets - 1));
}

// thresholds of the levels s_lev (sorted unless s_unsorted) when distinct neighbours are at
// least 2^-50 of the largest magnitude apart (state[3]); otherwise state[3] = 0 and the codes
// are found by the exact search.  (An earlier rule asked for exact fp64 distances: no nonzero
// value or level below 2^-29 of the largest magnitude.  Every second set of 10^8 normal values
// holds a smaller one, and its rounds took 520 us by the exact search instead of 104.)  With thresholds and a finite bucket scale the bucket
// table follows: for bucket b, c = the number of thresholds whose bucket is below b (all
// of them below every value of b) and n = the number inside b; entry b = (c | n << 8,
// threshold c or +inf).  A value's code is then c plus the count of the n thresholds
// c .. c + n - 1 at or below it.  Every thread of the workgroup calls it.
__device__ float level_thresholds(const FcParams& p, const float* s_lev, int nlev, int unsorted, int* s_bad, float vmin,
                                  float vmax) {
    const int tid = threadIdx.x;
    const double apart = 0x1p-50 * (double)fmaxf(fabsf(vmin), fabsf(vmax));
    // the boundary search costs a few microseconds per round: worth it only for large sets
    const bool wanted = p.bucketed || fc_thr_wanted(p);
    if (tid == 0) *s_bad = (unsorted || !wanted) ? 1 : 0;
    __syncthreads();
    if (tid + 1 < nlev && s_lev[tid] != s_lev[tid + 1] && (double)s_lev[tid + 1] - (double)s_lev[tid] < apart) *s_bad = 1;
    __syncthreads();
    const int ok = *s_bad == 0;
    float t = __builtin_inff();
    if (tid < nlev) {
        t = (ok && tid + 1 < nlev) ? level_threshold(tid, s_lev, nlev, vmin, vmax) : __builtin_inff();
        p.thr[tid] = t;
    }
    if (tid == 0) p.state[3] = ok;
    return t;
}

// the bucket table of thresholds t (thread q's threshold q)
__device__ void threshold_table(const FcParams& p, float t, int nlev, bool ok, float vmin, float vmax) {
    const int tid = threadIdx.x;
    __shared__ float s_t[kCbqMaxLevels];
    const float sc = (float)kFcBuckets / (vmax - vmin);
    const bool table = ok && vmax > vmin && sc > 0.0f && sc < __builtin_inff();  // the same in every thread
    if (tid == 0) p.range[3] = table ? sc : 0.0f;
    if (!table) return;
    // per bucket the number of thresholds in it; then each thread takes kPerThread consecutive
    // buckets, and c of its first bucket is the exclusive prefix sum of the threads before it
    static_assert(kFcBuckets % kCbqMaxLevels == 0, "whole runs of buckets per thread");
    constexpr int kPerThread = kFcBuckets / kCbqMaxLevels;
    __shared__ int s_n[kFcBuckets];
    __shared__ int s_wsum[kCbqMaxLevels / kWave];
    for (int b = tid; b < kFcBuckets; b += kCbqMaxLevels) s_n[b] = 0;
    if (tid < nlev) s_t[tid] = t;
    __syncthreads();
    if (tid + 1 < nlev) atomicAdd(&s_n[fc_bucket(t, vmin, sc)], 1);  // thresholds 0 .. nlev - 2
    __syncthreads();
    int n[kPerThread], tot = 0;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        n[i] = s_n[kPerThread * tid + i];
        tot += n[i];
    }
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    int inc = tot;  // inclusive scan over the wave
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int o = __shfl_up(inc, off);
        if (lane >= off) inc += o;
    }
    if (lane == kWave - 1) s_wsum[wave] = inc;
    __syncthreads();
    int c = inc - tot;
    for (int w = 0; w < wave; ++w) c += s_wsum[w];
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        const int b = kPerThread * tid + i;
        p.tbl[2 * b] = (unsigned)c | ((unsigned)n[i] << 8);
        p.tbl[2 * b + 1] = __float_as_uint(n[i] > 0 ? s_t[c] : __builtin_inff());
        c += n[i];
    }
}

__device__ void set_thresholds(const FcParams& p, const float* s_lev, int nlev, int unsorted, int* s_bad, float vmin,
                               float vmax) {
    const float t = level_thresholds(p, s_lev, nlev, unsorted, s_bad, vmin, vmax);
    threshold_table(p, t, nlev, *s_bad == 0, vmin, vmax);
}

// the uniform grid on [min, max]; clears the run state and the running sums
template <int NS>
__global__ __launch_bounds__(kCbqMaxLevels) void fc_grid_kernel(const FcStack<NS> st) {
    const FcParams& p = fc_set(st);
    const int nblk = p.G;
    __shared__ float s_lo, s_hi;
    __shared__ float s_lev[kCbqMaxLevels];
    __shared__ int s_unsorted, s_bad;
    __shared__ float s_w[2][kCbqMaxLevels / kWave];
    const int tid = threadIdx.x, nlev = 1 << p.bits;
    {  // the workgroups' minima and maxima: strided per thread, then across the wave and the waves
        float lo = __builtin_inff(), hi = -__builtin_inff();
        for (int b = tid; b < nblk; b += kCbqMaxLevels) {
            lo = fminf(lo, p.minmax[2 * b]);
            hi = fmaxf(hi, p.minmax[2 * b + 1]);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, off));
            hi = fmaxf(hi, __shfl_xor(hi, off));
        }
        if ((tid & (kWave - 1)) == 0) {
            s_w[0][tid / kWave] = lo;
            s_w[1][tid / kWave] = hi;
        }
    }
    __syncthreads();
    if (tid == 0) {
        float lo = s_w[0][0], hi = s_w[1][0];
        for (int w = 1; w < kCbqMaxLevels / kWave; ++w) {
            lo = fminf(lo, s_w[0][w]);
            hi = fmaxf(hi, s_w[1][w]);
        }
        s_lo = lo;
        s_hi = hi;
        p.range[0] = lo;
        p.range[1] = hi;
        s_unsorted = 0;
        p.state[0] = 0;  // not converged
        p.state[1] = 0;  // level updates made
    }
    __syncthreads();
    if (tid < nlev) {
        const double delta = ((double)s_hi - (double)s_lo) / (double)(nlev - 1);
        s_lev[tid] = (float)__dadd_rn((double)s_lo, __dmul_rn((double)tid, delta));
        p.lev[tid] = s_lev[tid];
    }
    for (int e = tid; e < nlev * kFcCols; e += blockDim.x) p.S[e] = 0ll;
    __syncthreads();
    if (tid + 1 < nlev && !(s_lev[tid] <= s_lev[tid + 1])) s_unsorted = 1;
    __syncthreads();
    if (tid == 0) p.state[2] = s_unsorted;
    set_thresholds(p, s_lev, nlev, s_unsorted, &s_bad, s_lo, s_hi);
}

// Each thread takes four scalars per step (r0 + 256 j, consecutive lanes consecutive
// scalars), their loads issued together; with sorted levels a code is the number of
// thresholds at or below the value (fp32 comparisons only).
// THR: the launch for rounds whose codes come from thresholds (true) or from the exact
// searches (false); the state decides on the device, and the other launch returns at once.
// Apart, the light threshold code keeps its register count low.
template <int NS, bool INIT, int NLEV, bool THR>
__global__ __launch_bounds__(kFcThreads) void fc_assign_kernel(const FcStack<NS> st) {
    const FcParams& p = fc_set(st);
    const int nblk = fc_blocks(st);
    if (NS > 1 && (int)blockIdx.x >= nblk) return;
    __shared__ __attribute__((aligned(16))) float s_lev[NLEV < 8 ? 8 : NLEV];
    __shared__ __attribute__((aligned(16))) float s_thr[NLEV < 8 ? 8 : NLEV];
    __shared__ unsigned long long s_dig[NLEV * kFcCols];
    __shared__ uint2 s_tbl[THR ? kFcBuckets : 1];
    // threshold rounds: per wave a queue of the scalars whose code changed (value, old and new
    // code), whose sums are moved 64 at a time by the whole wave
    constexpr int kQCap = 4 * kWave + kWave;  // a group step adds at most 4 per lane
    __shared__ float s_qv[THR ? kFcThreads / kWave : 1][THR ? kQCap : 1];
    __shared__ unsigned short s_qc[THR ? kFcThreads / kWave : 1][THR ? kQCap : 1];
    __shared__ int s_changed;
    if (fc_done(p)) return;
    if ((p.state[3] != 0) != THR) return;  // the other launch codes this round
    const int tid = threadIdx.x;
    for (int e = tid; e < NLEV; e += kFcThreads) {
        s_lev[e] = p.lev[e];
        s_thr[e] = p.thr[e];  // thr[NLEV - 1] is +inf
    }
    const float blo = p.range[0], bsc = p.range[3];
    const bool table = THR && bsc > 0.0f;  // the bucket table of this round's thresholds
    if (table)
        for (int e = tid; e < kFcBuckets; e += kFcThreads) s_tbl[e] = make_uint2(p.tbl[2 * e], p.tbl[2 * e + 1]);
    for (int e = tid; e < NLEV * kFcCols; e += kFcThreads) s_dig[e] = 0ull;
    if (tid == 0) s_changed = 0;
    __syncthreads();
    const bool sorted = p.state[2] == 0;
    float coarse[NLEV / 8 + 1], coarse_lev[NLEV / 8 + 1];
#pragma unroll
    for (int i = 0; i < NLEV / 8; ++i) {
        coarse[i] = s_thr[8 * i + 7];
        coarse_lev[i] = s_lev[8 * i + 7];
    }
    coarse[NLEV / 8] = coarse_lev[NLEV / 8] = 0.0f;
    int changed = 0;
    constexpr int kPer = 4;
    const long long m = p.m;
    // one instantiation per search (bucket table, thresholds, sorted levels, full scan): the choice is
    // the same for every scalar of the round
    auto run = [&](auto mode, auto weighted) {
        constexpr int kMode = decltype(mode)::value;
        constexpr bool kWeighted = decltype(weighted)::value;
        // the code of scalar r (value x, old code c); moves its exact contribution (weight
        // times value, and the weight into the count) when the code changes.  A weight of
        // zero or less contributes nothing, as in the single-workgroup quantizer.
        // the code of value x: the bucket table (two or more thresholds in the bucket: the
        // rest one by one), or a search of the thresholds or levels
        auto table_fixup = [&](float x, uint2 e, int q) {
            if (e.x >= 512u) {  // two or more thresholds in the bucket
                const int c = (int)(e.x & 255u), n = (int)(e.x >> 8);
                for (int j = 1; j < n; ++j) q += s_thr[c + j] <= x ? 1 : 0;
            }
            return q;
        };
        auto search = [&](float x) {
            if constexpr (kMode == 3) {
                const uint2 e = s_tbl[fc_bucket(x, blo, bsc)];
                return table_fixup(x, e, (int)(e.x & 255u) + (__uint_as_float(e.y) <= x ? 1 : 0));
            } else {
                return kMode == 0   ? code_from_thresholds<NLEV>(x, s_thr, coarse)
                       : kMode == 1 ? nearest_sorted_fast<NLEV>(x, s_lev, coarse_lev)
                                    : nearest_level(x, s_lev, NLEV);
            }
        };
        // scalar r (value x, old code c) takes code q: its exact contribution (weight times
        // value, and the weight into the count) moves when the code changes.  A weight of
        // zero or less contributes nothing, as in the single-workgroup quantizer.
        auto recode = [&](long long r, float x, int c, int q) {
            const int wt = kWeighted ? p.w[(unsigned)r / (unsigned)kDim] : 1;  // r < 2^31
            if (INIT) {
                if (wt > 0) {
                    add_exact(s_dig + q * kFcCols, x, (unsigned)wt);
                    atomicAdd(&s_dig[q * kFcCols + kDigits], (unsigned long long)wt);
                }
            } else if (q != c) {
                if (wt > 0) {
                    add_exact(s_dig + c * kFcCols, -x, (unsigned)wt);
                    add_exact(s_dig + q * kFcCols, x, (unsigned)wt);
                    atomicAdd(&s_dig[c * kFcCols + kDigits], (unsigned long long)(-(long long)wt));
                    atomicAdd(&s_dig[q * kFcCols + kDigits], (unsigned long long)wt);
                }
                changed = 1;
            }
            return q;
        };
        // the wave's queue of changed scalars (threshold rounds, unweighted): a lane whose scalar
        // changed appends (value, old code, new code) at the wave's count plus the number of
        // lower lanes appending; drain moves the sums of 64 entries at a time from the queue's
        // end, one per lane (all of them when `all`)
        const int wv = tid / kWave, ln = tid & (kWave - 1);
        int qn = 0;  // the same in every lane of the wave
        auto enqueue = [&](bool ch, float x, int c, int q) {
            if constexpr (THR) {
                const unsigned long long mk = __ballot(ch);
                if (mk == 0ull) return;
                changed = 1;
                if (ch) {
                    const int pos = qn + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mk >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((unsigned)mk, 0u));
                    s_qv[wv][pos] = x;
                    s_qc[wv][pos] = (unsigned short)(c | (q << 8));
                }
                qn += __popcll(mk);
            }
        };
        auto drain = [&](bool all) {
            if constexpr (THR) {
                while (qn >= kWave || (all && qn > 0)) {
                    __builtin_amdgcn_wave_barrier();  // this wave's queue writes come first
                    const int take = qn < kWave ? qn : kWave;
                    if (ln < take) {
                        const int at = qn - take + ln;
                        const float x = s_qv[wv][at];
                        const unsigned cq = s_qc[wv][at];
                        const int c = (int)(cq & 255u), q = (int)(cq >> 8);
                        add_exact(s_dig + c * kFcCols, -x, 1u);
                        add_exact(s_dig + q * kFcCols, x, 1u);
                        atomicAdd(&s_dig[c * kFcCols + kDigits], (unsigned long long)-1ll);
                        atomicAdd(&s_dig[q * kFcCols + kDigits], 1ull);
                    }
                    __builtin_amdgcn_wave_barrier();  // read before the slots are reused
                    qn -= take;
                }
            }
        };
        // the grouped loop for threshold rounds (the large sets); the exact searches (small
        // sets, weighted codebooks, data where thresholds are refused) take one scalar at a time
        if ((kMode == 0 || kMode == 3) && (reinterpret_cast<uintptr_t>(p.v) & 15u) == 0 &&
            (reinterpret_cast<uintptr_t>(p.codes) & 3u) == 0) {
            // groups of four scalars: one float4 of values and one word of four codes per
            // group, kGPer groups per thread and step, the next step's loaded while this one is
            // coded; a group whose codes change stores its word
            constexpr int kGPer = 2;
            const long long ng = m >> 2;
            const long long step = (long long)nblk * kFcThreads * kGPer;
            const float4* __restrict__ v4 = reinterpret_cast<const float4*>(p.v);
            unsigned* __restrict__ c4 = reinterpret_cast<unsigned*>(p.codes);
            auto load = [&](long long g0, float4 (&xv)[kGPer], unsigned (&cw)[kGPer]) {
#pragma unroll
                for (int j = 0; j < kGPer; ++j) {
                    const long long g = g0 + (long long)j * kFcThreads;
                    xv[j] = g < ng ? v4[g] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    cw[j] = (!INIT && g < ng) ? c4[g] : 0u;
                }
            };
            // the loop runs for the whole wave while its first lane has a group: the queue's count
            // must stay the same in every lane, and a drain needs all of them
            long long g0 = (long long)blockIdx.x * kFcThreads * kGPer + tid;
            // kDepth steps in flight: this one and the next (a sweep of groups per step and
            // depth kept 2 and 2)
            constexpr int kDepth = 2;
            float4 xb[kDepth][kGPer];
            unsigned cb[kDepth][kGPer];
#pragma unroll
            for (int d = 0; d < kDepth - 1; ++d)
                if (g0 - ln + d * step < ng) load(g0 + d * step, xb[d], cb[d]);
            for (; g0 - ln < ng; g0 += step) {
                if (g0 - ln + (kDepth - 1) * step < ng) load(g0 + (kDepth - 1) * step, xb[kDepth - 1], cb[kDepth - 1]);
                float4 (&xv)[kGPer] = xb[0];
                unsigned (&cw)[kGPer] = cb[0];
                float xs[kGPer][4];
#pragma unroll
                for (int j = 0; j < kGPer; ++j) {
                    xs[j][0] = xv[j].x;
                    xs[j][1] = xv[j].y;
                    xs[j][2] = xv[j].z;
                    xs[j][3] = xv[j].w;
                }
                int qs[kGPer][4];
                if constexpr (kMode == 3) {  // the step's table reads issued together
                    uint2 te[kGPer][4];
#pragma unroll
                    for (int j = 0; j < kGPer; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) te[j][e] = s_tbl[fc_bucket(xs[j][e], blo, bsc)];
                    unsigned many = 0u;
#pragma unroll
                    for (int j = 0; j < kGPer; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            qs[j][e] = (int)(te[j][e].x & 255u) + (__uint_as_float(te[j][e].y) <= xs[j][e] ? 1 : 0);
                            many |= te[j][e].x;
                        }
                    if (many >= 512u)
#pragma unroll
                        for (int j = 0; j < kGPer; ++j)
#pragma unroll
                            for (int e = 0; e < 4; ++e) qs[j][e] = table_fixup(xs[j][e], te[j][e], qs[j][e]);
                }
#pragma unroll
                for (int j = 0; j < kGPer; ++j) {
                    const long long g = g0 + (long long)j * kFcThreads;
                    const bool have = g < ng;
                    unsigned nw = 0u;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int q = kMode == 3 ? qs[j][e] : search(xs[j][e]);
                        const int c = (int)((cw[j] >> (8 * e)) & 255u);
                        if (INIT) {
                            if (have) recode(4 * g + e, xs[j][e], c, q);
                        } else {
                            enqueue(have && q != c, xs[j][e], c, q);
                        }
                        nw |= (unsigned)q << (8 * e);
                    }
                    if (have && (INIT || nw != cw[j])) c4[g] = nw;
                    if (!INIT) drain(false);
                }
#pragma unroll
                for (int d = 0; d + 1 < kDepth; ++d)
#pragma unroll
                    for (int j = 0; j < kGPer; ++j) {
                        xb[d][j] = xb[d + 1][j];
                        cb[d][j] = cb[d + 1][j];
                    }
            }
            if (!INIT) drain(true);
            if (blockIdx.x == 0)  // the last m % 4 scalars
                for (long long r = 4 * ng + tid; r < m; r += kFcThreads) {
                    const float x = p.v[r];
                    const int q = recode(r, x, INIT ? 0 : (int)p.codes[r], search(x));
                    if (INIT || q != (int)p.codes[r]) p.codes[r] = (uint8_t)q;
                }
        } else {
            const long long step = (long long)nblk * kFcThreads * kPer;
            for (long long r0 = (long long)blockIdx.x * kFcThreads * kPer + tid; r0 < m; r0 += step) {
                float x[kPer];
                int c[kPer];
#pragma unroll
                for (int j = 0; j < kPer; ++j) {
                    const long long r = r0 + (long long)j * kFcThreads;
                    x[j] = r < m ? p.v[r] : 0.0f;
                    c[j] = (!INIT && r < m) ? (int)p.codes[r] : 0;
                }
#pragma unroll
                for (int j = 0; j < kPer; ++j) {
                    const long long r = r0 + (long long)j * kFcThreads;
                    if (r >= m) continue;
                    const int q = recode(r, x[j], c[j], search(x[j]));
                    if (INIT || q != c[j]) p.codes[r] = (uint8_t)q;
                }
            }
        }
    };
    // weights or none: decided once, so unweighted scalars spend nothing on them
    auto pick = [&](auto mode) {
        if (p.w)
            run(mode, std::integral_constant<bool, true>{});
        else
            run(mode, std::integral_constant<bool, false>{});
    };
    if constexpr (THR) {  // never weighted
        if (table)
            run(std::integral_constant<int, 3>{}, std::integral_constant<bool, false>{});
        else
            run(std::integral_constant<int, 0>{}, std::integral_constant<bool, false>{});
    } else {
        if (sorted)
            pick(std::integral_constant<int, 1>{});
        else
            pick(std::integral_constant<int, 2>{});
    }
    if (changed) s_changed = 1;
    __syncthreads();
    // partial of level q at [q][workgroup]: a level's partials are contiguous for fc_sum_kernel
    unsigned long long* part = (unsigned long long*)p.part;
    for (int e = tid; e < NLEV * kFcCols; e += kFcThreads) {
        const int q = e / kFcCols, c = e - q * kFcCols;
        part[((size_t)q * nblk + blockIdx.x) * kFcCols + c] = s_dig[e];
    }
    if (tid == 0) p.wg_changed[blockIdx.x] = INIT ? 1 : s_changed;
}

template <int NS, bool INIT>
hipError_t launch_fc_assign(const FcStack<NS>& st, dim3 G, hipStream_t s) {
    // the threshold launch only where the state may choose thresholds (the sets of a launch are
    // one unweighted set, or codebooks, which never do)
    const bool thr = NS == 1 && fc_thr_wanted(st.L[0]);
    switch (st.L[0].bits) {
#define KQ_FC_CASE(B)                                                                                                \
    case B:                                                                                                          \
        if constexpr (NS == 1) {                                                                                     \
            if (thr) hipLaunchKernelGGL((fc_assign_kernel<1, INIT, (1 << B), true>), G, dim3(kFcThreads), 0, s, st); \
        }                                                                                                            \
        hipLaunchKernelGGL((fc_assign_kernel<NS, INIT, (1 << B), false>), G, dim3(kFcThreads), 0, s, st);            \
        break;
        KQ_FC_CASE(1)
        KQ_FC_CASE(2)
        KQ_FC_CASE(3)
        KQ_FC_CASE(4)
        KQ_FC_CASE(5)
        KQ_FC_CASE(6)
        KQ_FC_CASE(7)
        KQ_FC_CASE(8)
#undef KQ_FC_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// one workgroup per level, a thread per partial: thread b reads partial b (the partials of a level are
// contiguous); a workgroup whose codes did not change added nothing and is skipped (every
// first-pass partial is read)
constexpr int kFcSumThreads = kFcGrid;
template <int NS>
__global__ __launch_bounds__(kFcSumThreads) void fc_sum_kernel(const FcStack<NS> st) {
    const FcParams& p = fc_set(st);
    const int nblk = p.G;
    __shared__ long long s_acc[kFcSumThreads / kWave][kFcCols];
    if (fc_done(p)) return;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    long long a[kFcCols], run = 0;
#pragma unroll
    for (int c = 0; c < kFcCols; ++c) a[c] = 0;
    if (tid < kFcCols) run = p.S[q * kFcCols + tid];  // the level's running sums, loaded while the partials are
    if (tid < nblk && p.wg_changed[tid] != 0) {
        const long long* src = p.part + ((size_t)q * nblk + tid) * kFcCols;
#pragma unroll
        for (int c = 0; c < kFcCols; ++c) a[c] = src[c];
    }
#pragma unroll
    for (int c = 0; c < kFcCols; ++c) a[c] = wave_sum_i64(a[c]);
    if (lane == 0)
        for (int c = 0; c < kFcCols; ++c) s_acc[wave][c] = a[c];
    __syncthreads();
    if (wave != 0) return;
    // lane c adds column c (by one thread, column after column: 2 us a launch longer)
    if (tid < kFcCols) {
#pragma unroll 4
        for (int w = 0; w < (int)blockDim.x / kWave; ++w) run += s_acc[w][tid];
        p.S[q * kFcCols + tid] = run;
    }
    auto column = [&](int c) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)run, c);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)run >> 32), c);
        return (unsigned long long)hi << 32 | lo;
    };
    unsigned long long S[kDigits];
#pragma unroll
    for (int c = 0; c < kDigits; ++c) S[c] = column(c);
    const long long W = (long long)column(kDigits);
    if (tid == 0) p.lev_next[q] = W > 0 ? (float)(digits_to_double(S) / (double)W) : p.lev[q];
}

// run state: stop after a round without a changed code, else take the candidates
template <int NS>
__global__ __launch_bounds__(kCbqMaxLevels) void fc_state_kernel(const FcStack<NS> st) {
    const FcParams& p = fc_set(st);
    const int nblk = p.G;
    __shared__ int s_any, s_unsorted, s_bad;
    __shared__ float s_lev[kCbqMaxLevels];
    if (fc_done(p)) return;
    const int tid = threadIdx.x, nlev = 1 << p.bits;
    if (tid == 0) {
        s_any = 0;
        s_unsorted = 0;
    }
    __syncthreads();
    for (int b = tid; b < nblk; b += blockDim.x)
        if (p.wg_changed[b]) s_any = 1;
    __syncthreads();
    const bool update = s_any && p.state[1] < p.iters;
    if (update && tid < nlev) {
        s_lev[tid] = p.lev_next[tid];
        p.lev[tid] = s_lev[tid];
    }
    __syncthreads();
    if (update && tid + 1 < nlev && !(s_lev[tid] <= s_lev[tid + 1])) s_unsorted = 1;
    __syncthreads();
    if (update) set_thresholds(p, s_lev, nlev, s_unsorted, &s_bad, p.range[0], p.range[1]);  // uniform
    if (tid == 0) {
        if (update) {
            p.state[1] += 1;
            p.state[2] = s_unsorted;
        } else {
            p.state[0] = 1;
        }
    }
}

template <int NS>
__global__ __launch_bounds__(kFcThreads) void fc_output_kernel(const FcStack<NS> st) {
    const FcParams& p = fc_set(st);
    const int nblk = fc_blocks(st);
    if (NS > 1 && (int)blockIdx.x >= nblk) return;
    __shared__ float s_lev[kCbqMaxLevels];
    const int tid = threadIdx.x, nlev = 1 << p.bits;
    for (int e = tid; e < nlev; e += kFcThreads) s_lev[e] = p.lev[e];
    __syncthreads();
    if (blockIdx.x == 0) {
        for (int e = tid; e < nlev; e += kFcThreads) p.levels_out[e] = s_lev[e];
        if (tid == 0 && p.rounds_out) *p.rounds_out = p.state[1];
    }
    if (!p.v_hat) return;
    long long r0 = 0;  // scalars from here on: one at a time
    if ((reinterpret_cast<uintptr_t>(p.v_hat) & 15u) == 0 && (reinterpret_cast<uintptr_t>(p.codes) & 3u) == 0) {
        // a word of four codes in, a float4 out; four groups per thread in flight
        constexpr int kPer = 4;
        const long long ng = p.m >> 2;
        const unsigned* __restrict__ c4 = reinterpret_cast<const unsigned*>(p.codes);
        float4* __restrict__ o4 = reinterpret_cast<float4*>(p.v_hat);
        for (long long g0 = (long long)blockIdx.x * kFcThreads * kPer + tid; g0 < ng;
             g0 += (long long)nblk * kFcThreads * kPer) {
            unsigned cw[kPer];
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const long long g = g0 + (long long)j * kFcThreads;
                cw[j] = g < ng ? c4[g] : 0u;
            }
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const long long g = g0 + (long long)j * kFcThreads;
                if (g < ng)
                    o4[g] = make_float4(s_lev[cw[j] & 255u], s_lev[(cw[j] >> 8) & 255u], s_lev[(cw[j] >> 16) & 255u],
                                        s_lev[cw[j] >> 24]);
            }
        }
        r0 = 4 * ng;
    }
    for (long long r = r0 + (long long)blockIdx.x * kFcThreads + tid; r < p.m; r += (long long)nblk * kFcThreads)
        p.v_hat[r] = s_lev[p.codes[r]];
}

int fc_grid(long long m) {
    const long long b = (m + 4 * kFcThreads - 1) / (4 * kFcThreads);
    return (int)(b < kFcGrid ? (b < 1 ? 1 : b) : kFcGrid);
}

template <int NS>
hipError_t launch_fc_sets(const FcParams* sets, int n, hipStream_t s) {
    FcStack<NS> st;
    memset(&st, 0, sizeof(st));
    int gmax = 1;
    for (int l = 0; l < n; ++l) {
        st.L[l] = sets[l];
        st.L[l].G = fc_grid(sets[l].m);
        gmax = st.L[l].G > gmax ? st.L[l].G : gmax;
    }
    const int nlev = 1 << sets[0].bits, iters = sets[0].iters;
    const dim3 G(gmax, n), one(1, n);
    // level sums by as many threads as there are partials (ten codebooks of 20,727 to 69,111 scalars,
    // 1024 threads a level: 14.5 us a launch, now 7.0; the whole compression pass 12.19 ms, now 12.00)
    const int sum_threads = (gmax + kWave - 1) / kWave * kWave;
    hipLaunchKernelGGL(fc_minmax_kernel<NS>, G, dim3(kFcThreads), 0, s, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fc_grid_kernel<NS>, one, dim3(kCbqMaxLevels), 0, s, st);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // the initial codes and sums, then `iters` rounds of (levels, codes)
    for (int r = 0; r <= iters; ++r) {
        e = r == 0 ? launch_fc_assign<NS, true>(st, G, s) : launch_fc_assign<NS, false>(st, G, s);
        if (e != hipSuccess) return e;
        if (r == iters) break;  // the last codes need no further levels
        hipLaunchKernelGGL(fc_sum_kernel<NS>, dim3(nlev, n), dim3(sum_threads), 0, s, st);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(fc_state_kernel<NS>, one, dim3(kCbqMaxLevels), 0, s, st);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fc_output_kernel<NS>, G, dim3(kFcThreads), 0, s, st);
    return hipGetLastError();
}

// ---- large unweighted sets: rounds on a set partitioned by value ----------------------------
// A round of scalar k-means needs, per threshold t, how many values lie below t and their exact
// sum; a pass over the set per round reads 5 bytes a scalar (104 us for 102,760,448 scalars, at
// the rate of a copy).  So the set is partitioned once, by value, into kFsBuckets buckets of about
// equal size (splitters: quantiles of a sorted sample), with the exact sum and count of the buckets
// before each one.  A round then reads only the buckets that a threshold falls into (63 of 1024).
// The partitioned copy lives in v_hat, which the final pass overwrites; the bucket tables live in
// the region of the coding launches' partials.
//   fs_split_kernel    one workgroup: sorts a sample of kFsSample values, splitters, clears counters
//   fs_hist_kernel     bucket counts, and the set's minimum and maximum
//   fc_grid_kernel     the first levels and thresholds
//   fs_base_kernel     one workgroup: where each bucket begins
//   fs_scatter_kernel  values to their buckets, in tiles of 32768 sorted by bucket in LDS (ranks from
//                      LDS counters, one reservation per tile and bucket; the order within a bucket
//                      is free), so that a bucket's share of a tile, about 128 bytes, is written at
//                      once (straight from the registers: 856 us at 102,760,448 values)
//   fs_sum_kernel      per bucket the exact sum, minimum and maximum (equal shares of the copy)
//   fs_prefix_kernel   one workgroup: exact sums of the buckets before each one
//   per round: fs_cut_kernel (kFsParts workgroups per threshold add its bucket's members below
//   it), fs_state_kernel (level sums as differences of neighbouring cuts, levels, thresholds)
//   fs_output_kernel   codes against the final levels and v_hat, from the original values
// Codes, and with them the end after a round that changed none, depend only on the cuts' counts:
// {v < t} can only change when its size does.  Sums are exact integers, so levels are those of the
// coding launches, bit for bit.  When a round's levels allow no thresholds (neighbours closer than
// 2^-50 of the largest magnitude), this and the rounds after it code every scalar in full scans of
// the set, in the same launches.
// fc6's 102,760,448 scalars, 30 rounds: 4.43 -> 1.60 ms; 4,096,000: 0.87 -> 0.46 ms.
constexpr int kFsBuckets = 1024;
constexpr int kFsSample = 4 * kFsBuckets;
constexpr int kFsThreads = 1024;
constexpr int kFsPer = 32;                       // values per thread and tile
constexpr int kFsTile = kFsPer * kFsThreads;
constexpr int kFsCells = 2048;                   // cells of equal width that index the splitters
constexpr int kFsParts = 16;                     // workgroups per threshold
constexpr int kFsCutThreads = 256;
// A value that fills at least this many buckets (one scalar in 32) needs no search among its run of
// equal splitters, is counted by ballots instead of LDS atomics, all lanes of which would meet at one
// address, and its share of a tile is written by the whole workgroup: a pruned layer's zeros (the set above 691 us, now
// 565; 20,000,000 scalars, 90 % zero, 3 bits, 30 rounds 955, now 624).
constexpr int kFsHeavyRun = kFsBuckets / 32;
enum { kFsDone = 0, kFsUpdates = 1, kFsThr = 3, kFsScan = 4, kFsPrev = 5 };  // state words

struct FsView {
    float* rng;                  // [2] the sample's minimum and maximum: the range of the cells
    int* heavy;                  // [2] a bucket of one value that a large share of the set has, or -1; the value
    float* spl;                  // [kFsBuckets] bucket b holds spl[b] <= v < spl[b + 1] (spl[0] = -inf)
    unsigned *cnt, *base, *cur;  // members, first position ([kFsBuckets + 1]), next free position
    unsigned *kmin, *kmax;       // ordered keys of a bucket's smallest and largest value
    unsigned long long *dig, *pre;  // [.][kDigits] sum of a bucket, of the buckets before ([kFsBuckets + 1])
    unsigned long long* cut;     // [levels][kFsParts][kFcCols] a threshold's bucket members below it
    unsigned* nprev;             // [levels] the previous cuts' counts
    int* tb;                     // [levels] threshold's bucket to read, or -1 - b: the cut is where bucket b begins
    size_t bytes;
};
__host__ __device__ inline FsView fs_view(const FcParams& p) {
    FsView f;
    unsigned char* b = (unsigned char*)p.part;
    size_t o = 0;
    const size_t nlev = (size_t)1 << p.bits;
    auto take = [&](size_t n) {
        unsigned char* const at = b + o;
        o += (n + 255) & ~size_t(255);
        return at;
    };
    f.rng = (float*)take(sizeof(float) * 2 + sizeof(int) * 2);
    f.heavy = (int*)(f.rng + 2);
    f.spl = (float*)take(sizeof(float) * kFsBuckets);
    f.cnt = (unsigned*)take(sizeof(unsigned) * kFsBuckets);
    f.base = (unsigned*)take(sizeof(unsigned) * (kFsBuckets + 1));
    f.cur = (unsigned*)take(sizeof(unsigned) * kFsBuckets);
    f.kmin = (unsigned*)take(sizeof(unsigned) * kFsBuckets);
    f.kmax = (unsigned*)take(sizeof(unsigned) * kFsBuckets);
    f.dig = (unsigned long long*)take(sizeof(long long) * kFsBuckets * kDigits);
    f.pre = (unsigned long long*)take(sizeof(long long) * (kFsBuckets + 1) * kDigits);
    f.cut = (unsigned long long*)take(sizeof(long long) * nlev * kFsParts * kFcCols);
    f.nprev = (unsigned*)take(sizeof(unsigned) * nlev);
    f.tb = (int*)take(sizeof(int) * nlev);
    f.bytes = o;
    return f;
}

// The sort is bitonic with four consecutive keys per thread: partners within a thread or a wave
// meet in registers, those further apart in one of two LDS buffers in turn (one barrier a step, 10
// of the 78 steps; all in LDS: 37 us a launch, now 21).
__global__ __launch_bounds__(kFsThreads) void fs_split_kernel(const FcParams p) {
    constexpr int kOwn = kFsSample / kFsThreads;
    static_assert(kOwn == 4, "a thread's keys are one uint4");
    __shared__ uint4 s_key[2][kFsThreads];
    const FsView f = fs_view(p);
    const int tid = threadIdx.x;
    unsigned a[kOwn];
#pragma unroll
    for (int e = 0; e < kOwn; ++e) a[e] = ordered_key(p.v[(long long)(kOwn * tid + e) * (p.m - 1) / (kFsSample - 1)]);
    for (int e = tid; e < kFsBuckets * kDigits; e += kFsThreads) f.dig[e] = 0ull;
    f.cnt[tid] = 0u;
    f.kmin[tid] = 0xffffffffu;
    f.kmax[tid] = 0u;
    static_assert(kFsThreads == kFsBuckets, "one thread per bucket");
    // keys i and i ^ d meet; runs of k keys ascend where i & k is clear
    auto meet = [&](int k, int d, const unsigned (&o)[kOwn]) {
#pragma unroll
        for (int e = 0; e < kOwn; ++e) {
            const int i = kOwn * tid + e;
            a[e] = ((i & d) == 0) == ((i & k) == 0) ? min(a[e], o[e]) : max(a[e], o[e]);
        }
    };
    int buf = 0;
    for (int k = 2; k <= kFsSample; k *= 2) {
        int d = k / 2;
        for (; d >= kOwn * kWave; d /= 2, buf ^= 1) {
            s_key[buf][tid] = make_uint4(a[0], a[1], a[2], a[3]);
            __syncthreads();
            const uint4 w = s_key[buf][tid ^ (d / kOwn)];
            const unsigned o[kOwn] = {w.x, w.y, w.z, w.w};
            meet(k, d, o);
        }
        for (; d >= kOwn; d /= 2) {
            unsigned o[kOwn];
#pragma unroll
            for (int e = 0; e < kOwn; ++e) o[e] = (unsigned)__shfl_xor((int)a[e], d / kOwn);
            meet(k, d, o);
        }
        if (d == 2) {
            const unsigned o[kOwn] = {a[2], a[3], a[0], a[1]};
            meet(k, 2, o);
        }
        const unsigned o[kOwn] = {a[1], a[0], a[3], a[2]};
        meet(k, 1, o);
    }
    static_assert(kFsSample / kFsBuckets == kOwn, "a thread's first key is its bucket's splitter");
    // A value that fills several buckets gets one of its own: the last splitter of a run of equal
    // ones moves up to the next fp32 value.  A bucket of a single value is never read in a round;
    // with the value's neighbours in it, a threshold among them read them all (4,096,000 scalars, 99 %
    // of them zero, 6 bits, 30 rounds: 4483 us, with this 691).
    __shared__ unsigned s_spl[kFsThreads + 1];
    __shared__ int s_heavy;  // run length of the most frequent value's splitters << 10 | its bucket
    s_spl[tid] = a[0];
    if (tid == 0) {
        s_spl[kFsThreads] = 0xffffffffu;  // past the last run (no finite value's key)
        s_heavy = 0;
    }
    __syncthreads();
    const bool own = tid > 0 && s_spl[tid - 1] == a[0] && s_spl[tid + 1] != a[0] && a[0] < ordered_key(3.402823466e38f);
    f.spl[tid] = tid == 0 ? -__builtin_inff() : key_value(a[0] + (own ? 1u : 0u));
    if (own) {
        int l = -1, h = tid;  // the run's first splitter: s_spl[l] < a[0] <= s_spl[h]
        while (h - l > 1) {
            const int c = (l + h) / 2;
            if (s_spl[c] < a[0]) l = c;
            else h = c;
        }
        atomicMax(&s_heavy, (tid - h + 1) << 10 | (tid - 1));
    }
    __syncthreads();
    if (tid == 0) {
        const bool is = s_heavy >> 10 >= kFsHeavyRun;
        f.heavy[0] = is ? s_heavy & (kFsBuckets - 1) : -1;
        f.heavy[1] = __float_as_int(is ? key_value(s_spl[(s_heavy & (kFsBuckets - 1)) + 1]) : __builtin_nanf(""));
    }
    if (tid == 0) f.rng[0] = key_value(a[0]);
    if (tid == kFsThreads - 1) f.rng[1] = key_value(a[kOwn - 1]);
}

// the splitters and their index in LDS: cell c of equal-width cells over the sample's range (the
// first and last take what lies outside) holds the
// number of splitters in lower cells and, << 16, in the cell itself
struct FsIndex {
    float spl[kFsBuckets];
    unsigned cell[kFsCells];
    unsigned wsum[kFsThreads / kWave];
};
__device__ __forceinline__ int fs_cell(float x, float lo, float sc) {
    return (int)fminf(fmaxf((x - lo) * sc, 0.0f), (float)(kFsCells - 1));  // monotone (NaN to 0)
}
__device__ __forceinline__ float fs_scale(const FsView& f) {
    const float sc = (float)kFsCells / (f.rng[1] - f.rng[0]);
    return sc > 0.0f && sc < __builtin_inff() ? sc : 0.0f;  // 0: one cell
}
__device__ __forceinline__ void fs_index(const FsView& f, FsIndex& s, float lo, float sc) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    constexpr int kPer = kFsCells / kFsThreads;
    const float x = f.spl[tid];
    s.spl[tid] = x;
    for (int c = tid; c < kFsCells; c += kFsThreads) s.cell[c] = 0u;
    __syncthreads();
    if (tid > 0) atomicAdd(&s.cell[fs_cell(x, lo, sc)], 1u);
    __syncthreads();
    unsigned n[kPer], tot = 0u;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        n[i] = s.cell[kPer * tid + i];
        tot += n[i];
    }
    unsigned inc = tot;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const unsigned o = __shfl_up(inc, off);
        if (lane >= off) inc += o;
    }
    if (lane == kWave - 1) s.wsum[wave] = inc;
    __syncthreads();
    unsigned at = inc - tot;
    for (int w = 0; w < wave; ++w) at += s.wsum[w];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        s.cell[kPer * tid + i] = at | (n[i] << 16);
        at += n[i];
    }
    __syncthreads();
}
// the buckets of B values: the splitters at or below each, by the index and then a binary search
// within the cell (the B searches go in step); HEAVY: those of value hv are in bucket heavy
template <int B, bool HEAVY>
__device__ __forceinline__ void fs_buckets(const FsIndex& s, const float* x, int* b, float lo, float sc, int heavy,
                                           float hv) {
    int at[B], n[B];
    int any = 0;
#pragma unroll
    for (int i = 0; i < B; ++i) {
        const unsigned e = s.cell[fs_cell(x[i], lo, sc)];
        const bool known = HEAVY && x[i] == hv;
        at[i] = known ? heavy : (int)(e & 0xffffu);
        n[i] = known ? 0 : (int)(e >> 16);
        any |= n[i];
    }
    while (__any(any)) {
        any = 0;
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int h = n[i] >> 1;
            const bool up = n[i] > 0 && s.spl[min(at[i] + 1 + h, kFsBuckets - 1)] <= x[i];
            at[i] = up ? at[i] + h + 1 : at[i];
            n[i] = up ? n[i] - h - 1 : h;
            any |= n[i];
        }
    }
#pragma unroll
    for (int i = 0; i < B; ++i) b[i] = at[i];
}
// this thread's values of a tile (position i of the tile: 4096 u + 4 tid + e from an aligned set,
// 1024 u + tid otherwise); past the set's end 0, ok false
template <typename F>
__device__ __forceinline__ void fs_tile(const FcParams& p, long long t0, float (&x)[kFsPer], F&& ok) {
    const int tid = threadIdx.x;
    if ((reinterpret_cast<uintptr_t>(p.v) & 15u) == 0) {
        const float4* __restrict__ v4 = reinterpret_cast<const float4*>(p.v);
#pragma unroll
        for (int u = 0; u < kFsPer / 4; ++u) {
            const long long r = t0 + 4ll * (u * kFsThreads + tid);
            float4 w = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (r + 3 < p.m) {
                w = v4[r >> 2];
            } else {
                if (r < p.m) w.x = p.v[r];
                if (r + 1 < p.m) w.y = p.v[r + 1];
                if (r + 2 < p.m) w.z = p.v[r + 2];
            }
            x[4 * u] = w.x;
            x[4 * u + 1] = w.y;
            x[4 * u + 2] = w.z;
            x[4 * u + 3] = w.w;
#pragma unroll
            for (int e = 0; e < 4; ++e) ok(4 * u + e, r + e < p.m);
        }
    } else {
#pragma unroll
        for (int u = 0; u < kFsPer; ++u) {
            const long long r = t0 + u * kFsThreads + tid;
            x[u] = r < p.m ? p.v[r] : 0.0f;
            ok(u, r < p.m);
        }
    }
}

__global__ __launch_bounds__(kFsThreads) void fs_hist_kernel(const FcParams p) {
    __shared__ FsIndex s;
    __shared__ unsigned s_n[kFsBuckets];
    const FsView f = fs_view(p);
    const int tid = threadIdx.x;
    __shared__ float s_lo[kFsThreads / kWave], s_hi[kFsThreads / kWave];
    const float lo = f.rng[0], sc = fs_scale(f);
    const int heavy = f.heavy[0];
    const float hv = __int_as_float(f.heavy[1]);
    unsigned nheavy = 0u;  // the wave's members of the heavy bucket
    float vlo = __builtin_inff(), vhi = -__builtin_inff();
    fs_index(f, s, lo, sc);
    s_n[tid] = 0u;
    __syncthreads();
    auto tiles = [&](auto frequent) {
        constexpr bool kHeavy = decltype(frequent)::value;
        for (long long t0 = (long long)blockIdx.x * kFsTile; t0 < p.m; t0 += (long long)gridDim.x * kFsTile) {
            float x[kFsPer];
            unsigned have = 0u;
            fs_tile(p, t0, x, [&](int i, bool h) { have |= h ? 1u << i : 0u; });
#pragma unroll
            for (int q = 0; q < kFsPer; q += 8) {
                int b[8];
                fs_buckets<8, kHeavy>(s, x + q, b, lo, sc, heavy, hv);
                unsigned put = have >> q;
                if constexpr (kHeavy) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const bool is = (put >> i & 1u) && b[i] == heavy;
                        nheavy += (unsigned)__popcll(__ballot(is));
                        put &= is ? ~(1u << i) : ~0u;
                    }
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (have >> (q + i) & 1u) {
                        if (put >> i & 1u) atomicAdd(&s_n[b[i]], 1u);
                        vlo = fminf(vlo, x[q + i]);
                        vhi = fmaxf(vhi, x[q + i]);
                    }
            }
        }
    };
    if (heavy >= 0)  // (100,000,000 values without a frequent one: both in one loop 196 us a launch, apart 169)
        tiles(std::true_type{});
    else
        tiles(std::false_type{});
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        vlo = fminf(vlo, __shfl_xor(vlo, off));
        vhi = fmaxf(vhi, __shfl_xor(vhi, off));
    }
    if ((tid & (kWave - 1)) == 0) {
        s_lo[tid / kWave] = vlo;
        s_hi[tid / kWave] = vhi;
        if (nheavy) atomicAdd(&s_n[heavy], nheavy);
    }
    __syncthreads();
    if (s_n[tid]) atomicAdd(&f.cnt[tid], s_n[tid]);
    if (tid == 0) {
        for (int w = 1; w < kFsThreads / kWave; ++w) {
            vlo = fminf(vlo, s_lo[w]);
            vhi = fmaxf(vhi, s_hi[w]);
        }
        p.minmax[2 * blockIdx.x] = vlo;
        p.minmax[2 * blockIdx.x + 1] = vhi;
    }
}

__global__ __launch_bounds__(kFsThreads) void fs_base_kernel(const FcParams p) {
    __shared__ unsigned s_w[kFsThreads / kWave];
    const FsView f = fs_view(p);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    if (tid == 0) {
        p.state[kFsScan] = p.state[kFsThr] ? 0 : 1;  // the first levels' thresholds are valid, or not
        p.state[kFsPrev] = 0;
    }
    const unsigned n = f.cnt[tid];
    unsigned inc = n;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const unsigned o = __shfl_up(inc, off);
        if (lane >= off) inc += o;
    }
    if (lane == kWave - 1) s_w[wave] = inc;
    __syncthreads();
    unsigned at = inc - n;
    for (int w = 0; w < wave; ++w) at += s_w[w];
    f.base[tid] = at;
    f.cur[tid] = at;
    if (tid == kFsBuckets - 1) f.base[kFsBuckets] = at + n;
}

__global__ __launch_bounds__(kFsThreads) void fs_scatter_kernel(const FcParams p) {
    __shared__ FsIndex s;
    __shared__ unsigned s_n[kFsBuckets], s_at[kFsBuckets];  // members in the tile; first place in the set
    __shared__ unsigned s_first[kFsBuckets];                // first place in the tile
    __shared__ float s_val[kFsTile];                        // the tile by bucket
    const FsView f = fs_view(p);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    if (p.state[kFsScan]) return;
    const float lo = f.rng[0], sc = fs_scale(f);
    const int heavy = f.heavy[0];
    const float hv = __int_as_float(f.heavy[1]);
    fs_index(f, s, lo, sc);
    float* __restrict__ out = p.v_hat;
    auto tiles = [&](auto frequent) {
        constexpr bool kHeavy = decltype(frequent)::value;
        for (long long t0 = (long long)blockIdx.x * kFsTile; t0 < p.m; t0 += (long long)gridDim.x * kFsTile) {
            s_n[tid] = 0u;
            float x[kFsPer];
            unsigned have = 0u, br[kFsPer];  // bucket | rank << 10
            fs_tile(p, t0, x, [&](int i, bool h) { have |= h ? 1u << i : 0u; });
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kFsPer; q += 8) {
                int b[8];
                fs_buckets<8, kHeavy>(s, x + q, b, lo, sc, heavy, hv);
                unsigned put = have >> q;
#pragma unroll
                for (int i = 0; i < 8; ++i) br[q + i] = (unsigned)b[i];
                if constexpr (kHeavy) {  // the wave's members take consecutive ranks
                    unsigned n = 0u, r[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const bool is = (put >> i & 1u) && b[i] == heavy;
                        const unsigned long long m = __ballot(is);
                        r[i] = is ? n + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u)) : 0u;
                        n += (unsigned)__popcll(m);
                        put &= is ? ~(1u << i) : ~0u;
                    }
                    unsigned first = 0u;
                    if (lane == 0 && n) first = atomicAdd(&s_n[heavy], n);
                    first = (unsigned)__builtin_amdgcn_readfirstlane((int)first);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (b[i] == heavy) br[q + i] |= (first + r[i]) << 10;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (put >> i & 1u) br[q + i] |= atomicAdd(&s_n[b[i]], 1u) << 10;
            }
            __syncthreads();
            const unsigned n = s_n[tid];
            s_at[tid] = n ? atomicAdd(&f.cur[tid], n) : 0u;
            unsigned inc = n;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const unsigned o = __shfl_up(inc, off);
                if (lane >= off) inc += o;
            }
            if (lane == kWave - 1) s.wsum[wave] = inc;
            __syncthreads();
            unsigned at = inc - n;
            for (int w = 0; w < wave; ++w) at += s.wsum[w];
            s_first[tid] = at;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kFsPer; ++q)
                if (have >> q & 1u) s_val[s_first[br[q] & (kFsBuckets - 1)] + (br[q] >> 10)] = x[q];
            __syncthreads();
            // half a wave per bucket
            constexpr int kHalves = 2 * kFsThreads / kWave;
            const int h = 2 * wave + (lane >> 5), l = lane & 31;
#pragma unroll 4
            for (int b = h; b < kFsBuckets; b += kHalves) {
                const unsigned c = kHeavy && b == heavy ? 0u : s_n[b], g = s_at[b], v = s_first[b];
                for (unsigned i = l; i < c; i += 32) out[g + i] = s_val[v + i];
            }
            if constexpr (kHeavy) {
                const unsigned c = s_n[heavy], g = s_at[heavy], v = s_first[heavy];
                for (unsigned i = tid; i < c; i += kFsThreads) out[g + i] = s_val[v + i];
            }
            __syncthreads();
        }
    };
    if (heavy >= 0)
        tiles(std::true_type{});
    else
        tiles(std::false_type{});
}

// Exact sum of values in registers: three 32-bit digits from digit d0 on, as 64-bit counts (each
// value adds less than 2^32 to a digit).  A value with bits below digit d0 goes to the LDS digits.
struct FsSum {
    long long a0, a1, a2;
};
__device__ __forceinline__ void fs_add(FsSum& s, float x, int d0, unsigned long long* low) {
    const unsigned u = __float_as_uint(x), e = (u >> 23) & 0xffu;
    const unsigned mant = (u & 0x7fffffu) | (e ? 0x800000u : 0u);
    const int sh = (e ? (int)e - 1 : 0) - 32 * d0;  // x 2^149 = mant 2^(sh + 32 d0)
    if (sh < 0) {
        if (mant) add_exact(low, x, 1u);
        return;
    }
    const unsigned long long P = (unsigned long long)mant << (sh & 31);
    long long l = (long long)(P & 0xffffffffull), h = (long long)(P >> 32);
    if (u >> 31) {
        l = -l;
        h = -h;
    }
    const bool up = sh >= 32;  // (sh < 64: d0 fits the largest magnitude)
    s.a0 += up ? 0ll : l;
    s.a1 += up ? l : h;
    s.a2 += up ? h : 0ll;
}
// the lowest digit for values of magnitude at most M
__device__ __forceinline__ int fs_digit(float M) {
    const int e = (int)((__float_as_uint(M) >> 23) & 0xffu);
    const int d = (e ? e - 1 : 0) >> 5;
    return d > 0 ? d - 1 : 0;
}
// the largest magnitude a member of bucket b can have
__device__ __forceinline__ float fs_bound(const FcParams& p, const FsView& f, int b) {
    const float l = b == 0 ? p.range[0] : f.spl[b], h = b == kFsBuckets - 1 ? p.range[1] : f.spl[b + 1];
    return fmaxf(fabsf(l), fabsf(h));
}

__global__ __launch_bounds__(kFsCutThreads) void fs_sum_kernel(const FcParams p) {
    __shared__ unsigned long long s_dig[kDigits];
    __shared__ unsigned s_lo, s_hi;
    __shared__ int s_b;
    const FsView f = fs_view(p);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    if (p.state[kFsScan]) return;
    const long long len = (p.m + gridDim.x - 1) / gridDim.x;
    const long long i0 = blockIdx.x * len, i1 = i0 + len < p.m ? i0 + len : p.m;
    if (i0 >= i1) return;
    if (tid == 0) {  // the bucket of position i0: the last one that begins at or before it and is not empty
        int l = 0, h = kFsBuckets;
        while (h - l > 1) {
            const int c = (l + h) / 2;
            if ((long long)f.base[c] <= i0) l = c;
            else h = c;
        }
        s_b = l;
    }
    __syncthreads();
    int b = s_b;
    for (long long a = i0; a < i1; ++b) {  // (uniform: every thread walks the same buckets)
        const long long end = f.base[b + 1], z = end < i1 ? end : i1;
        if (z <= a) continue;
        if (tid < kDigits) s_dig[tid] = 0ull;
        if (tid == 0) s_lo = 0xffffffffu, s_hi = 0u;
        __syncthreads();
        const int d0 = fs_digit(fs_bound(p, f, b));
        FsSum s = {0, 0, 0};
        unsigned lo = 0xffffffffu, hi = 0u;
        const float* __restrict__ w = p.v_hat;
        for (long long r = a + tid; r < z; r += 8 * kFsCutThreads) {
            float x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = r + q * kFsCutThreads < z ? w[r + q * kFsCutThreads] : 0.0f;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (r + q * kFsCutThreads < z) {
                    const unsigned k = ordered_key(x[q]);
                    lo = min(lo, k);
                    hi = max(hi, k);
                    fs_add(s, x[q], d0, s_dig);
                }
        }
        s.a0 = wave_sum_i64(s.a0);
        s.a1 = wave_sum_i64(s.a1);
        s.a2 = wave_sum_i64(s.a2);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            lo = min(lo, (unsigned)__shfl_xor((int)lo, off));
            hi = max(hi, (unsigned)__shfl_xor((int)hi, off));
        }
        if (lane == 0) {
            atomicAdd(&s_dig[d0], (unsigned long long)s.a0);
            atomicAdd(&s_dig[d0 + 1], (unsigned long long)s.a1);
            atomicAdd(&s_dig[d0 + 2], (unsigned long long)s.a2);
            atomicMin(&s_lo, lo);
            atomicMax(&s_hi, hi);
        }
        __syncthreads();
        if (tid < kDigits && s_dig[tid]) atomicAdd(&f.dig[b * kDigits + tid], s_dig[tid]);
        if (tid == 0) {
            atomicMin(&f.kmin[b], s_lo);
            atomicMax(&f.kmax[b], s_hi);
        }
        __syncthreads();
        a = z;
    }
}

// a threshold's place: the bucket whose members have to be looked at, or -1 - b when every member
// below it lies in a bucket before b and none in b or after
__device__ __forceinline__ int fs_place(const float* spl, const unsigned* cnt, const unsigned* kmin, const unsigned* kmax,
                                        float t) {
    if (t == __builtin_inff()) return -1 - kFsBuckets;
    int l = 0, h = kFsBuckets;  // spl[l] <= t < spl[h]
    while (h - l > 1) {
        const int c = (l + h) / 2;
        if (spl[c] <= t) l = c;
        else h = c;
    }
    if (cnt[l] == 0u || t <= key_value(kmin[l])) return -1 - l;
    if (t > key_value(kmax[l])) return -1 - (l + 1);
    return l;
}

__global__ __launch_bounds__(kFsThreads) void fs_prefix_kernel(const FcParams p) {
    const FsView f = fs_view(p);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), c = tid / kWave;
    if (p.state[kFsScan]) return;
    static_assert(kFsThreads / kWave >= kDigits, "a wave per digit");
    if (c < kDigits) {
        constexpr int kPer = kFsBuckets / kWave;  // consecutive buckets per lane
        unsigned long long n[kPer], tot = 0ull;
#pragma unroll
        for (int i = 0; i < kPer; ++i) n[i] = f.dig[(lane * kPer + i) * kDigits + c];
#pragma unroll
        for (int i = 0; i < kPer; ++i) tot += n[i];
        unsigned long long inc = tot;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const unsigned long long o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        unsigned long long at = inc - tot;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            f.pre[(lane * kPer + i) * kDigits + c] = at;
            at += n[i];
        }
        if (lane == kWave - 1) f.pre[kFsBuckets * kDigits + c] = at;
    }
    const int nlev = 1 << p.bits;
    if (tid + 1 < nlev) f.tb[tid] = fs_place(f.spl, f.cnt, f.kmin, f.kmax, p.thr[tid]);
}

// workgroups of a full-scan round
__device__ __forceinline__ int fs_scan_blocks(const FcParams& p) { return min(p.G, (1 << p.bits) * kFsParts); }

// kFsParts workgroups per threshold: the count and exact sum of the members of its bucket below it.
// Full-scan rounds: the first fs_scan_blocks workgroups code every scalar, by the coding launches' search,
// and add the levels' sums, or from the second such round on their changes, to the running sums.
// 20,000,000 scalars, half of them near 1e-17 of the others, 30 rounds at 6 and 8 bits: by the scan of
// all levels and whole sums, added up by the state's workgroup, 15.2 and 53.7 ms; now 2.7 and 3.4; by
// the exact search of the coding launches 3.1 and 2.8.
template <int NLEV>
__global__ __launch_bounds__(kFsCutThreads) void fs_cut_kernel(const FcParams p) {
    __shared__ unsigned long long s_dig[NLEV * kFcCols];
    __shared__ __attribute__((aligned(16))) float s_lev[NLEV];
    __shared__ float s_old[NLEV];
    __shared__ int s_changed;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const FsView f = fs_view(p);
    const int q = blockIdx.x / kFsParts, part = blockIdx.x - q * kFsParts;
    // one batch of loads: the run's state, this threshold and its place
    const int done = p.state[kFsDone], scan = p.state[kFsScan], b = f.tb[q];
    const float t = p.thr[q];
    asm volatile("" ::"s"(done), "s"(scan), "s"(b), "s"(t));
    if (done) return;
    if (scan) {
        const int nblk = fs_scan_blocks(p);
        if ((int)blockIdx.x >= nblk) return;
        // The first one forms codes and sums; the later ones move what changed its code.
        const int prev = p.state[kFsPrev];
        const bool sorted = p.state[2] == 0;
        for (int e = tid; e < NLEV * kFcCols; e += kFsCutThreads) s_dig[e] = 0ull;
        for (int e = tid; e < NLEV; e += kFsCutThreads) {
            s_lev[e] = p.lev[e];
            s_old[e] = p.lev_next[e];  // the thresholds of the round before the first full scan
        }
        if (tid == 0) s_changed = prev == 0 ? 1 : 0;
        __syncthreads();
        float coarse[NLEV / 8 + 1];
#pragma unroll
        for (int i = 0; i < NLEV / 8; ++i) coarse[i] = s_lev[8 * i + 7];
        coarse[NLEV / 8] = 0.0f;
        constexpr int kPer = 4;  // scalars in flight per thread
        const long long step = (long long)nblk * kFsCutThreads * kPer;
        for (long long r0 = (long long)blockIdx.x * kFsCutThreads * kPer + tid; r0 < p.m; r0 += step) {
            float x[kPer];
            int c[kPer];
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const long long r = r0 + u * kFsCutThreads;
                x[u] = r < p.m ? p.v[r] : 0.0f;
                c[u] = prev == 2 && r < p.m ? (int)p.codes[r] : 0;
            }
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const long long r = r0 + u * kFsCutThreads;
                if (r >= p.m) continue;
                const int q = sorted ? nearest_sorted_fast<NLEV>(x[u], s_lev, coarse) : nearest_level_loop(x[u], s_lev, NLEV);
                if (prev == 1)
                    for (int i = 0; i + 1 < NLEV; ++i) c[u] += s_old[i] <= x[u] ? 1 : 0;
                if (q != c[u]) s_changed = 1;
                if (prev == 2 && q == c[u]) continue;
                p.codes[r] = (uint8_t)q;
                if (prev == 2) {
                    add_exact(s_dig + c[u] * kFcCols, -x[u], 1u);
                    atomicAdd(&s_dig[c[u] * kFcCols + kDigits], (unsigned long long)-1ll);
                }
                add_exact(s_dig + q * kFcCols, x[u], 1u);
                atomicAdd(&s_dig[q * kFcCols + kDigits], 1ull);
            }
        }
        __syncthreads();
        unsigned long long* S = (unsigned long long*)p.S;  // (cleared with the first levels)
        for (int e = tid; e < NLEV * kFcCols; e += kFsCutThreads)
            if (s_dig[e]) atomicAdd(&S[e], s_dig[e]);
        if (tid == 0) p.wg_changed[blockIdx.x] = s_changed;
        return;
    }
    if (q + 1 >= NLEV || b < 0) return;
    if (tid < kFcCols) s_dig[tid] = 0ull;
    __syncthreads();
    const int d0 = fs_digit(fs_bound(p, f, b));
    const long long a = f.base[b], n = (long long)f.base[b + 1] - a;
    const long long i0 = a + n * part / kFsParts, i1 = a + n * (part + 1) / kFsParts;
    FsSum s = {0, 0, 0};
    long long cnt = 0;
    const float* __restrict__ w = p.v_hat;
    for (long long r = i0 + tid; r < i1; r += 8 * kFsCutThreads) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = r + u * kFsCutThreads < i1 ? w[r + u * kFsCutThreads] : __builtin_inff();
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (x[u] < t) {
                ++cnt;
                fs_add(s, x[u], d0, s_dig);
            }
    }
    s.a0 = wave_sum_i64(s.a0);
    s.a1 = wave_sum_i64(s.a1);
    s.a2 = wave_sum_i64(s.a2);
    cnt = wave_sum_i64(cnt);
    if (lane == 0) {
        atomicAdd(&s_dig[d0], (unsigned long long)s.a0);
        atomicAdd(&s_dig[d0 + 1], (unsigned long long)s.a1);
        atomicAdd(&s_dig[d0 + 2], (unsigned long long)s.a2);
        atomicAdd(&s_dig[kDigits], (unsigned long long)cnt);
    }
    __syncthreads();
    if (tid < kFcCols) f.cut[((size_t)q * kFsParts + part) * kFcCols + tid] = s_dig[tid];
}

// One workgroup: the launch is a chain of memory round trips, so everything whose address is
// known at the start is loaded in one batch (the tables that place the new thresholds among
// them), and only the sums before a threshold's bucket wait for the bucket's number.  With a
// load after each result, 256 threads: 8.9 us, now 6.5; a whole 4,096,000-scalar call 552 us, now 480.
__global__ __launch_bounds__(kFsThreads) void fs_state_kernel(const FcParams p) {
    __shared__ unsigned long long s_S[kCbqMaxLevels * kFcCols];  // per level boundary, then per level
    __shared__ float s_lev[kCbqMaxLevels], s_spl[kFsBuckets];
    __shared__ unsigned s_cnt[kFsBuckets], s_kmin[kFsBuckets], s_kmax[kFsBuckets];
    __shared__ int s_any, s_unsorted, s_bad;
    const int tid = threadIdx.x, nlev = 1 << p.bits;
    const FsView f = fs_view(p);
    const int done = p.state[kFsDone], updates = p.state[kFsUpdates], prev = p.state[kFsPrev];
    const bool scan = p.state[kFsScan] != 0;
    // (not used after a full scan)
    const float spl = f.spl[tid];
    const unsigned cnt = f.cnt[tid], kmin = f.kmin[tid], kmax = f.kmax[tid];
    auto cut_of = [&](int e, int& tb, unsigned long long (&part)[kFsParts]) {  // e = boundary, column
        const int q = e / kFcCols, c = e - q * kFcCols;
        tb = q + 1 < nlev ? f.tb[q] : -1 - kFsBuckets;
#pragma unroll
        for (int w = 0; w < kFsParts; ++w) part[w] = f.cut[((size_t)q * kFsParts + w) * kFcCols + c];
    };
    int tb0 = -1;
    unsigned long long part0[kFsParts];
#pragma unroll
    for (int w = 0; w < kFsParts; ++w) part0[w] = 0ull;
    if (tid < nlev * kFcCols) cut_of(tid, tb0, part0);
    const unsigned nprev = tid < nlev ? f.nprev[tid] : 0u;
    asm volatile("" ::"v"(spl), "v"(cnt), "v"(kmin), "v"(kmax), "v"(tb0), "v"(nprev), "v"(part0[0]), "v"(part0[kFsParts - 1]));
    if (done) return;
    s_spl[tid] = spl;
    s_cnt[tid] = cnt;
    s_kmin[tid] = kmin;
    s_kmax[tid] = kmax;
    if (tid == 0) s_any = !scan && prev == 0 ? 1 : 0;
    if (tid == 0) s_unsorted = 0;
    __syncthreads();
    if (scan) {
        for (int e = tid; e < nlev * kFcCols; e += kFsThreads) s_S[e] = (unsigned long long)p.S[e];
        for (int w = tid; w < fs_scan_blocks(p); w += kFsThreads)
            if (p.wg_changed[w]) s_any = 1;
        __syncthreads();
    } else {
        // the sums and counts below each threshold (the last boundary: the whole set)
        for (int e = tid; e < nlev * kFcCols; e += kFsThreads) {
            if (e != tid) cut_of(e, tb0, part0);
            const int c = e % kFcCols, b = tb0 < 0 ? -1 - tb0 : tb0;
            unsigned long long t = c == kDigits ? (unsigned long long)f.base[b] : f.pre[(size_t)b * kDigits + c];
            if (tb0 >= 0)
#pragma unroll
                for (int w = 0; w < kFsParts; ++w) t += part0[w];
            s_S[e] = t;
        }
        __syncthreads();
        if (tid + 1 < nlev) {
            const unsigned n = (unsigned)s_S[tid * kFcCols + kDigits];
            if (prev != 0 && nprev != n) s_any = 1;
            f.nprev[tid] = n;
        }
        __syncthreads();
    }
    const bool update = s_any && updates < p.iters;
    if (!update) {  // (uniform)
        if (tid == 0) p.state[kFsDone] = 1;
        return;
    }
    if (tid < nlev) {
        unsigned long long S[kDigits], W = s_S[tid * kFcCols + kDigits];
#pragma unroll
        for (int c = 0; c < kDigits; ++c) S[c] = s_S[tid * kFcCols + c];
        if (!scan && tid > 0) {  // a level's members lie between its two boundaries
            W -= s_S[(tid - 1) * kFcCols + kDigits];
#pragma unroll
            for (int c = 0; c < kDigits; ++c) S[c] -= s_S[(tid - 1) * kFcCols + c];
        }
        const float L = W > 0ull ? (float)(digits_to_double(S) / (double)W) : p.lev[tid];
        s_lev[tid] = L;
        p.lev[tid] = L;
        if (!scan) p.lev_next[tid] = p.thr[tid];  // the thresholds of the codes so far
    }
    __syncthreads();
    if (tid + 1 < nlev && !(s_lev[tid] <= s_lev[tid + 1])) s_unsorted = 1;
    __syncthreads();
    const float t = level_thresholds(p, s_lev, nlev, s_unsorted, &s_bad, p.range[0], p.range[1]);
    __syncthreads();
    const bool ok = s_bad == 0;
    if (!scan && ok && tid + 1 < nlev) f.tb[tid] = fs_place(s_spl, s_cnt, s_kmin, s_kmax, t);
    if (tid == 0) {
        p.state[kFsUpdates] = updates + 1;
        p.state[2] = s_unsorted;
        if (!scan && !ok) p.state[kFsScan] = 1;
        p.state[kFsPrev] = scan ? 2 : 1;
    }
}

// the bucket table of the final thresholds
__global__ __launch_bounds__(kCbqMaxLevels) void fs_table_kernel(const FcParams p) {
    const int tid = threadIdx.x, nlev = 1 << p.bits;
    if (p.state[kFsScan]) return;
    threshold_table(p, tid < nlev ? p.thr[tid] : __builtin_inff(), nlev, true, p.range[0], p.range[1]);
}

// the codes of the final levels, v_hat and the levels
template <int NLEV>
__global__ __launch_bounds__(kFcThreads) void fs_output_kernel(const FcParams p) {
    __shared__ float s_lev[NLEV], s_thr[NLEV];
    __shared__ uint2 s_tbl[kFcBuckets];
    const int tid = threadIdx.x;
    for (int e = tid; e < NLEV; e += kFcThreads) {
        s_lev[e] = p.lev[e];
        s_thr[e] = p.thr[e];
    }
    const bool scan = p.state[kFsScan] != 0, sorted = p.state[2] == 0;
    const float blo = p.range[0], bsc = p.range[3];
    const bool table = bsc > 0.0f;
    if (!scan && table)
        for (int e = tid; e < kFcBuckets; e += kFcThreads) s_tbl[e] = make_uint2(p.tbl[2 * e], p.tbl[2 * e + 1]);
    __syncthreads();
    if (blockIdx.x == 0) {
        for (int e = tid; e < NLEV; e += kFcThreads) p.levels_out[e] = s_lev[e];
        if (tid == 0 && p.rounds_out) *p.rounds_out = p.state[kFsUpdates];
    }
    auto code = [&](float x) {
        if (scan) return sorted ? nearest_sorted(x, s_lev, NLEV) : nearest_level_loop(x, s_lev, NLEV);
        int c = 0, n = NLEV - 1;
        if (table) {
            const uint2 e = s_tbl[fc_bucket(x, blo, bsc)];
            c = (int)(e.x & 255u);
            n = (int)(e.x >> 8);
            if (n <= 1) return c + (__uint_as_float(e.y) <= x ? 1 : 0);
        }
        int q = c;
        for (int j = 0; j < n; ++j) q += s_thr[c + j] <= x ? 1 : 0;
        return q;
    };
    long long r0 = 0;  // scalars from here on: one at a time
    if (((reinterpret_cast<uintptr_t>(p.v) | reinterpret_cast<uintptr_t>(p.v_hat)) & 15u) == 0 &&
        (reinterpret_cast<uintptr_t>(p.codes) & 3u) == 0) {
        constexpr int kPer = 4;  // groups of four scalars in flight
        const long long ng = p.m >> 2;
        const float4* __restrict__ v4 = reinterpret_cast<const float4*>(p.v);
        unsigned* __restrict__ c4 = reinterpret_cast<unsigned*>(p.codes);
        float4* __restrict__ o4 = reinterpret_cast<float4*>(p.v_hat);
        for (long long g0 = (long long)blockIdx.x * kFcThreads * kPer + tid; g0 < ng;
             g0 += (long long)gridDim.x * kFcThreads * kPer) {
            float4 x[kPer];
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const long long g = g0 + (long long)j * kFcThreads;
                x[j] = g < ng ? v4[g] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const long long g = g0 + (long long)j * kFcThreads;
                if (g >= ng) continue;
                const int a = code(x[j].x), b = code(x[j].y), c = code(x[j].z), d = code(x[j].w);
                c4[g] = (unsigned)a | (unsigned)b << 8 | (unsigned)c << 16 | (unsigned)d << 24;
                o4[g] = make_float4(s_lev[a], s_lev[b], s_lev[c], s_lev[d]);
            }
        }
        r0 = 4 * ng;
    }
    for (long long r = r0 + (long long)blockIdx.x * kFcThreads + tid; r < p.m; r += (long long)gridDim.x * kFcThreads) {
        const int q = code(p.v[r]);
        p.codes[r] = (uint8_t)q;
        p.v_hat[r] = s_lev[q];
    }
}

// whether a set takes the partitioned rounds: unweighted, with a v_hat of its own for the
// partitioned copy, room for the tables, and large enough (or thresholds asked for), with rounds
// enough to pay for the partition.  300,000 scalars take 492 us by the exact search, which the
// partition does not reach.  What the partition costs and a round then saves, 6 bits: 786,432 scalars
// 86 and 10 us, 1,000,003: 80 and 11, 4,096,000: 82 and 16, 20,000,000: 133 and 28, 100,000,000: 410 and
// 103 us; at 3 bits a round of the two smaller sets saves 6.5, at 8 bits 4.5 to 6.5 us.  The rounds asked for
// lie where both are about even over the widths: 12, 7 from 2^21 scalars on, 5 from 2^24 (1,000,003
// scalars at one round 125 us partitioned, 54 otherwise; at 15 rounds 275 and 343).  A set that converges
// sooner still pays: one round of 30, 20,000,000 scalars on a grid of 255 values, 435 us for 388.
constexpr long long kFsMin = 3ll << 18;
int fs_min_rounds(long long m) { return m < 1ll << 21 ? 12 : m < 1ll << 24 ? 7 : 5; }
bool fs_usable(const FcParams& p) {
    if (p.w != nullptr || p.v_hat == nullptr || p.thr_mode == 1 || p.bits < 3) return false;
    if (p.thr_mode == 0 && (p.m < kFsMin || p.iters < fs_min_rounds(p.m))) return false;
    const char *v = (const char*)p.v, *o = (const char*)p.v_hat;
    const long long nb = p.m * (long long)sizeof(float);
    if (v < o + nb && o < v + nb) return false;  // in place
    return fs_view(p).bytes <= sizeof(long long) * (size_t)fc_grid(p.m) * ((size_t)1 << p.bits) * kFcCols;
}

hipError_t launch_fs_quantize(const FcParams& set, hipStream_t s) {
    FcParams p = set;
    p.G = fc_grid(p.m);
    p.bucketed = 1;
    FcStack<1> st;
    st.L[0] = p;
    const int nlev = 1 << p.bits;
    const long long tiles = (p.m + kFsTile - 1) / kFsTile;
    const int Gt = (int)(tiles < 256 ? tiles : 256), Gs = 2 * p.G;
    hipError_t e = hipSuccess;
    auto run = [&](auto kernel, int grid, int threads, const auto& arg) {
        if (e != hipSuccess) return;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, s, arg);
        e = hipGetLastError();
    };
    run(fs_split_kernel, 1, kFsThreads, p);
    run(fs_hist_kernel, Gt, kFsThreads, p);
    st.L[0].G = Gt;  // the minima and maxima are those of fs_hist_kernel's workgroups
    run(fc_grid_kernel<1>, 1, kCbqMaxLevels, st);
    run(fs_base_kernel, 1, kFsThreads, p);
    run(fs_scatter_kernel, Gt, kFsThreads, p);
    run(fs_sum_kernel, Gs, kFsCutThreads, p);
    run(fs_prefix_kernel, 1, kFsThreads, p);
    auto rounds = [&](auto lev) {
        constexpr int NLEV = decltype(lev)::value;
        for (int r = 0; r < p.iters; ++r) {
            run(fs_cut_kernel<NLEV>, nlev * kFsParts, kFsCutThreads, p);
            run(fs_state_kernel, 1, kFsThreads, p);
        }
        run(fs_table_kernel, 1, kCbqMaxLevels, p);
        run(fs_output_kernel<NLEV>, p.G, kFcThreads, p);
    };
    switch (p.bits) {
        case 3: rounds(std::integral_constant<int, 8>{}); break;
        case 4: rounds(std::integral_constant<int, 16>{}); break;
        case 5: rounds(std::integral_constant<int, 32>{}); break;
        case 6: rounds(std::integral_constant<int, 64>{}); break;
        case 7: rounds(std::integral_constant<int, 128>{}); break;
        case 8: rounds(std::integral_constant<int, 256>{}); break;
        default: return hipErrorInvalidValue;
    }
    return e;
}

hipError_t launch_fc_quantize(const FcParams* sets, int n, hipStream_t s) {
    if (n == 1 && fs_usable(sets[0])) return launch_fs_quantize(sets[0], s);
    return n == 1 ? launch_fc_sets<1>(sets, 1, s) : launch_fc_sets<KQ_MAX_STACK>(sets, n, s);
}

hipError_t launch_cbq(const CbqParams& p, hipStream_t s) {
    int mmax = 0;
    for (int l = 0; l < p.nlayers; ++l) mmax = p.L[l].k * kDim > mmax ? p.L[l].k * kDim : mmax;
    const bool fast = p.bits == 6;
    if (mmax <= kCbqLdsScalars && fast)
        hipLaunchKernelGGL((cbq_kernel<true, true>), dim3(p.nlayers), dim3(kCbqThreads), 0, s, p);
    else if (mmax <= kCbqLdsScalars)
        hipLaunchKernelGGL((cbq_kernel<true, false>), dim3(p.nlayers), dim3(kCbqThreads), 0, s, p);
    else if (fast)
        hipLaunchKernelGGL((cbq_kernel<false, true>), dim3(p.nlayers), dim3(kCbqThreads), 0, s, p);
    else
        hipLaunchKernelGGL((cbq_kernel<false, false>), dim3(p.nlayers), dim3(kCbqThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace kq
