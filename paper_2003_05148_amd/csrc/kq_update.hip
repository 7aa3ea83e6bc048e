// Update step of kernel-level quantization (Sec. 3.1, Eq. 1): every codebook entry
// becomes the mean of its kernel set S_j; an empty set keeps its entry.
//
// The member sums are exact integers: each value is mapped to q(x) = rint(x * 2^s) with a
// per-layer shift s = min(62 - ceil(log2 n), 51) - e, max |x| < 2^e, so |q| <= 2^62 / n
// and no sum over at most n kernels can overflow int64, at any magnitude of the weights
// (each q is added as kFixedBias + q, the bit pattern of one fp64 fma, and the finish
// takes count * kFixedBias back off).
// Integer addition is associative, so the sums, and with them the new codebook, do not
// depend on the order in which blocks or lanes add.  absmax_kernel takes the maxima of |x|
// per block of 32768 values, once per call or once per fit, before any sum is formed; with a
// range check shift_kernel turns them into each layer's s (and flags non-finite values),
// otherwise the first launch that forms sums does (derive_shift: every workgroup takes the
// layer's largest block maximum, one of them stores s for the launches after).
//
// update_kernel: one launch covers every layer of a stack.  A layer's kernels are cut
// into chunks and its codebook into ranges of at most 768 entries; a workgroup of 1024
// threads takes one (chunk, range) pair: it reads the chunk's indices, one 36-byte row per
// thread and step (consecutive lanes, consecutive rows, two steps in flight; with several
// ranges it lists the range's members first: add_listed), loads the
// rows whose entry lies in its range and adds them to a private LDS histogram of the range
// ([768][9] int64 sums + [768] counts at most, ds_add_u64), then stores the histogram
// into the chunk's partial ([chunks][k][10] int64).  Chunk sizes give about one workgroup
// per CU for the whole launch.  The LDS atomics, not the loads, bound it: a layout with
// fully coalesced dword loads, where each float fetched its kernel's entry with
// ds_bpermute, added LDS work and ran slower.  Asked for the distortion of a standalone
// assignment, it also sums, in a fixed order, the fp32 distances of its rows to their old
// entries.
// Codebook gradient step (Eq. 2): the same sums over a gradient tensor G instead of the
// kernels, with the same shift rule applied to max |g|; the finish then writes
// c - gamma * mean instead of the mean.
// update_finish_kernel: a workgroup of 960 threads owns 16 entries of one layer; six
// groups of 160 threads add a sixth of the partials each, nine loads in flight per thread
// (one batch for the 54 partials of the largest ResNet-18 layers; any order gives the same
// integers), then it divides and writes the codebook and the counts.  Fewer, fuller
// workgroups measured faster: the launch is short, and the workgroups dispatched last
// start up to 2 us after the first (528 workgroups of 640 threads at 8 entries each; 2
// or 4 entries each were slower still).  One more workgroup per layer adds the distortion
// partials in a fixed order with its first 640 threads (those of the assignment kernel
// when the distortion comes from there).  The kernel boundary orders every partial before
// its use, so no fence or atomic counter is needed.
#include "kq_internal.h"

namespace kq {

__device__ __forceinline__ float sqdist9u(const float* x, const float* __restrict__ c) {
    float acc = 0.0f;
#pragma unroll
    for (int d = 0; d < kDim; ++d) {
        const float t = x[d] - c[d];
        acc = __fmaf_rn(t, t, acc);
    }
    return acc;
}

// the nine values of a row
__device__ __forceinline__ void mem_row_of(float (&x)[kDim], const float* __restrict__ r) {
#pragma unroll
    for (int d = 0; d < kDim; ++d) x[d] = r[d];
}

struct UpdateCtx {
    unsigned long long* s_sum;  // [krange][9]
    unsigned* s_cnt;            // [krange]
    const float* C_old;
    double scale;               // 2^s of q(x) = rint(x * 2^s)
    int j0, kr;                 // the entry range [j0, j0 + kr)
    bool sums, want_dist;
};

// add one kernel (row x, entry j) to the histogram if j is in the range
__device__ __forceinline__ void add_kernel(const UpdateCtx& c, const float (&x)[kDim], int j, double& dacc) {
    const int jr = j - c.j0;
    if ((unsigned)jr >= (unsigned)c.kr) return;
    if (c.want_dist) dacc += (double)sqdist9u(x, c.C_old + (size_t)j * kDim);
    atomicAdd(&c.s_cnt[jr], 1u);
    if (c.sums) {
#pragma unroll
        for (int d = 0; d < kDim; ++d) atomicAdd(&c.s_sum[jr * kDim + d], fixed_bits(x[d], c.scale));
    }
}

// Thread t takes kernels i, i + 1024, ... (i = first + t): consecutive lanes read
// consecutive 36-byte rows with 9 dword loads each, two kernels in flight per thread; a row
// is loaded only when its entry lies in the workgroup's range (with a single range every
// row is, and the row loads need not wait for the indices).
template <bool NEED_X, bool RANGED>
__device__ __forceinline__ void add_rows(const UpdateCtx& c, const float* __restrict__ X,
                                         const int32_t* __restrict__ idx, int i, int i1, double& dacc) {
    for (; i < i1; i += 2 * kUpdateThreads) {
        const int ib = i + kUpdateThreads;
        const bool two = ib < i1;
        const int ja = idx[i], jb = two ? idx[ib] : -1;  // -1: nothing to add
        const bool ina = !RANGED || (unsigned)(ja - c.j0) < (unsigned)c.kr;
        const bool inb = !RANGED || (unsigned)(jb - c.j0) < (unsigned)c.kr;
        float xa[kDim], xb[kDim];
        if (NEED_X) {
            const float* pa = X + (size_t)i * kDim;
            const float* pb = X + (size_t)(two ? ib : i) * kDim;
#pragma unroll
            for (int d = 0; d < kDim; ++d) {
                xa[d] = ina ? pa[d] : 0.0f;
                xb[d] = inb ? pb[d] : 0.0f;
            }
        } else {
#pragma unroll
            for (int d = 0; d < kDim; ++d) xa[d] = xb[d] = 0.0f;
        }
        add_kernel(c, xa, ja, dacc);
        add_kernel(c, xb, jb, dacc);
    }
}

// One of several ranges: few rows of a wave lie in it, so the members are listed first and their
// values then added densely, one per lane (consecutive lanes read a member's row).  kTileKernels
// indices at a time; list entries are the kernel's place in the tile | entry of the range << 16.
// Whole passes, a row per thread and step before: the VGG-16 stack with k = 60 .. 1088 3452 us,
// listed 3309; the ResNet-18 stack with k = 609 .. 7679 12.61 and 12.20 ms; 1,048,576 kernels, k =
// 4096, 10 rounds 2918 and 2835 us.  Two barriers a tile and the gathers of 36-byte pieces bound it
// (a launch on these stacks 24 and 53 us before, now 16 and 31).
constexpr int kTileBatch = 4;
constexpr int kTileKernels = kTileBatch * kUpdateThreads;
constexpr int kValueBatch = 8;  // values in flight per thread
__device__ __forceinline__ void add_listed(const UpdateCtx& c, const float* __restrict__ X, const int32_t* __restrict__ idx,
                                           int i0, int i1, unsigned* s_list, unsigned* s_n) {
    const int tid = threadIdx.x, lane = tid & 63;
    int j[kTileBatch];
    auto load = [&](int t0) {
#pragma unroll
        for (int u = 0; u < kTileBatch; ++u) {
            const int o = u * kUpdateThreads + tid;
            j[u] = o < i1 - t0 ? idx[t0 + o] : -1;
        }
    };
    load(i0);
    int par = 0;  // the counter of this tile; the other one is cleared for the next
    for (int t0 = i0; t0 < i1; par ^= 1) {  // (uniform; the counters start at zero)
        if (tid == 0) s_n[par ^ 1] = 0u;
        unsigned before[kTileBatch], total = 0u;
        bool in[kTileBatch];
#pragma unroll
        for (int u = 0; u < kTileBatch; ++u) {
            in[u] = (unsigned)(j[u] - c.j0) < (unsigned)c.kr;
            const unsigned long long m = __ballot(in[u]);
            before[u] = total + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            total += (unsigned)__popcll(m);
        }
        unsigned at = 0u;
        if (lane == 0 && total) at = atomicAdd(&s_n[par], total);
        at = (unsigned)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
        for (int u = 0; u < kTileBatch; ++u)
            if (in[u]) {
                const unsigned jr = (unsigned)(j[u] - c.j0);
                s_list[at + before[u]] = (unsigned)(u * kUpdateThreads + tid) | jr << 16;
                atomicAdd(&c.s_cnt[jr], 1u);
            }
        const float* __restrict__ Xt = X + (size_t)t0 * kDim;
        const bool more = i1 - t0 > kTileKernels;
        if (more) load(t0 + kTileKernels);  // in flight while this tile is added
        __syncthreads();
        const unsigned nv = s_n[par] * kDim;
        for (unsigned v0 = (unsigned)tid; v0 < nv; v0 += kValueBatch * kUpdateThreads) {
            float x[kValueBatch];
            unsigned e[kValueBatch];
#pragma unroll
            for (int u = 0; u < kValueBatch; ++u) {
                const unsigned v = v0 + u * kUpdateThreads;
                if (v < nv) {
                    const unsigned m = v / kDim, q = v - m * kDim, w = s_list[m];
                    x[u] = Xt[(w & 0xffffu) * kDim + q];
                    e[u] = (w >> 16) * kDim + q;
                }
            }
#pragma unroll
            for (int u = 0; u < kValueBatch; ++u)
                if (v0 + u * kUpdateThreads < nv) atomicAdd(&c.s_sum[e[u]], fixed_bits(x[u], c.scale));
        }
        if (!more) break;
        t0 += kTileKernels;
        __syncthreads();  // the list is free
    }
}

__global__ __launch_bounds__(kUpdateThreads) void update_kernel(const StackParams p) {
    extern __shared__ unsigned long long s_dyn[];  // [krange][9] sums, then [krange] u32 counts
    __shared__ unsigned s_list[kTileKernels], s_n[2];
    __shared__ double s_wd[kUpdateThreads / kWave];
    __shared__ unsigned s_mx;

    const int li = find_layer(p, blockIdx.x);
    const DevLayer& L = p.L[li];
    const int u = blockIdx.x - L.unit_begin;
    const int chunk = u / L.ranges, range = u - chunk * L.ranges;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = L.n, k = L.k;
    UpdateCtx c;
    c.j0 = range * L.krange;
    c.kr = min(k - c.j0, L.krange);
    c.s_sum = s_dyn;
    c.s_cnt = (unsigned*)(s_dyn + (size_t)c.kr * kDim);
    c.C_old = L.C_old;
    c.sums = (L.flags & kFlagCountsOnly) == 0;
    int shift = 0;
    if (c.sums) {  // set by shift_kernel before this launch, or formed here from the block maxima
        if (p.derive_shift) {
            shift = derive_shift<kUpdateThreads>(L, &s_mx);
            if (u == 0 && tid == 0) L.xmax[L.nxmax] = (unsigned)shift;  // for the launches after
        } else {
            shift = (int)L.xmax[L.nxmax];
        }
    }
    c.scale = fixed_scale(shift);
    c.want_dist = L.part != nullptr;
    const bool need_x = c.sums || c.want_dist;

    for (int e = tid; e < c.kr * kDim; e += kUpdateThreads) c.s_sum[e] = 0ull;
    for (int e = tid; e < c.kr; e += kUpdateThreads) c.s_cnt[e] = 0u;
    if (tid < 2) s_n[tid] = 0u;
    __syncthreads();

    double dacc = 0.0;
    const int i0 = chunk * L.chunk;
    const int i1 = min(n, i0 + L.chunk);
    if (!need_x)
        add_rows<false, false>(c, L.X, L.idx, i0 + tid, i1, dacc);
    else if (L.ranges == 1)
        add_rows<true, false>(c, L.X, L.idx, i0 + tid, i1, dacc);
    else if (c.want_dist)  // (the distances are added in the order of the rows)
        add_rows<true, true>(c, L.X, L.idx, i0 + tid, i1, dacc);
    else
        add_listed(c, L.X, L.idx, i0, i1, s_list, s_n);

    __syncthreads();
    unsigned long long* __restrict__ out = (unsigned long long*)L.hist + ((size_t)chunk * k + c.j0) * 10;
    for (int e = tid; e < c.kr * 10; e += kUpdateThreads) {
        const int j = e / 10, d = e - 10 * j;
        out[e] = (d == 9) ? (unsigned long long)c.s_cnt[j] : c.s_sum[j * kDim + d];
    }
    if (c.want_dist) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) dacc += __shfl_xor(dacc, off);
        if (lane == 0) s_wd[wave] = dacc;
        __syncthreads();
        if (tid == 0) {
            double v = s_wd[0];
            for (int w = 1; w < kUpdateThreads / kWave; ++w) v += s_wd[w];
            L.part[u] = v;
        }
    }
}

constexpr int kFinishGroups = 6;
constexpr int kFinishBatch = 9;
constexpr int kFinishDirectWgs = 16;  // workgroups per layer in the direct form
constexpr int kFinishDirectK = kFinishDirectWgs * kFinishEntries;  // 256
constexpr int kFinishThreads = kFinishEntries * 10 * kFinishGroups;  // 960
static_assert(kFinishThreads >= kSumThreads, "the distortion sum uses the first kSumThreads threads");

// GROUPS 6: six threads share a value's partials, 16 entries per workgroup.  GROUPS 1: one thread
// per value, 96 entries per workgroup.
template <int GROUPS>
__global__ __launch_bounds__(kFinishThreads) void update_finish_kernel(const StackParams p) {
    constexpr int kE = kFinishEntries * kFinishGroups / GROUPS;  // entries per workgroup
    __shared__ unsigned long long s_S[GROUPS][kE * 10];
    __shared__ double s_w[kSumThreads / kWave];
    const int b = blockIdx.x;
    // The launch is short, and every dependent load of the arguments is a memory round trip.
    // With every codebook of at most kFinishDirectK entries (p.finish_direct) layer l owns
    // workgroups kFinishDirectWgs l .., so the fields of layer b / kFinishDirectWgs are read in
    // the first batch; otherwise the table of first workgroups gives the layer and its fields
    // come in later batches.
    const int ld = min(b / kFinishDirectWgs, KQ_MAX_STACK - 1);
    const DevLayer& Ld = p.L[ld];
    int k = Ld.k, nb = Ld.nchunks, flags = Ld.flags, nx = Ld.nxmax, ub = Ld.unit_begin;
    const unsigned long long* __restrict__ h = (const unsigned long long*)Ld.hist;
    const unsigned* xm = Ld.xmax;
    const float* C_old = Ld.C_old;
    const int total = p.total_units, direct = p.finish_direct;
    asm volatile("" ::"s"(k), "s"(nb), "s"(flags), "s"(nx), "s"(ub), "s"(h), "s"(xm), "s"(C_old), "s"(total),
                 "s"(direct));
    if (b >= total) {  // the last nlayers workgroups: the distortion of layer b - total
        const DevLayer& L = p.L[b - total];
        double* const dist = L.dist;
        const double *const ap = L.apart, *const pp = L.part;
        const int na = L.napart, nu = L.nunits;
        asm volatile("" ::"s"(dist), "s"(ap), "s"(pp), "s"(na), "s"(nu));
        const double* const src = ap ? ap : pp;
        const int m = ap ? na : nu;
        if (dist == nullptr) return;
        const double a = block_fixed_sum<kSumThreads>(src, m, s_w);
        if (threadIdx.x == 0) *dist = a;
        return;
    }
    const int lt = direct ? ld : find_layer(p, b);  // the layer
    const int li = lt;
    if (!direct) {  // layer and entry range from the table: each layer owns ceil(k / kE) workgroups
        const DevLayer& Lt = p.L[lt];
        k = Lt.k;
        nb = Lt.nchunks;
        flags = Lt.flags;
        nx = Lt.nxmax;
        ub = Lt.unit_begin;
        h = (const unsigned long long*)Lt.hist;
        xm = Lt.xmax;
        C_old = Lt.C_old;
    }
    const DevLayer& L = p.L[li];
    const int j0 = (b - ub) * kE;
    const int tid = threadIdx.x;
    const int g = tid / (kE * 10), v = tid - g * (kE * 10);
    const int j = j0 + v / 10, d = v - 10 * (v / 10);
    // the entry's old value and the layer's shift, in flight with the partials
    const bool writes_c = g == 0 && j < k && d < kDim && (flags & kFlagCountsOnly) == 0;
    float old = 0.0f;
    int shift = 0;
    if (writes_c) {
        old = C_old[(size_t)j * kDim + d];
        shift = (int)xm[nx];
    }

    unsigned long long s = 0ull;
    if (j < k) {
        const size_t stride = (size_t)k * 10;
        const unsigned long long* hp = h + (size_t)j * 10 + d;
        // partials g, g + GROUPS, ...: kFinishBatch loads in flight at a time
#pragma unroll 1
        for (int q0 = g; q0 < nb; q0 += kFinishBatch * GROUPS) {
            unsigned long long v[kFinishBatch];
#pragma unroll
            for (int r = 0; r < kFinishBatch; ++r) {
                const int q = q0 + r * GROUPS;
                v[r] = q < nb ? hp[(size_t)q * stride] : 0ull;
            }
#pragma unroll
            for (int r = 0; r < kFinishBatch; ++r) s += v[r];
        }
    }
    s_S[g][v] = s;
    __syncthreads();
    if (g == 0 && j < k) {
        unsigned long long S = 0, z = 0;  // wrapping sums
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
            S += s_S[q][v];
            z += s_S[q][(v / 10) * 10 + 9];
        }
        S -= z * kFixedBias;  // the exact sum of q(x) over the entry's kernels
        if (d == 9) {
            if (L.counts) L.counts[j] = (int32_t)z;
        } else if (writes_c) {
            float c = old;
            if (z > 0) {
                const double mean = ((double)(long long)S * ldexp(1.0, -shift)) / (double)z;
                // Eq. (2): c - gamma * mean gradient; Eq. (1): the mean of the kernels
                c = (flags & kFlagGrad) ? (float)((double)old - (double)L.gamma * mean) : (float)mean;
            }
            L.C[(size_t)j * kDim + d] = c;
        }
    }
}

// The whole update of layers of at most kUpdateSmallN kernels in one launch: a workgroup owns 16
// entries, reads all of the layer's indices, lists its members in LDS, adds their rows (one value
// per thread: the list is dense) to LDS sums and finishes its entries.  Every workgroup reads the
// indices again (k / 16 times 4 n bytes: 1.2 MB at n = 4096, k = 1228), which costs less than the
// partials and the second launch of the general path: 4096 kernels, k = 700: 5.1 + 3.8 us and the
// gap between them, now 4.3 us.  An entry with most of the kernels (a pruned layer's zeros) leaves its
// workgroup alone with them: the list is built by ballots, and from kHeavyMembers members on a sample of
// it tells the most frequent entry, whose rows are then added in registers, a row per thread.  A fit of
// 16384 kernels, 20 rounds, none, half and 90 % of them zero: k = 256 with LDS atomics per member and
// value 308, 652 and 942 us, now 305, 432 and 459 (member sums fused into the assignment 350 us all
// three); k = 1000 335, 683 and 988, now 333, 475 and 498 (update and finish 402).  The last nlayers
// workgroups add the distortion partials.
constexpr int kSmallThreads = 1024;
constexpr int kHeavyMembers = 3072;
__global__ __launch_bounds__(kSmallThreads, 8) void update_small_kernel(const StackParams p) {
    __shared__ unsigned s_list[kUpdateSmallN];  // kernel | entry of the workgroup << 16
    __shared__ unsigned long long s_sum[kFinishEntries * kDim];
    __shared__ unsigned s_cnt[kFinishEntries];
    __shared__ unsigned s_n, s_mx;
    __shared__ double s_w[kSumThreads / kWave];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1);
    if (b >= p.total_units) {  // the distortion of layer b - total
        const DevLayer& L = p.L[b - p.total_units];
        if (L.dist == nullptr) return;
        const double a = block_fixed_sum<kSumThreads>(L.apart, L.napart, s_w);
        if (tid == 0) *L.dist = a;
        return;
    }
    const DevLayer& L = p.L[find_layer(p, b)];
    const int n = L.n, k = L.k, flags = L.flags, j0 = (b - L.unit_begin) * kFinishEntries;
    const int32_t* __restrict__ idx = L.idx;
    const float* __restrict__ X = L.X;
    const bool sums = (flags & kFlagCountsOnly) == 0;
    constexpr int kBatch = 8;
    int jb[kBatch];  // the first indices, in flight with the shift
#pragma unroll
    for (int u = 0; u < kBatch; ++u) jb[u] = tid + u * kSmallThreads < n ? idx[tid + u * kSmallThreads] : -1;
    int shift = 0;
    if (sums) {
        if (p.derive_shift) {
            shift = derive_shift<kSmallThreads>(L, &s_mx);
            if (j0 == 0 && tid == 0) L.xmax[L.nxmax] = (unsigned)shift;  // for the launches after
        } else {
            shift = (int)L.xmax[L.nxmax];
        }
    }
    const int e = tid / 10, d = tid - 10 * e, j = j0 + e;  // the value this thread finishes (tid < 160)
    const bool mine = tid < kFinishEntries * 10 && j < k;
    const float old = mine && d < kDim && sums ? L.C_old[(size_t)j * kDim + d] : 0.0f;
    if (tid < kFinishEntries * kDim) s_sum[tid] = 0ull;
    if (tid < kFinishEntries) s_cnt[tid] = 0u;
    if (tid == 0) s_n = 0u;
    __syncthreads();
    for (int i0 = 0; i0 < n; i0 += kBatch * kSmallThreads) {  // (uniform)
        if (i0 != 0) {
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int i = i0 + u * kSmallThreads + tid;
                jb[u] = i < n ? idx[i] : -1;
            }
        }
        unsigned before[kBatch], found = 0u;
        bool in[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            in[u] = (unsigned)(jb[u] - j0) < (unsigned)kFinishEntries && jb[u] < k;  // (others are ignored)
            const unsigned long long m = __ballot(in[u]);
            before[u] = found + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            found += (unsigned)__popcll(m);
        }
        unsigned at = 0u;
        if (lane == 0 && found) at = atomicAdd(&s_n, found);
        at = (unsigned)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (in[u]) s_list[at + before[u]] = (unsigned)(i0 + u * kSmallThreads + tid) | (unsigned)(jb[u] - j0) << 16;
    }
    __syncthreads();
    const int total = (int)s_n;
    const double scale = fixed_scale(shift);
    int heavy = -1;  // an entry with at least a quarter of many members
    if (total >= kHeavyMembers) {
        const unsigned own = s_list[(unsigned)lane * (unsigned)total / kWave] >> 16;
        int most = kWave / 4 - 1;
#pragma unroll
        for (int q = 0; q < kFinishEntries; ++q) {
            const int c = __popcll(__ballot(own == (unsigned)q));
            heavy = c > most ? q : heavy;
            most = c > most ? c : most;
        }
    }
    if (heavy < 0) {
        for (int m = tid; m < total; m += kSmallThreads) atomicAdd(&s_cnt[s_list[m] >> 16], 1u);
        if (sums)
            for (unsigned v = tid; v < (unsigned)total * kDim; v += kSmallThreads) {
                const unsigned m = v / kDim, q = v - m * kDim, w = s_list[m];
                atomicAdd(&s_sum[(w >> 16) * kDim + q], fixed_bits(X[(size_t)(w & 0xffffu) * kDim + q], scale));
            }
    } else {
        long long acc[kDim];
        unsigned z = 0u;
#pragma unroll
        for (int q = 0; q < kDim; ++q) acc[q] = 0;
        constexpr int kRows = 2;  // rows in flight per thread
        for (int m0 = tid; m0 < total; m0 += kRows * kSmallThreads) {
            unsigned w[kRows];
            float x[kRows][kDim];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const int m = m0 + u * kSmallThreads;
                w[u] = s_list[m < total ? m : m0];
                if (sums) mem_row_of(x[u], X + (size_t)(w[u] & 0xffffu) * kDim);
            }
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                if (m0 + u * kSmallThreads >= total) continue;
                const unsigned jr = w[u] >> 16;
                if ((int)jr == heavy) {
                    ++z;
                    if (sums)
#pragma unroll
                        for (int q = 0; q < kDim; ++q) acc[q] += (long long)fixed_bits(x[u][q], scale);
                } else {
                    atomicAdd(&s_cnt[jr], 1u);
                    if (sums)
#pragma unroll
                        for (int q = 0; q < kDim; ++q) atomicAdd(&s_sum[jr * kDim + q], fixed_bits(x[u][q], scale));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < kDim; ++q) acc[q] = wave_sum_i64(acc[q]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) z += (unsigned)__shfl_xor((int)z, off);
        if (lane == 0) {
            atomicAdd(&s_cnt[heavy], z);
#pragma unroll
            for (int q = 0; q < kDim; ++q) atomicAdd(&s_sum[heavy * kDim + q], (unsigned long long)acc[q]);
        }
    }
    __syncthreads();
    if (!mine) return;
    const unsigned z = s_cnt[e];
    if (d == 9) {
        if (L.counts) L.counts[j] = (int32_t)z;
    } else if (sums) {
        const unsigned long long S = s_sum[e * kDim + d] - (unsigned long long)z * kFixedBias;
        L.C[(size_t)j * kDim + d] = z > 0 ? (float)(((double)(long long)S * ldexp(1.0, -shift)) / (double)z) : old;
    }
}

hipError_t launch_update_small(const StackParams& p, hipStream_t s) {
    StackParams q = p;
    int blk = 0;
    for (int l = 0; l < q.nlayers; ++l) {
        q.L[l].unit_begin = blk;
        blk += (q.L[l].k + kFinishEntries - 1) / kFinishEntries;
    }
    q.total_units = blk;  // followed by one workgroup per layer for the distortion
    set_unit_table(q);
    hipLaunchKernelGGL(update_small_kernel, dim3(blk + q.nlayers), dim3(kSmallThreads), 0, s, q);
    return hipGetLastError();
}

// per-block maximum of |v| over 32768 values of a layer (the kernels, or the gradients of
// Eq. 2) as fp32 bits with the sign cleared: an integer maximum, so a NaN counts as the
// largest value and shift_kernel can flag it.  Blocks of 1024 threads: a grid of many small
// workgroups is slow to dispatch (the last start microseconds after the first)
__global__ __launch_bounds__(kAbsMaxThreads) void absmax_kernel(const StackParams p) {
    __shared__ unsigned s_mx;
    const int li = find_layer(p, blockIdx.x);
    const DevLayer& L = p.L[li];
    const int b = blockIdx.x - L.unit_begin;
    const long long count = (long long)L.n * kDim;
    const long long base = (long long)b * kAbsMaxPerBlock;
    if (threadIdx.x == 0) s_mx = 0u;
    __syncthreads();
    unsigned m = 0u;
    const unsigned* __restrict__ V = reinterpret_cast<const unsigned*>(L.X);
    if ((reinterpret_cast<uintptr_t>(L.X) & 15u) == 0 && base + kAbsMaxPerBlock <= count) {
        // a whole block from a 16-byte aligned tensor: eight 16-byte loads per thread in flight
        const uint4* __restrict__ V4 = reinterpret_cast<const uint4*>(V + base);
        constexpr int kPer = kAbsMaxPerBlock / (4 * kAbsMaxThreads);
        uint4 v[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) v[u] = V4[threadIdx.x + kAbsMaxThreads * u];
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            m = max(m, max(max(v[u].x & 0x7fffffffu, v[u].y & 0x7fffffffu), max(v[u].z & 0x7fffffffu, v[u].w & 0x7fffffffu)));
    } else {
#pragma unroll 4
        for (int q = threadIdx.x; q < kAbsMaxPerBlock; q += kAbsMaxThreads) {
            const long long e = base + q;
            if (e < count) m = max(m, V[e] & 0x7fffffffu);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, off));
    if ((threadIdx.x & 63) == 0) atomicMax(&s_mx, m);  // LDS
    __syncthreads();
    if (threadIdx.x == 0) L.xmax[b] = s_mx;
}

// one workgroup per layer: the largest of its block maxima gives the layer's shift
// (xmax[nxmax]); range_flags[layer] records whether any value was NaN or infinite
__global__ __launch_bounds__(256) void shift_kernel(const StackParams p) {
    __shared__ unsigned s_mx;
    const DevLayer& L = p.L[blockIdx.x];
    if (threadIdx.x == 0) s_mx = 0u;
    __syncthreads();
    unsigned m = 0u;
    for (int q = threadIdx.x; q < L.nxmax; q += 256) m = max(m, L.xmax[q]);
    atomicMax(&s_mx, m);  // LDS
    __syncthreads();
    if (threadIdx.x == 0) {
        L.xmax[L.nxmax] = (unsigned)layer_shift(s_mx, L.shift);
        if (p.range_flags) p.range_flags[blockIdx.x] = s_mx >= 0x7f800000u ? 1u : 0u;
    }
}

hipError_t launch_absmax(const StackParams& p, hipStream_t s, bool with_shift) {
    StackParams q = p;
    int blk = 0;
    for (int l = 0; l < q.nlayers; ++l) {
        q.L[l].unit_begin = blk;
        blk += q.L[l].nxmax;
    }
    q.total_units = blk;
    set_unit_table(q);
    hipLaunchKernelGGL(absmax_kernel, dim3(blk), dim3(kAbsMaxThreads), 0, s, q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !with_shift) return e;
    hipLaunchKernelGGL(shift_kernel, dim3(q.nlayers), dim3(256), 0, s, q);
    return hipGetLastError();
}

__global__ void fill_zero_kernel(uint4* p, size_t n16, unsigned char* tail, size_t ntail) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n16; e += stride) p[e] = make_uint4(0, 0, 0, 0);
    if (blockIdx.x == 0)
        for (size_t e = threadIdx.x; e < ntail; e += blockDim.x) tail[e] = 0;
}

hipError_t launch_update(const StackParams& p, hipStream_t s) {
    size_t lds = 0;
    for (int l = 0; l < p.nlayers; ++l) {
        const size_t b = (size_t)p.L[l].krange * (kDim * sizeof(unsigned long long) + sizeof(unsigned));
        lds = b > lds ? b : lds;
    }
    hipLaunchKernelGGL(update_kernel, dim3(p.total_units), dim3(kUpdateThreads), lds, s, p);
    return hipGetLastError();
}

// The finishing launch numbers its workgroups per layer: ceil(k / entries) each.  Where 16 entries
// a workgroup would make more workgroups than the chip holds twice over and a value has few
// partials, one thread adds them all and a workgroup takes 96 entries (the ResNet-18 stack with
// k = 609 .. 7679, 3462 workgroups of 960 threads: 18.7 us a launch, now 8.8; the whole compression pass
// 12.00 ms, now 11.67; a single k = 4096 layer, 256 workgroups, 6.9 us, stays with six threads).
constexpr int kFinishManyWgs = 1024, kFinishFewPartials = 2 * kFinishBatch;
hipError_t launch_update_finish(const StackParams& p, hipStream_t s) {
    StackParams q = p;
    bool direct = true;  // every codebook fits kFinishDirectWgs workgroups
    for (int l = 0; l < q.nlayers; ++l) direct &= q.L[l].k <= kFinishDirectK;
    q.finish_direct = direct ? 1 : 0;
    int wgs = 0, most = 0;
    for (int l = 0; l < q.nlayers; ++l) {
        wgs += (q.L[l].k + kFinishEntries - 1) / kFinishEntries;
        most = q.L[l].nchunks > most ? q.L[l].nchunks : most;
    }
    const bool wide = wgs > kFinishManyWgs && most <= kFinishFewPartials;  // (then not direct: that has at most 256)
    const int per = wide ? kFinishEntries * kFinishGroups : kFinishEntries;
    int blk = 0;
    for (int l = 0; l < q.nlayers; ++l) {
        q.L[l].unit_begin = blk;
        blk += direct ? kFinishDirectWgs : (q.L[l].k + per - 1) / per;
    }
    q.total_units = blk;  // followed by one workgroup per layer for the distortion
    set_unit_table(q);
    // nunits keeps the number of update workgroups (partials to add)
    if (wide)
        hipLaunchKernelGGL(update_finish_kernel<1>, dim3(blk + q.nlayers), dim3(kFinishThreads), 0, s, q);
    else
        hipLaunchKernelGGL(update_finish_kernel<kFinishGroups>, dim3(blk + q.nlayers), dim3(kFinishThreads), 0, s, q);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void* ws, size_t bytes, hipStream_t s) {
    const size_t n16 = bytes / 16;
    unsigned char* tail = (unsigned char*)ws + n16 * 16;
    const size_t ntail = bytes - n16 * 16;
    size_t blocks = (n16 + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint4*)ws, n16, tail, ntail);
    return hipGetLastError();
}

}  // namespace kq
