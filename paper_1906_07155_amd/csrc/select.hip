// select.hip -- per-category proposal selection: greedy NMS or Soft-NMS.
//
// A two-stage detector turns each image's (or class's) scored boxes into proposals
// with NMS; the paper runs its bbox operations on the GPU (§1) and lists Soft-NMS
// among its general modules (§2).  One call selects within every category of a batch:
// one category per image (or class), each category independent.  Definition (candidate
// rule, rank order, decay, dropping, ties) in include/roi_extract.h.
//
// Up to kSelMaxBoxes boxes and kSelMaxCategories categories (and the workspace
// box_nms_batched_workspace_size asks for), kernels on one stream:
//   sel_count_kernel     candidates (score >= threshold, valid category) per range of boxes
//                        and category
//   sel_place_kernel     category starts, the blocks and list room of every category, and
//                        each candidate's key to a slot of its category's range
//   sel_rank_kernel      64 candidates per workgroup: their ranks counted against the keys
//                        of their category (as box_nms does), boxes and scores in rank order
//   greedy: sel_overlap_kernel and sel_resolve_kernel, the suppression of nms.hpp with a
//                        workgroup per category deciding its boxes
//   Soft-NMS: sel_soft_kernel, per category one wave up to 64 candidates, 8 up to 512, 16 up
//                        to 4096
// Past those limits (or with a smaller workspace):
//   nmsb_clear / count / scan / place_kernel, nmsb_select_kernel
//                        counting, placement, and one 1024-thread workgroup per category
//                        that sorts its candidates (bitonic network in LDS, or in global
//                        memory above kSegLds) and walks them in order; the parallel
//                        kernels run the same body for a single category past their limits.
//
// 16 categories of 2000 boxes, greedy, 1000 kept: 389 -> 52 us for the call; 80 categories of 1000
// boxes, 310 of them candidates, linear Soft-NMS, 100 kept: 193 -> 91 us.
#include "nms.hpp"

namespace rex {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSegLds = 8192;    // candidates a category sorts in LDS (64 KiB of keys)
constexpr int kSoftReg = 4;      // Soft-NMS candidates per thread held in registers
constexpr int kSoftLdsBoxes = 3072;   // Soft-NMS: categories up to this size keep boxes in LDS

__global__ __launch_bounds__(256) void nmsb_clear_kernel(int32_t *count, int32_t n) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        count[i] = 0;
}

__device__ __forceinline__ int nmsb_category(const NmsBatchArgs &a, int32_t i) {
    const int c = a.categories ? a.categories[i] : 0;
    // a candidate: a category of the batch and a score at or above the threshold (a NaN
    // score never is)
    return (c >= 0 && c < a.C && a.scores[i] >= a.score_threshold) ? c : -1;
}

// Candidate counting and placement work on contiguous ranges of kPlaceRange boxes per
// workgroup: the workgroup counts its boxes per category in LDS and touches each
// category's device counter once.  Device-scope atomics to one address are serialised
// beyond the per-XCD L2 (about 0.2 us each), so one per box and category -- thousands
// on each of a few counters -- would dominate the selection.
constexpr int kPlaceThreads = 256;
constexpr int kPlaceRange = 4096;

__device__ __forceinline__ void nmsb_range(const NmsBatchArgs &a, int32_t &i0, int32_t &i1) {
    i0 = static_cast<int32_t>(blockIdx.x) * kPlaceRange;
    i1 = min(a.N, i0 + kPlaceRange);
}

__global__ __launch_bounds__(kPlaceThreads) void nmsb_count_kernel(NmsBatchArgs a) {
    extern __shared__ int32_t hist[];   // [C]
    for (int c = threadIdx.x; c < a.C; c += kPlaceThreads) hist[c] = 0;
    __syncthreads();
    int32_t i0, i1;
    nmsb_range(a, i0, i1);
    for (int32_t i = i0 + threadIdx.x; i < i1; i += kPlaceThreads) {
        const int c = nmsb_category(a, i);
        if (c >= 0) atomicAdd(&hist[c], 1);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < a.C; c += kPlaceThreads)
        if (hist[c] > 0) atomicAdd(&a.count[c], hist[c]);
}

__global__ __launch_bounds__(kSelThreads) void nmsb_scan_kernel(NmsBatchArgs a) {
    extern __shared__ int32_t smem[];
    int32_t *hist = smem;              // [C]
    int32_t *part = smem + a.C;        // scan scratch
    for (int i = threadIdx.x; i < a.C; i += kSelThreads) hist[i] = a.count[i];
    __syncthreads();
    const int total = block_exclusive_scan(hist, a.C, part);
    for (int i = threadIdx.x; i < a.C; i += kSelThreads) {
        a.start[i] = hist[i];
        a.count[i] = hist[i];   // becomes the placement cursor
    }
    if (threadIdx.x == 0) a.start[a.C] = total;
}

// Every candidate of the workgroup's range to a slot of its category: the range's count
// per category reserves a run of slots with one device atomic, then LDS cursors deal the
// run out.  The order inside a category is free (the selection sorts it).
__global__ __launch_bounds__(kPlaceThreads) void nmsb_place_kernel(NmsBatchArgs a) {
    extern __shared__ int32_t cur[];   // [C]: counts, then cursors
    for (int c = threadIdx.x; c < a.C; c += kPlaceThreads) cur[c] = 0;
    __syncthreads();
    int32_t i0, i1;
    nmsb_range(a, i0, i1);
    for (int32_t i = i0 + threadIdx.x; i < i1; i += kPlaceThreads) {
        const int c = nmsb_category(a, i);
        if (c >= 0) atomicAdd(&cur[c], 1);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < a.C; c += kPlaceThreads)
        if (cur[c] > 0) cur[c] = atomicAdd(&a.count[c], cur[c]);
    __syncthreads();
    for (int32_t i = i0 + threadIdx.x; i < i1; i += kPlaceThreads) {
        const int c = nmsb_category(a, i);
        if (c < 0) continue;
        const int slot = atomicAdd(&cur[c], 1);
        if (slot >= 0 && slot < a.N) a.sidx[slot] = i;
    }
}

// t / n, correctly rounded, for the small integers of the series: with the reciprocal rounded
// to nearest, one correction step leaves the quotient within one unit and a second makes it
// the rounded one (Markstein, IBM J. Res. Dev. 34, 1990; compared with the division on 3.2e8
// values).  Five operations instead of the division's twenty-odd.
__device__ __forceinline__ double soft_div(double t, int n) {
    const double d = static_cast<double>(n), rn = 1.0 / d;
    double q = t * rn;
    if ((n & (n - 1)) == 0) return q;   // a power of two: exact
    q = fma(fma(-d, q, t), rn, q);
    return fma(fma(-d, q, t), rn, q);
}

// Gaussian decay weight exp(-iou^2 / sigma) rounded to binary32.  exp is evaluated in
// double by scaling and squaring: the argument is halved until it lies in [-1/2, 0], a
// degree-16 Taylor polynomial is summed in Horner form, and the result is squared back;
// every double operation is rounded once, in the written order, so the weight -- which
// decides the next selection -- does not depend on the machine's exp.  Below -128 the
// exponential rounds to +0.
__device__ __forceinline__ float soft_gauss_weight(float iou, float sigma) {
    if (!(iou > 0.0f)) return 1.0f;
    double x = -(static_cast<double>(iou) * static_cast<double>(iou)) / static_cast<double>(sigma);
    if (!(x >= -128.0)) return 0.0f;
    int k = 0;
    while (x < -0.5) {
        x = x * 0.5;
        ++k;
    }
    double e = 1.0;
#pragma unroll
    for (int n = 16; n >= 1; --n) e = 1.0 + soft_div(x * e, n);
    for (int i = 0; i < k; ++i) e = e * e;
    return static_cast<float>(e);
}

// New current score of a candidate after the box `m` was selected; NaN IoU: unchanged.
__device__ __forceinline__ float soft_decay(const NmsBatchArgs &a, float4 m, float4 b, float s) {
    const float iou = nms_iou(m, b);
    if (iou != iou) return s;
    if (a.method == kNmsLinear) {
        if (iou > a.iou_threshold) {
            const float w = 1.0f - iou;
            s = s * w;
        }
        return s;
    }
    return s * soft_gauss_weight(iou, a.sigma);
}

// Ascending sort of keys[0, n) with every position >= n taken as +infinity: the bitonic
// network in the form whose every comparator puts the smaller key at the lower position
// (each merge stage starts by comparing a position with its mirror in the block, then
// halves), so a comparator with its partner past n is a no-op and any n works.  Called
// by the whole workgroup; `keys` in LDS or global memory (sync after every stage).
template <typename Ptr>
__device__ void bitonic_sort_n(Ptr keys, int n) {
    int P = 1;
    while (P < n) P <<= 1;
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int q = threadIdx.x; q < P / 2; q += kSelThreads) {
                int i, p;
                if (j == (k >> 1)) {   // mirror step
                    i = (q / j) * k + (q % j);
                    p = i ^ (k - 1);
                } else {
                    i = ((q & ~(j - 1)) << 1) | (q & (j - 1));
                    p = i + j;
                }
                if (p < n) {
                    const uint64_t x = keys[i], y = keys[p];
                    if (x > y) {
                        keys[i] = y;
                        keys[p] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
}

__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t w = __shfl_xor(v, o, 64);
        v = w < v ? w : v;
    }
    return v;
}

// Greedy NMS over the sorted candidates [base, base + n) of category c, 64 at a time: every wave
// tests them against its share of the kept list and of their own pairs, one wave decides.  The
// kept list is in LDS up to kKeptLds boxes, beyond that in the workspace.  (One wave for the
// pairs and the kept list in the workspace, 32 categories of 8000 boxes: 1948 us against 999.)
constexpr int kKeptLds = kSegLds / 2 - 100;
__device__ void select_greedy(const NmsBatchArgs &a, int c, int base, int n, uint64_t *lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float4 *kl = reinterpret_cast<float4 *>(lds);                      // [kKeptLds]
    float4 *cand = kl + kKeptLds;                                      // [64] the block
    uint64_t *over = reinterpret_cast<uint64_t *>(cand + 64);          // [64] its earlier overlaps
    unsigned long long *hit = reinterpret_cast<unsigned long long *>(over + 64);   // [1]
    int32_t *s_kept = reinterpret_cast<int32_t *>(hit + 1);            // [1]
    static_assert((kKeptLds + 64) * sizeof(float4) + 66 * sizeof(uint64_t) <= kSegLds * sizeof(uint64_t),
                  "select_category's LDS");
    const int limit = a.max_keep;
    int kept = 0;
    for (int b0 = 0; b0 < n && kept < limit; b0 += 64) {
        const int nb = min(64, n - b0);
        if (tid < 64 && tid < nb) cand[tid] = a.sbox[base + b0 + tid];
        if (tid == 0) *hit = 0;
        __syncthreads();
        {
            const float4 mine = lane < nb ? cand[lane] : make_float4(0, 0, 0, 0);
            bool h = false;
            for (int k = wave; k < min(kept, kKeptLds); k += kSelWaves)
                h = h || (nms_iou(kl[k], mine) > a.iou_threshold);
            for (int k = kKeptLds + wave; k < kept; k += kSelWaves)
                h = h || (nms_iou(a.kbox[base + k], mine) > a.iou_threshold);
            const uint64_t bits = __ballot(h && lane < nb);
            if (lane == 0 && bits) atomicOr(hit, static_cast<unsigned long long>(bits));
            // bit t of over[u] marks an earlier candidate t of the block that would remove u
            for (int u = wave; u < nb; u += kSelWaves) {
                const uint64_t m = __ballot(lane < u && nms_iou(mine, cand[u]) > a.iou_threshold);
                if (lane == 0) over[u] = m;
            }
        }
        __syncthreads();
        if (wave == 0) {
            const uint64_t own = lane < nb ? over[lane] : 0;
            const uint64_t h0 = *hit;
            uint64_t U = ~((static_cast<uint64_t>(static_cast<uint32_t>(uniform_i(static_cast<int>(h0 >> 32))))
                            << 32) | static_cast<uint32_t>(uniform_i(static_cast<int>(h0))));
            if (nb < 64) U &= (uint64_t(1) << nb) - 1;
            uint64_t K = 0;   // U: undecided, K: kept
            for (;;) {
                const bool on = (U >> lane) & 1;
                const uint64_t rm = __ballot(on && (own & K) != 0);
                U &= ~rm;
                const uint64_t kn = __ballot(on && (own & (U | K)) == 0) & U;
                K |= kn;
                U &= ~kn;
                if ((rm | kn) == 0) break;
            }
            const int r = kept + __popcll(K & ((uint64_t(1) << lane) - 1));
            if (((K >> lane) & 1) && r < limit) {
                const int pos = base + b0 + lane;
                if (r < kKeptLds) kl[r] = cand[lane];
                else a.kbox[base + r] = cand[lane];
                a.keep[static_cast<int64_t>(c) * limit + r] = a.sidx[pos];
                a.kept_scores[static_cast<int64_t>(c) * limit + r] = a.sscore[pos];
            }
            if (lane == 0) *s_kept = min(kept + __popcll(K), limit);
        }
        __syncthreads();
        kept = *s_kept;
        __syncthreads();   // the block's LDS is rewritten next
    }
    for (int r = kept + tid; r < limit; r += kSelThreads) {
        a.keep[static_cast<int64_t>(c) * limit + r] = -1;
        a.kept_scores[static_cast<int64_t>(c) * limit + r] = 0.0f;
    }
    if (tid == 0) a.num_keep[c] = kept;
}

// Soft-NMS over the sorted candidates [base, base + n) of category c.  Candidates are
// dealt to threads (position r to thread r % 1024); up to kSoftReg per thread live in
// registers, the rest of a long category in global memory.
__device__ void select_soft(const NmsBatchArgs &a, int c, int base, int n, uint64_t *lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint64_t *wmin = lds;                                        // [2][kSelWaves]
    float4 *sbox = reinterpret_cast<float4 *>(lds + 2 * kSelWaves);   // [kSoftLdsBoxes]
    const bool lds_boxes = n <= kSoftLdsBoxes;
    if (lds_boxes)
        for (int r = tid; r < n; r += kSelThreads) sbox[r] = a.sbox[base + r];
    for (int r = kSoftReg * kSelThreads + tid; r < n; r += kSelThreads) a.skey[base + r] = 1;
    float s[kSoftReg];
    float4 bx[kSoftReg];
    uint32_t alive = 0;
#pragma unroll
    for (int m = 0; m < kSoftReg; ++m) {
        const int r = tid + m * kSelThreads;
        s[m] = 0.0f;
        bx[m] = make_float4(0, 0, 0, 0);
        if (r < n) {
            s[m] = a.sscore[base + r];
            bx[m] = a.sbox[base + r];
            alive |= 1u << m;
        }
    }
    __syncthreads();
    const int limit = a.max_keep;
    float4 last = make_float4(0, 0, 0, 0);
    bool have_last = false;
    int kept = 0;
    for (int it = 0; kept < limit; ++it) {
        // decay against the last selected box, drop, and this thread's best key
        uint64_t best = ~uint64_t(0);
#pragma unroll
        for (int m = 0; m < kSoftReg; ++m) {
            if (!((alive >> m) & 1)) continue;
            if (have_last) {
                s[m] = soft_decay(a, last, bx[m], s[m]);
                if (s[m] < a.score_threshold) {
                    alive &= ~(1u << m);
                    continue;
                }
            }
            const uint64_t key = (static_cast<uint64_t>(nms_key(s[m])) << 32) |
                                 static_cast<uint32_t>(tid + m * kSelThreads);
            best = key < best ? key : best;
        }
        // positions past the register slots keep their state in global memory: the
        // current score in sscore, alive in skey (free once the category is sorted)
        for (int r = tid + kSoftReg * kSelThreads; r < n; r += kSelThreads) {
            if (a.skey[base + r] == 0) continue;
            float sr = a.sscore[base + r];
            if (have_last) {
                sr = soft_decay(a, last, a.sbox[base + r], sr);
                a.sscore[base + r] = sr;
                if (sr < a.score_threshold) {
                    a.skey[base + r] = 0;
                    continue;
                }
            }
            const uint64_t key = (static_cast<uint64_t>(nms_key(sr)) << 32) | static_cast<uint32_t>(r);
            best = key < best ? key : best;
        }
        best = wave_min_u64(best);
        uint64_t *slot = wmin + (it & 1) * kSelWaves;
        if (lane == 0) slot[wave] = best;
        __syncthreads();
        uint64_t g = ~uint64_t(0);
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) g = slot[w] < g ? slot[w] : g;
        if (g == ~uint64_t(0)) break;   // uniform: no candidate left
        const int r = static_cast<int>(static_cast<uint32_t>(g));
        // the owner outputs the selected candidate with its current score and retires it
        if (r % kSelThreads == tid) {
            const int m = r / kSelThreads;
            float sc = 0.0f;
            if (m < kSoftReg) {
#pragma unroll
                for (int q = 0; q < kSoftReg; ++q)
                    if (q == m) sc = s[q];
                alive &= ~(1u << m);
            } else {
                sc = a.sscore[base + r];
                a.skey[base + r] = 0;
            }
            a.keep[static_cast<int64_t>(c) * limit + kept] = a.sidx[base + r];
            a.kept_scores[static_cast<int64_t>(c) * limit + kept] = sc;
        }
        ++kept;
        // every thread reads the selected box (its position is known to all)
        last = lds_boxes ? sbox[r] : a.sbox[base + r];
        have_last = true;
    }
    for (int q = kept + tid; q < limit; q += kSelThreads) {
        a.keep[static_cast<int64_t>(c) * limit + q] = -1;
        a.kept_scores[static_cast<int64_t>(c) * limit + q] = 0.0f;
    }
    if (tid == 0) a.num_keep[c] = kept;
}

// Candidates [base, base + n) into rank order, with their boxes and scores.
__device__ void sort_category(const NmsBatchArgs &a, int base, int n, uint64_t *lds) {
    // rank order: score rank key, then box index (unique keys)
    uint64_t *gkeys = a.skey + base;
    const bool in_lds = n <= kSegLds;
    for (int r = threadIdx.x; r < n; r += kSelThreads) {
        const int i = a.sidx[base + r];
        const uint64_t key = (static_cast<uint64_t>(nms_key(a.scores[i])) << 32) |
                             static_cast<uint32_t>(i);
        if (in_lds) lds[r] = key;
        else gkeys[r] = key;
    }
    __syncthreads();
    if (in_lds) bitonic_sort_n(lds, n);
    else bitonic_sort_n(gkeys, n);
    for (int r = threadIdx.x; r < n; r += kSelThreads) {
        const uint64_t key = in_lds ? lds[r] : gkeys[r];
        const int i = static_cast<int>(static_cast<uint32_t>(key));
        a.sidx[base + r] = i;
        const float *bp = a.boxes + 4 * static_cast<int64_t>(i);
        a.sbox[base + r] = make_float4(bp[0], bp[1], bp[2], bp[3]);
        a.sscore[base + r] = a.scores[i];
    }
    __syncthreads();   // sorted arrays complete; the LDS is reused below
}

// One category by one workgroup: sorts its candidates (unless sel_rank_kernel has) and selects in
// order.
__device__ void select_category(const NmsBatchArgs &a, int c, uint64_t *lds, bool sorted) {
    const int base = a.start[c];
    const int n = a.start[c + 1] - base;
    if (!sorted) sort_category(a, base, n, lds);
    if (a.method == kNmsHard) select_greedy(a, c, base, n, lds);
    else select_soft(a, c, base, n, lds);
}
__global__ __launch_bounds__(kSelThreads) void nmsb_select_kernel(NmsBatchArgs a) {
    __shared__ uint64_t lds[kSegLds];   // sort keys, then the selection's working set
    for (int c = blockIdx.x; c < a.C; c += gridDim.x) {
        select_category(a, c, lds, false);
        __syncthreads();   // before the next category reuses the LDS
    }
}

// ---------------------------------------------------------------------------
// The parallel selection
// ---------------------------------------------------------------------------

// hist[c] += 1 for every lane with c >= 0; returns the lane's slot (the value before).  When
// the wave's candidates are of one category (boxes often come grouped by image), one lane
// adds for all: 64 adds to one LDS address would take turns.
__device__ __forceinline__ int sel_add(int32_t *hist, int c) {
    const uint64_t m = __ballot(c >= 0);
    if (m == 0) return 0;
    const int lane = threadIdx.x & 63;
    const int first = __builtin_ctzll(m);
    const int c0 = __builtin_amdgcn_readlane(c, first);
    if (__ballot(c >= 0 && c != c0) == 0) {
        int at = 0;
        if (lane == first) at = atomicAdd(&hist[c0], __popcll(m));
        return __builtin_amdgcn_readlane(at, first) + __popcll(m & ((uint64_t(1) << lane) - 1));
    }
    return c >= 0 ? atomicAdd(&hist[c], 1) : 0;
}

// Boxes per range: whole rounds of a workgroup, at most kSelRanges ranges.
__host__ __device__ inline int sel_range(int N) {
    const int per = (N + kSelRanges - 1) / kSelRanges;
    const int r = (per + kSelThreads - 1) / kSelThreads * kSelThreads;
    return r < 2 * kSelThreads ? 2 * kSelThreads : r;
}

__global__ __launch_bounds__(kSelThreads) void sel_count_kernel(NmsBatchArgs a) {
    extern __shared__ int32_t hist[];   // [C]
    for (int c = threadIdx.x; c < a.C; c += kSelThreads) hist[c] = 0;
    __syncthreads();
    const int range = sel_range(a.N);
    const int i0 = static_cast<int>(blockIdx.x) * range, i1 = min(a.N, i0 + range);
    for (int i = i0 + static_cast<int>(threadIdx.x); i - static_cast<int>(threadIdx.x) < i1;
         i += kSelThreads)
        sel_add(hist, i < i1 ? nmsb_category(a, i) : -1);
    __syncthreads();
    for (int c = threadIdx.x; c < a.C; c += kSelThreads)
        a.hist[static_cast<int64_t>(blockIdx.x) * a.C + c] = hist[c];
}

// Every workgroup sums the ranges' counts itself (a few KiB), so no kernel between the count
// and the placement scans them; workgroup 0 also writes the tables of the categories.
__global__ __launch_bounds__(kSelThreads) void sel_place_kernel(NmsBatchArgs a, int ranges, int fast_n) {
    extern __shared__ int32_t smem[];
    int32_t *cur = smem;               // [C] category starts, then cursors
    int32_t *tab = smem + a.C;         // [C]
    int32_t *part = smem + 2 * a.C;    // scan scratch
    const int tid = threadIdx.x;
    const int me = static_cast<int>(blockIdx.x);
    int before = 0, n = 0;             // this thread's category (C <= 1024 threads)
    if (tid < a.C) {
#pragma unroll 8
        for (int g = 0; g < ranges; ++g) {
            const int v = a.hist[static_cast<int64_t>(g) * a.C + tid];
            n += v;
            before += g < me ? v : 0;
        }
        cur[tid] = n;
    }
    __syncthreads();
    const int total = block_exclusive_scan(cur, a.C, part);
    if (me == 0) {
        if (tid < a.C) {
            a.start[tid] = cur[tid];
            tab[tid] = (n + 63) >> 6;
        }
        if (tid == 0) a.start[a.C] = total;
        __syncthreads();
        const int blocks = block_exclusive_scan(tab, a.C, part);
        if (tid < a.C) a.bfirst[tid] = tab[tid];
        if (tid == 0) a.bfirst[a.C] = blocks;
        for (int g = tid; g < blocks; g += kSelThreads) {
            int lo = 0, hi = a.C;      // tab[lo] <= g, and the next category starts after g
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (tab[mid] <= g) lo = mid;
                else hi = mid;
            }
            a.bcat[g] = lo;
        }
        __syncthreads();
        // (at most 2^18 candidates of 81 words: the sum fits 32 bits)
        const int w = n > 0 && n <= fast_n ? static_cast<int>(nms_words(n)) : 0;
        if (tid < a.C) tab[tid] = w;
        __syncthreads();
        if (block_exclusive_scan(tab, a.C, part) <= a.word_cap) {
            if (tid < a.C) a.wfirst[tid] = w > 0 ? tab[tid] : -1;
        } else {
            // not room for all: in index order, every category that still fits
            if (tid < a.C) tab[tid] = w;
            __syncthreads();
            if (tid == 0) {
                int at = 0;
                for (int c = 0; c < a.C; ++c) {
                    const int words = tab[c];
                    const bool fits = words > 0 && at + words <= a.word_cap;
                    a.wfirst[c] = fits ? at : -1;
                    at += fits ? words : 0;
                }
            }
        }
    }
    if (tid < a.C) cur[tid] += before;
    __syncthreads();
    const int range = sel_range(a.N);
    const int i0 = me * range, i1 = min(a.N, i0 + range);
    for (int i = i0 + tid; i - tid < i1; i += kSelThreads) {
        const int c = i < i1 ? nmsb_category(a, i) : -1;
        const int slot = sel_add(cur, c);
        if (c >= 0 && slot >= 0 && slot < a.N) {
            a.sidx[slot] = i;
            a.skey[slot] = (static_cast<uint64_t>(nms_key(a.scores[i])) << 32) |
                           static_cast<uint32_t>(i);
        }
    }
}

// The category and block of a workgroup of the block grids; false past the last block.
__device__ __forceinline__ bool sel_block(const NmsBatchArgs &a, int g, int &c, int &ib, int &base,
                                          int &n) {
    if (g >= a.bfirst[a.C]) return false;
    c = uniform_i(max(0, min(a.bcat[g], a.C - 1)));
    ib = g - a.bfirst[c];
    base = a.start[c];
    n = a.start[c + 1] - base;
    return true;
}

constexpr int kSelRankThreads = 1024;
constexpr int kSelRankTile = 1024;

__global__ __launch_bounds__(kSelRankThreads) void sel_rank_kernel(NmsBatchArgs a) {
    __shared__ uint64_t keys[kSelRankTile];
    __shared__ int32_t part[kSelRankThreads / 64][64];
    int c, ib, base, n;
    if (!sel_block(a, static_cast<int>(blockIdx.x), c, ib, base, n)) return;
    if (n > kSegLds) return;   // sorted by its workgroup
    const int lane = threadIdx.x & 63;
    const int wave = uniform_i(threadIdx.x >> 6);
    const int r = ib * 64 + lane;
    const uint64_t ki = r < n ? a.skey[base + r] : 0;
    int cnt = 0;
    for (int t0 = 0; t0 < n; t0 += kSelRankTile) {
        const int tn = min(kSelRankTile, n - t0);
        __syncthreads();
        static_assert(kSelRankTile == kSelRankThreads, "one key per thread");
        const int j = threadIdx.x;
        keys[j] = j < tn ? a.skey[base + t0 + j] : ~uint64_t(0);   // padding precedes nothing
        __syncthreads();
        // the wave's sixteenth of the tile's keys
        const int per = ((tn + 15) / 16 + 7) & ~7;
        const int j0 = min(wave * per, kSelRankTile), j1 = min(j0 + per, kSelRankTile);
        for (int q = j0; q < j1; q += 8) {
#pragma unroll
            for (int u = 0; u < 8; ++u) cnt += keys[q + u] < ki ? 1 : 0;
        }
    }
    part[wave][lane] = cnt;
    __syncthreads();
    if (wave == 0 && r < n) {
        int at = base;
#pragma unroll
        for (int w = 0; w < kSelRankThreads / 64; ++w) at += part[w][lane];
        const int i = static_cast<int>(static_cast<uint32_t>(ki));
        a.sidx[at] = i;
        const float *bp = a.boxes + 4 * static_cast<int64_t>(i);
        a.sbox[at] = make_float4(bp[0], bp[1], bp[2], bp[3]);
        a.sscore[at] = a.scores[i];
    }
}

__global__ __launch_bounds__(kNmsOverlapThreads) void sel_overlap_kernel(NmsBatchArgs a, float share) {
    __shared__ int32_t count;
    int c, ib, base, n;
    if (!sel_block(a, static_cast<int>(blockIdx.x) >> kSelSplitLog, c, ib, base, n)) return;
    const int w = a.wfirst[c];
    const int s = static_cast<int>(blockIdx.x) & ((1 << kSelSplitLog) - 1);
    // (a single block has no lists, so its other splits have nothing to write)
    if (w < 0 || (n <= 64 && s > 0)) return;
    overlap_rows(a.sbox + base, nullptr, n, a.iou_threshold, share, a.words + w, ib, s, kSelSplitLog, &count);
}

__global__ __launch_bounds__(kSelThreads) void sel_resolve_kernel(NmsBatchArgs a) {
    union Smem {
        ResolveSmem<8> r;
        uint64_t lds[kSegLds];
    };
    __shared__ Smem sm;
    const int c = static_cast<int>(blockIdx.x);
    const int base = a.start[c];
    const int n = a.start[c + 1] - base;
    if (n > 0 && a.wfirst[c] < 0) {
        select_category(a, c, sm.lds, n <= kSegLds);
        return;
    }
    const int limit = a.max_keep;
    const int64_t out = static_cast<int64_t>(c) * limit;
    int count = 0;
    if (n > 0) {
        resolve_rows<8, kSelSplitLog>(a.words + a.wfirst[c], n, sm.r);
        const int lane = threadIdx.x & 63;
        const int nb = (n + 63) >> 6;
        for (int b = static_cast<int>(threadIdx.x) >> 6; b < nb; b += kSelWaves) {
            const int before = kept_before(sm.r.kept, b, lane);
            const uint64_t kept = sm.r.kept[b];
            if ((kept >> lane) & 1) {
                const int r = before + __popcll(kept & ((uint64_t(1) << lane) - 1));
                if (r < limit) {
                    a.keep[out + r] = a.sidx[base + b * 64 + lane];
                    a.kept_scores[out + r] = a.sscore[base + b * 64 + lane];
                }
            }
        }
        count = min(kept_before(sm.r.kept, nb, lane), limit);
    }
    for (int r = count + static_cast<int>(threadIdx.x); r < limit; r += kSelThreads) {
        a.keep[out + r] = -1;
        a.kept_scores[out + r] = 0.0f;
    }
    if (threadIdx.x == 0) a.num_keep[c] = count;
}

// Minimum of a value over the first LANES (16 or 64) lanes (uniform), in DPP moves (see
// wave_inclusive_scan).
template <int LANES>
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
    constexpr int kNone = -1;   // lanes shifted in from outside: the largest value
    auto step = [](uint32_t v, int moved) {
        const uint32_t o = static_cast<uint32_t>(moved);
        return o < v ? o : v;
    };
    x = step(x, __builtin_amdgcn_update_dpp(kNone, static_cast<int>(x), 0x111, 0xf, 0xf, false));
    x = step(x, __builtin_amdgcn_update_dpp(kNone, static_cast<int>(x), 0x112, 0xf, 0xf, false));
    x = step(x, __builtin_amdgcn_update_dpp(kNone, static_cast<int>(x), 0x114, 0xf, 0xf, false));
    x = step(x, __builtin_amdgcn_update_dpp(kNone, static_cast<int>(x), 0x118, 0xf, 0xf, false));
    if constexpr (LANES == 64) {
        x = step(x, __builtin_amdgcn_update_dpp(kNone, static_cast<int>(x), 0x142, 0xa, 0xf, false));
        x = step(x, __builtin_amdgcn_update_dpp(kNone, static_cast<int>(x), 0x143, 0xc, 0xf, false));
    }
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), LANES - 1));
}

// Soft-NMS over the n <= 64 W R sorted candidates [base, base + n) of a category by W waves:
// candidate m of a lane is rank 64 W m + 64 wave + lane, held in registers with its rank key.
// A selection is: decay against the last selected box (the weights only where some lane
// overlaps it), each lane's best, a wave minimum by DPP moves and, with more than one wave,
// one barrier with the waves' bests in LDS.  The selected ranks and scores are kept in LDS
// and written at the end, so no memory access sits between two selections.
template <int R>
struct SoftSmem {
    uint32_t key[2][16], rank[2][16];
    float score[2][16];
    float4 box[2][16];
    uint16_t sel[64 * 16 * R];
    float sel_score[64 * 16 * R];
};

template <int W, int R>
__device__ __forceinline__ void sel_soft(const NmsBatchArgs &a, int c, int base, int n, float share,
                                         SoftSmem<R> &sm) {
    const int lane = threadIdx.x & 63;
    const int wave = W == 1 ? 0 : uniform_i(threadIdx.x >> 6);
    float s[R];
    float4 bx[R];
    uint32_t key[R];
    uint32_t alive = 0;
#pragma unroll
    for (int m = 0; m < R; ++m) {
        const int r = 64 * W * m + 64 * wave + lane;
        s[m] = 0.0f;
        bx[m] = make_float4(0, 0, 0, 0);
        key[m] = 0xffffffffu;
        if (r < n) {
            s[m] = a.sscore[base + r];
            bx[m] = a.sbox[base + r];
            key[m] = nms_key(s[m]);
            alive |= 1u << m;
        }
    }
    const int limit = min(a.max_keep, n);
    // Linear decay changes a score only where IoU > threshold, which overlap_part dismisses for
    // most boxes without the division; Gaussian decay wherever boxes meet (share is NaN: no
    // dismissal).
    float part[R];
#pragma unroll
    for (int m = 0; m < R; ++m)
        part[m] = overlap_part((bx[m].z - bx[m].x) * (bx[m].w - bx[m].y), share);
    float4 last = make_float4(0, 0, 0, 0);
    int kept = 0;
    for (int it = 0; kept < limit; ++it) {
        if (it > 0) {
            const float lpart = overlap_part((last.z - last.x) * (last.w - last.y), share);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                if (64 * W * m >= n) continue;
                const float iw = fminf(last.z, bx[m].z) - fmaxf(last.x, bx[m].x);
                const float ih = fminf(last.w, bx[m].w) - fmaxf(last.y, bx[m].y);
                // without an intersection the IoU is 0 or NaN and the score stays (a negative
                // linear threshold lets 0 pass: weight 1 - 0); only a changed score can fall
                // below the threshold
                const bool meet = ((alive >> m) & 1) && iw > 0.0f && ih > 0.0f &&
                                  !(iw * ih < part[m] + lpart);
                if (__ballot(meet) == 0) continue;
                if (meet) {
                    s[m] = soft_decay(a, last, bx[m], s[m]);
                    key[m] = nms_key(s[m]);
                    if (s[m] < a.score_threshold) alive &= ~(1u << m);
                }
            }
        }
        uint32_t bk = 0xffffffffu, br = 0xffffffffu;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            // ranks ascend with m: an equal key keeps the earlier one
            const bool b = ((alive >> m) & 1) && (key[m] < bk || br == 0xffffffffu);
            bk = b ? key[m] : bk;
            br = b ? static_cast<uint32_t>(64 * W * m + 64 * wave + lane) : br;
        }
        uint32_t gk = wave_min_u32<64>(bk);
        uint64_t tie = __ballot(br != 0xffffffffu && bk == gk);
        uint32_t gr = 0xffffffffu;   // uniform: the wave's best rank, none if no lane has one
        if (tie != 0)
            gr = (tie & (tie - 1)) == 0
                     ? static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(br), __builtin_ctzll(tie)))
                     : wave_min_u32<64>(br != 0xffffffffu && bk == gk ? br : 0xffffffffu);
        float gs = 0.0f;
        float4 gb = make_float4(0, 0, 0, 0);
        if (gr != 0xffffffffu) {
            const int l = static_cast<int>(gr & 63u);
            auto take = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
#pragma unroll
            for (int m = 0; m < R; ++m)
                if (static_cast<int>(gr) / (64 * W) == m) {
                    gs = take(s[m]);
                    gb = make_float4(take(bx[m].x), take(bx[m].y), take(bx[m].z), take(bx[m].w));
                }
        }
        if constexpr (W > 1) {
            const int p = it & 1;
            if (lane == 0) {
                sm.key[p][wave] = gk;
                sm.rank[p][wave] = gr;
                sm.score[p][wave] = gs;
                sm.box[p][wave] = gb;
            }
            __syncthreads();
            // every wave reduces the W bests (lanes past W hold none)
            const uint32_t k = lane < W ? sm.key[p][lane] : 0xffffffffu;
            const uint32_t r = lane < W ? sm.rank[p][lane] : 0xffffffffu;
            gk = wave_min_u32<16>(r != 0xffffffffu ? k : 0xffffffffu);
            gr = wave_min_u32<16>(k == gk ? r : 0xffffffffu);
            if (gr != 0xffffffffu) {
                const int w = static_cast<int>(gr / 64u) % W;
                gs = sm.score[p][w];
                gb = sm.box[p][w];
            }
        }
        if (gr == 0xffffffffu) break;   // no candidate left, in any wave
        if (lane == static_cast<int>(gr & 63u) && static_cast<int>(gr / 64u) % W == wave)
            alive &= ~(1u << (gr / (64u * W)));
        if (lane == 0 && wave == 0) {
            sm.sel[kept] = static_cast<uint16_t>(gr);
            sm.sel_score[kept] = gs;
        }
        ++kept;
        last = gb;
    }
    if constexpr (W > 1) __syncthreads();
    else wave_sync();
    const int64_t out = static_cast<int64_t>(c) * a.max_keep;
    for (int q = static_cast<int>(threadIdx.x); q < a.max_keep; q += 64 * W) {
        a.keep[out + q] = q < kept ? a.sidx[base + sm.sel[q]] : -1;
        a.kept_scores[out + q] = q < kept ? sm.sel_score[q] : 0.0f;
    }
    if (threadIdx.x == 0) a.num_keep[c] = kept;
}

// One candidate per lane while 16 waves hold them, in one wave up to 64 candidates and in 8 up
// to 512 (80 categories of 310: 108 us with one wave and five candidates per lane, 91 with 16
// waves, 77 with 8); four per lane up to 4096; a longer category is walked by select_category.
//
// The waves a category does not need end before the first barrier, and nothing follows the
// selection: the hardware's barrier waits for the waves of a workgroup that have not ended
// (CDNA instruction set guides, s_barrier).  Kept to the barriers instead, eight idle waves cost
// each of the selections (80 categories of 310: 91 -> 106 us for the call).
__global__ __launch_bounds__(kSelThreads) void sel_soft_kernel(NmsBatchArgs a, float share) {
    union Smem {
        SoftSmem<1> s1;
        SoftSmem<4> s4;
        uint64_t lds[kSegLds];
    };
    __shared__ Smem sm;
    const int c = static_cast<int>(blockIdx.x);
    const int base = a.start[c];
    const int n = a.start[c + 1] - base;
    const int threads = n <= 64 ? 64 : n <= 512 ? 512 : kSelThreads;
    if (static_cast<int>(threadIdx.x) >= threads) return;   // whole waves
    if (n <= 64) sel_soft<1, 1>(a, c, base, n, share, sm.s1);
    else if (n <= 512) sel_soft<8, 1>(a, c, base, n, share, sm.s1);
    else if (n <= 1024) sel_soft<16, 1>(a, c, base, n, share, sm.s1);
    else if (n <= 4096) sel_soft<16, 4>(a, c, base, n, share, sm.s4);
    else select_category(a, c, sm.lds, n <= kSegLds);
}

static hipError_t launch_sel(const NmsBatchArgs &a, hipStream_t stream) {
    const int ranges = (a.N + sel_range(a.N) - 1) / sel_range(a.N);
    const size_t cats = static_cast<size_t>(a.C) * sizeof(int32_t);
    hipError_t e;
    sel_count_kernel<<<ranges, kSelThreads, cats, stream>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    sel_place_kernel<<<ranges, kSelThreads, 2 * cats + 64 * sizeof(int32_t), stream>>>(
        a, ranges, a.method == kNmsHard ? kNmsMaxBoxes : 0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int blocks = a.N / 64 + a.C;   // at least the categories' blocks
    sel_rank_kernel<<<blocks, kSelRankThreads, 0, stream>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.method != kNmsHard) {
        sel_soft_kernel<<<a.C, kSelThreads, 0, stream>>>(
            a, a.method == kNmsLinear ? nms_share(a.iou_threshold) : __builtin_nanf(""));
        return hipGetLastError();
    }
    sel_overlap_kernel<<<blocks << kSelSplitLog, kNmsOverlapThreads, 0, stream>>>(
        a, nms_share(a.iou_threshold));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    sel_resolve_kernel<<<a.C, kSelThreads, 0, stream>>>(a);
    return hipGetLastError();
}

hipError_t launch_nms_batched(const NmsBatchArgs &a, hipStream_t stream) {
    if (a.words) return launch_sel(a, stream);
    nmsb_clear_kernel<<<std::max(1, std::min((a.C + 255) / 256, 256)), 256, 0, stream>>>(a.count,
                                                                                         a.C);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // contiguous ranges of kPlaceRange boxes, one workgroup each (N <= 2^24: at most 4096)
    const int blocks = static_cast<int>((static_cast<int64_t>(a.N) + kPlaceRange - 1) / kPlaceRange);
    const size_t hist_bytes = static_cast<size_t>(a.C) * sizeof(int32_t);
    if (a.N > 0) {
        nmsb_count_kernel<<<blocks, kPlaceThreads, hist_bytes, stream>>>(a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const size_t shmem = static_cast<size_t>(a.C + kSelThreads) * sizeof(int32_t);
    nmsb_scan_kernel<<<1, kSelThreads, shmem, stream>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.N > 0) {
        nmsb_place_kernel<<<blocks, kPlaceThreads, hist_bytes, stream>>>(a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    nmsb_select_kernel<<<std::min(a.C, 4096), kSelThreads, 0, stream>>>(a);
    return hipGetLastError();
}

}  // namespace rex
