// nms.hpp -- greedy suppression in parallel, shared by box_nms (nms.hip) and the
// per-category selection (select.hip).
//
// Input: boxes in rank order.  Greedy NMS keeps a box unless a kept box of higher rank
// overlaps it.  Two kernels' bodies:
//
//   overlap_rows   for 64 boxes at a time, which boxes of higher rank each overlaps by IoU >
//                  threshold, as 64-bit words.  Overlaps are sparse: the words of a block's
//                  own boxes are stored as they are, of the others only the nonzero ones, in
//                  a list with their row and word index.
//   resolve_rows   one workgroup decides all boxes.  The definition fixes a box as soon as
//                  every box it overlaps is decided (removed by a kept one, kept if there is
//                  none), so each round looks at all listed words of undecided boxes at once
//                  and then lets every block of 64 decide what it can, its own overlaps by
//                  ballots.  The lowest undecided block depends on decided boxes only, so a
//                  round decides all of it: at most as many rounds as blocks, in practice the
//                  length of the longest chain of overlaps (4 to 6).  Walking the blocks one
//                  after the other costs two barriers and up to 64 dependent steps for each
//                  (8192 boxes: 461 us against 23 us).
#pragma once

#include "internal.hpp"

namespace rex {

// The words of a row block are dealt to 2^lg workgroups (word w to split w % 2^lg), and each
// writes a list of its own: 8 in box_nms, whose one problem has at most 128 row blocks; 2 in
// the selection, whose many categories fill the chip with fewer, longer workgroups (16
// categories of 2000: 32 us with 8, 26 us with 2).
constexpr int kNmsSplitLog = 3;
constexpr int kSelSplitLog = 1;

// Workspace of n boxes in nb blocks: the blocks' own words [n], the lists' lengths
// [nb][2^lg], and per list room for all of its words (64-bit) and their tags (16-bit,
// row in the block | word << 6).
struct NmsLists {
    uint64_t *own;
    int32_t *len;
    uint64_t *word;
    uint16_t *tag;
};
// Words of split s before the diagonal of block ib, those of the splits before it, and the
// words of all lists before that of (ib, s).
__host__ __device__ inline int32_t nms_split_words(int32_t ib, int32_t s, int lg) {
    return (ib + (1 << lg) - 1 - s) >> lg;
}
__host__ __device__ inline int32_t nms_list_base(int32_t n, int32_t ib, int32_t s, int lg) {
    const int32_t rows = n - 64 * ib < 64 ? n - 64 * ib : 64;
    const int32_t r = ib & ((1 << lg) - 1);
    return 32 * ib * (ib - 1) + rows * (s * (ib >> lg) + (s < r ? s : r));
}
__host__ __device__ inline int32_t nms_list_words(int32_t n) {
    const int32_t nb = (n + 63) >> 6;
    return nb > 0 ? 32 * (nb - 1) * (nb - 2) + (n - 64 * (nb - 1)) * (nb - 1) : 0;
}
// The lists' lengths in 64-bit words (a single block has no lists).
__host__ __device__ inline int32_t nms_len_words(int32_t n) {
    const int32_t nb = (n + 63) >> 6;
    return nb > 1 ? nb << (kNmsSplitLog - 1) : 0;   // room for the most splits
}
// 64-bit words in all; never more than n * nb (the lists hold only half of the matrix).
__host__ __device__ inline int64_t nms_words(int32_t n) {
    const int64_t lw = nms_list_words(n);
    return n + nms_len_words(n) + lw + ((lw + 3) >> 2);
}
__device__ __forceinline__ NmsLists nms_lists(uint64_t *ws, int32_t n) {
    NmsLists l;
    l.own = ws;
    l.len = reinterpret_cast<int32_t *>(ws + n);
    l.word = ws + n + nms_len_words(n);
    l.tag = reinterpret_cast<uint16_t *>(l.word + nms_list_words(n));
    return l;
}

// IoU > t (t >= 0) needs an intersection I of at least t / (1 + t) of the areas' sum, up to
// the rounding of the definition's few operations.  A box's part is that share of its area,
// less 1e-6 (16 units of 2^-24; c = nms_share(t)): I < part_i + part_j then proves IoU <= t.
// Only pairs of positive sides can have I > 0, so no sum cancels; areas too small for the
// relative bound (denormal products), a NaN area and a negative threshold get a part that
// dismisses nothing.
inline float nms_share(float t) {
    return t >= 0.0f ? t / (1.0f + t) * (1.0f - 1e-6f) : __builtin_nanf("");
}
__device__ __forceinline__ float overlap_part(float area, float c) {
    const float p = c * area;
    return c == c && !(area < 1e-30f) ? p : -__builtin_inff();
}

// Rows of block ib, words s, s + 2^lg, ... <= ib, by 512 threads: wave v takes rows 8 v
// .. 8 v + 7, whose boxes it holds in scalar registers, and walks the words with lane =
// column box (the next word's boxes in flight); a compare writes the lanes' verdicts on a
// row, the row's word, as a scalar mask.  The definition's division runs only for the rows
// where some lane is not dismissed by overlap_part.  cats may be null (one category).  (64
// rows per wave, in LDS: 34 us against 23 us on 8192 boxes, 14 against 5 on 1000,
// where the chain of one wave is all there is.)
constexpr int kNmsOverlapThreads = 512;
__device__ __forceinline__ void overlap_rows(const float4 *boxes, const int32_t *cats, int n,
                                             float threshold, float share, uint64_t *ws, int ib,
                                             int s, int lg, int32_t *count) {
    const int lane = threadIdx.x & 63;
    const int v = uniform_i(threadIdx.x >> 6);
    const int r0 = 8 * v;
    const int i = ib * 64 + lane;
    const float none = __builtin_inff();
    if (threadIdx.x == 0) *count = 0;   // LDS: this list's length
    __syncthreads();
    const NmsLists out = nms_lists(ws, n);
    const int32_t list = nms_list_base(n, ib, s, lg);
    float rx1[8], ry1[8], rx2[8], ry2[8], rarea[8], rpart[8];
    int32_t rcat[8];
    {
        const bool on = i < n;
        const float4 b = on ? boxes[i] : make_float4(0, 0, 0, 0);
        const int c = on && cats ? cats[i] : 0;
        const float w = b.z - b.x;
        const float h = b.w - b.y;
        const float area = w * h;
        const float part = on ? overlap_part(area, share) : none;
        auto lane_f = [](float x, int l) {
            return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
        };
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            rx1[u] = lane_f(b.x, r0 + u);
            ry1[u] = lane_f(b.y, r0 + u);
            rx2[u] = lane_f(b.z, r0 + u);
            ry2[u] = lane_f(b.w, r0 + u);
            rarea[u] = lane_f(area, r0 + u);
            rpart[u] = lane_f(part, r0 + u);
            rcat[u] = __builtin_amdgcn_readlane(c, r0 + u);
        }
    }
    const bool mine = lane >= r0 && lane < r0 + 8 && i < n;   // lanes that store the wave's rows
    auto load = [&](int jb, float4 &b, int &c) {
        const int j = jb * 64 + lane;
        b = make_float4(0, 0, 0, 0);
        c = 0;
        if (jb <= ib && j < n) {
            b = boxes[j];
            if (cats) c = cats[j];
        }
    };
    float4 nxt;
    int ncat;
    load(s, nxt, ncat);
    for (int jb = s; jb <= ib; jb += 1 << lg) {
        const float4 bj = nxt;
        const int cj = ncat;
        load(jb + (1 << lg), nxt, ncat);
        const bool jon = jb * 64 + lane < n;
        const float wj = bj.z - bj.x;
        const float hj = bj.w - bj.y;
        const float area_j = wj * hj;
        const float part_j = jon ? overlap_part(area_j, share) : none;
        uint64_t cand[8], any = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            // (a negative height alone makes the product negative: dismissed as 0 is)
            const float iw = fmaxf(fminf(bj.z, rx2[u]) - fmaxf(bj.x, rx1[u]), 0.0f);
            const float ih = fminf(bj.w, ry2[u]) - fmaxf(bj.y, ry1[u]);
            cand[u] = __builtin_amdgcn_ballot_w64(!(iw * ih < part_j + rpart[u]));
            any |= cand[u];
        }
        if (any == 0 && jb != ib) continue;
        uint64_t bits = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (cand[u] == 0) continue;
            const float ix1 = fmaxf(bj.x, rx1[u]);
            const float iy1 = fmaxf(bj.y, ry1[u]);
            const float ix2 = fminf(bj.z, rx2[u]);
            const float iy2 = fminf(bj.w, ry2[u]);
            float iw = ix2 - ix1;
            float ih = iy2 - iy1;
            iw = fmaxf(iw, 0.0f);
            ih = fmaxf(ih, 0.0f);
            const float inter = iw * ih;
            const float sum = area_j + rarea[u];
            const float uni = sum - inter;
            const uint64_t hit = __builtin_amdgcn_ballot_w64(inter / uni > threshold &&
                                                             cj == rcat[u] && jon);
            bits = lane == r0 + u ? hit : bits;
        }
        if (jb == ib) {
            if (mine) out.own[i] = bits & ((uint64_t(1) << lane) - 1);   // higher ranks only
            continue;
        }
        const bool put = mine && bits != 0;
        const uint64_t pm = __ballot(put);
        if (pm == 0) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(count, __popcll(pm));
        at = uniform_i(at) + __popcll(pm & ((uint64_t(1) << lane) - 1));
        if (put) {
            out.word[list + at] = bits;
            out.tag[list + at] = static_cast<uint16_t>(lane | jb << 6);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && n > 64) out.len[(ib << lg) + s] = *count;
}

// Up to M blocks per wave: n <= 1024 M boxes; kCap listed words in LDS (the rest, if any, are
// read from memory in every round).
template <int M>
struct ResolveSmem {
    static constexpr int kCap = 1536 * M;
    uint64_t kept[16 * M];
    uint64_t done[16 * M];       // decided boxes
    uint64_t rem[16 * M];        // a kept box overlaps
    uint64_t pend[16 * M];       // an undecided box overlaps
    uint64_t word[kCap];
    uint16_t col[kCap];          // the word's index
    uint16_t row[kCap];          // its box
    int32_t first[(16 * M << kNmsSplitLog) + 1];   // each list's first entry
    int32_t part[40];
};

// Decides the n boxes; sm.kept holds the result after the call.  By 1024 threads: wave w has
// blocks w, w + 16, ..., lane = box.
constexpr int kNmsResolveThreads = 1024;
template <int M>
__device__ __forceinline__ void resolve_rows(uint64_t *ws, int n, int lg, ResolveSmem<M> &sm) {
    constexpr int kWaves = kNmsResolveThreads / 64;
    constexpr int kCap = ResolveSmem<M>::kCap;
    static_assert(kNmsResolveThreads == kPlanThreads, "block_exclusive_scan's workgroup");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = uniform_i(tid >> 6);
    const int nb = (n + 63) >> 6;
    const int nl = nb > 1 ? nb << lg : 0;
    const int sp = (1 << lg) - 1;
    const NmsLists in = nms_lists(ws, n);
    uint64_t own[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int i = (wave + kWaves * m) * 64 + lane;
        own[m] = i < n ? in.own[i] : 0;
    }
    for (int w = tid; w < kWaves * M; w += kNmsResolveThreads) {
        sm.kept[w] = 0;
        sm.done[w] = 0;
        sm.rem[w] = 0;
        sm.pend[w] = 0;
    }
    // (a length is at most the list's room: block b's rows by its words)
    for (int l = tid; l < nl; l += kNmsResolveThreads)
        sm.first[l] = max(0, min(in.len[l], 64 * nms_split_words(l >> lg, l & sp, lg)));
    __syncthreads();
    const int total = block_exclusive_scan(sm.first, nl, sm.part);
    if (tid == 0) sm.first[nl] = total;
    __syncthreads();
    // entry e: its word, word index and box
    auto entry = [&](int e, uint64_t &x, int &w, int &i) {
        int lo = 0, hi = nl;   // the list that holds e: first[lo] <= e < first[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (sm.first[mid] <= e) lo = mid;
            else hi = mid;
        }
        const int at = nms_list_base(n, lo >> lg, lo & sp, lg) + e - sm.first[lo];
        const int t = in.tag[at];
        x = in.word[at];
        w = min(t >> 6, lo >> lg);
        i = min((lo >> lg) * 64 + (t & 63), n - 1);
    };
    const int held = min(total, kCap);
    for (int e0 = tid; e0 < held; e0 += 4 * kNmsResolveThreads) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kNmsResolveThreads;
            if (e < held) {
                uint64_t x;
                int w, i;
                entry(e, x, w, i);
                sm.word[e] = x;
                sm.col[e] = static_cast<uint16_t>(w);
                sm.row[e] = static_cast<uint16_t>(i);
            }
        }
    }
    uint64_t und[M], kb[M];          // uniform: undecided and kept boxes of the block
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int rows = min(64, n - (wave + kWaves * m) * 64);
        und[m] = rows >= 64 ? ~uint64_t(0) : rows > 0 ? (uint64_t(1) << rows) - 1 : 0;
        kb[m] = 0;
    }
    int left;
    do {
        __syncthreads();   // the last round's verdicts (or the entries) are in LDS
        // every listed word of an undecided box against the decided ones
        auto look = [&](uint64_t x, int w, int i) {
            const uint64_t bit = uint64_t(1) << (i & 63);
            if (sm.done[i >> 6] & bit) return;
            if (x & sm.kept[w])
                atomicOr(reinterpret_cast<unsigned long long *>(&sm.rem[i >> 6]), bit);
            else if (x & ~sm.done[w])
                atomicOr(reinterpret_cast<unsigned long long *>(&sm.pend[i >> 6]), bit);
        };
        for (int e = tid; e < held; e += kNmsResolveThreads) look(sm.word[e], sm.col[e], sm.row[e]);
        for (int e = held + tid; e < total; e += kNmsResolveThreads) {
            uint64_t x;
            int w, i;
            entry(e, x, w, i);
            look(x, w, i);
        }
        __syncthreads();
        bool more = false;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            if (und[m] == 0) continue;
            const int b = wave + kWaves * m;
            uint64_t U = und[m] & ~sm.rem[b];
            uint64_t K = kb[m];
            const uint64_t P = sm.pend[b];
            for (;;) {
                const bool on = (U >> lane) & 1;
                const uint64_t rm = __ballot(on && (own[m] & K) != 0);
                U &= ~rm;
                const uint64_t kn = __ballot(on && (own[m] & (U | K)) == 0) & U & ~P;
                K |= kn;
                U &= ~kn;
                if ((rm | kn) == 0) break;
            }
            und[m] = U;
            kb[m] = K;
            if (lane == 0) {
                sm.kept[b] = K;
                sm.done[b] = ~U;
                sm.pend[b] = 0;
            }
            more = more || U != 0;
        }
        left = __syncthreads_or(more);
    } while (left);
}

// Kept boxes of all blocks, and those before block b (every lane of a wave).
__device__ __forceinline__ int kept_before(const uint64_t *kept, int b, int lane) {
    int before = 0;
    for (int c = lane; c < b; c += 64) before += __popcll(kept[c]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
    return before;
}

}  // namespace rex
