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
//                  none), so the waves take the blocks of 64 in turn without a barrier between
//                  them: each reads its block's listed words once, sees in LDS what the other
//                  waves have decided, waits only for the boxes it depends on, and decides its
//                  own overlaps by ballots.
//                  (8192 boxes of two images that hardly overlap: 22 us; around 10 objects an
//                  image, 300 thousand listed words: the call 300 us.  All words again in every
//                  round, barriers between the rounds: 22 us, the call 4150; one block after the
//                  other, barriers for each: 461 us, the call 445.)
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

// OR over the 64 lanes (uniform), in DPP moves (see wave_inclusive_scan).
__device__ __forceinline__ uint32_t wave_or_u32(uint32_t x) {
    int v = static_cast<int>(x);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(v, 63));
}
// Bits `row` of the lanes with `on`.
__device__ __forceinline__ uint64_t wave_rows(bool on, int row) {
    if (__ballot(on) == 0) return 0;
    const uint64_t bit = on ? uint64_t(1) << row : 0;
    return static_cast<uint64_t>(wave_or_u32(static_cast<uint32_t>(bit >> 32))) << 32 |
           wave_or_u32(static_cast<uint32_t>(bit));
}

// Up to M blocks per wave: n <= 1024 M boxes.
constexpr int kNmsResolveThreads = 1024;
constexpr int kNmsResolveWaves = kNmsResolveThreads / 64;
constexpr int kNmsWaiting = 256;    // words of a block that wait, per wave
template <int M>
struct ResolveSmem {
    uint64_t kept[kNmsResolveWaves * M];   // decided boxes of each block: kept, and
    uint64_t gone[kNmsResolveWaves * M];   // removed
    int32_t len[kNmsResolveWaves * M << kNmsSplitLog];
    uint64_t word[kNmsResolveWaves][kNmsWaiting];
    uint16_t tag[kNmsResolveWaves][kNmsWaiting];
};

// A word of other waves' LDS state.  Bits of kept and gone are only ever set, each by the one
// wave that has the block, so a reader needs no order between them: a bit not seen yet reads as
// undecided and is looked at again.
__device__ __forceinline__ uint64_t nms_peek(const uint64_t &x) {
    return __hip_atomic_load(&x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void nms_post(uint64_t &x, uint64_t v) {
    __hip_atomic_store(&x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Decides the n boxes; sm.kept holds the result after the call.  By 1024 threads: wave w has
// blocks w, w + 16, ... in this order, lane = box.  A block's listed words are read once: a word
// with a kept box removes its row, one whose boxes are all removed is done with, and one with
// undecided boxes waits in LDS.  Then the wave looks at the waiting words of its undecided rows
// until all rows are decided, which needs blocks before its own only: of the blocks not decided,
// the first is the one its wave works on, and nothing it waits for is left, so every wait ends.
// The scan of a block ends when its rows are all removed, as in a crowd they soon are.
template <int M, int LG>
__device__ __forceinline__ void resolve_rows(uint64_t *ws, int n, ResolveSmem<M> &sm) {
    constexpr int kWaves = kNmsResolveWaves;
    constexpr int kLists = 1 << LG;
    constexpr int kGroup = 4;   // loads of 64 words in flight
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = uniform_i(tid >> 6);
    const int nb = (n + 63) >> 6;
    const NmsLists in = nms_lists(ws, n);
    for (int w = tid; w < kWaves * M; w += kNmsResolveThreads) {
        sm.kept[w] = 0;
        sm.gone[w] = 0;
    }
    // (a length is at most the list's room: block b's rows by its words; one block has no lists)
    for (int l = tid; l < nb << LG; l += kNmsResolveThreads)
        sm.len[l] = nb > 1 ? max(0, min(in.len[l], min(64, n - 64 * (l >> LG)) *
                                                       nms_split_words(l >> LG, l & (kLists - 1), LG)))
                           : 0;
    __syncthreads();

    // A block's lists as one sequence: list s holds the entries from end[s - 1] to end[s].
    struct Lists {
        int b, total;
        int end[kLists];
    };
    auto lists_of = [&](int b, Lists &q) {
        q.b = b;
        q.total = 0;
        if (b >= nb) return;
        const int incl = wave_inclusive_scan(lane < kLists ? sm.len[(b << LG) + (lane & (kLists - 1))] : 0, lane);
#pragma unroll
        for (int s = 0; s < kLists; ++s) q.end[s] = __builtin_amdgcn_readlane(incl, s);
        q.total = q.end[kLists - 1];
    };
    struct Group {
        uint64_t x[kGroup];
        int t[kGroup];
    };
    auto load = [&](const Lists &q, int e0, Group &g) {   // entries [e0, e0 + 64 kGroup)
        const int rows = min(64, n - 64 * q.b);
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            g.x[u] = 0;
            g.t[u] = 0;
            if (e0 + 64 * u >= q.total) continue;
            const int e = e0 + 64 * u + lane;
            int s = 0, from = 0;
#pragma unroll
            for (int l = 0; l + 1 < kLists; ++l) {
                s += e >= q.end[l] ? 1 : 0;
                from = e >= q.end[l] ? q.end[l] : from;
            }
            if (e < q.total) {
                const int at = 32 * q.b * (q.b - 1) + e - from +
                               rows * (s * (q.b >> LG) + min(s, q.b & (kLists - 1)));
                g.x[u] = in.word[at];
                g.t[u] = in.tag[at];
            }
        }
    };

    uint64_t *const wword = sm.word[wave];
    uint16_t *const wtag = sm.tag[wave];
    auto own_of = [&](int b) { return b * 64 + lane < n ? in.own[b * 64 + lane] : uint64_t(0); };
    Lists cur;
    Group grp;
    lists_of(wave, cur);
    uint64_t own = wave < nb ? own_of(wave) : 0;
    load(cur, 0, grp);
    for (int b = wave; b < nb; b += kWaves) {
        const int rows = min(64, n - 64 * b);
        const uint64_t all = rows >= 64 ? ~uint64_t(0) : (uint64_t(1) << rows) - 1;
        uint64_t U = all, K = 0;   // uniform: the block's undecided and kept boxes
        Lists nxt;
        lists_of(b + kWaves, nxt);
        const uint64_t own_next = b + kWaves < nb ? own_of(b + kWaves) : 0;
        int waiting = 0;
        // One word of row t & 63, of block t >> 6's boxes: removes the row, waits or neither.
        auto look = [&](uint64_t x, int t, bool &rem, bool &wait) {
            const int w = min(t >> 6, b - 1);
            const bool on = x != 0 && ((U >> (t & 63)) & 1);
            const uint64_t k = on ? nms_peek(sm.kept[w]) : 0;
            const uint64_t g = on ? nms_peek(sm.gone[w]) : 0;
            rem = (x & k) != 0;
            wait = on && !rem && (x & ~g) != 0;
        };
        auto put = [&](uint64_t x, int t, bool wait, int at) {
            const uint64_t m = __ballot(wait);
            const int p = at + __popcll(m & ((uint64_t(1) << lane) - 1));
            if (wait) {
                wword[p] = x;
                wtag[p] = static_cast<uint16_t>(t);
            }
            return __popcll(m);
        };
        // Another look at the waiting words; returns the rows that still wait.
        auto sweep = [&]() {
            uint64_t pend = 0;
            int left = 0;
            wave_sync();
            for (int e = 0; e < waiting; e += 64) {
                const bool in_queue = e + lane < waiting;
                const uint64_t x = in_queue ? wword[e + lane] : 0;
                const int t = in_queue ? wtag[e + lane] : 0;
                bool rem, wait;
                look(x, t, rem, wait);
                wave_sync();   // read before the words before them move down
                U &= ~wave_rows(rem, t & 63);
                pend |= wave_rows(wait, t & 63);
                left += put(x, t, wait, left);
            }
            waiting = left;
            wave_sync();
            return pend;
        };
        // What the block can decide itself, but for the rows in pend, and the word of it.
        auto decide = [&](uint64_t pend) {
            for (;;) {
                const bool on = (U >> lane) & 1;
                const uint64_t rm = __ballot(on && (own & K) != 0);
                U &= ~rm;
                const uint64_t kn = __ballot(on && (own & (U | K)) == 0) & U & ~pend;
                K |= kn;
                U &= ~kn;
                if ((rm | kn) == 0) break;
            }
            if (lane == 0) {
                nms_post(sm.kept[b], K);
                nms_post(sm.gone[b], all & ~(U | K));
            }
        };

        const Group g0 = grp;
        if (cur.total <= 64) {   // few overlaps: the words stay in registers
            load(nxt, 0, grp);
            for (;;) {
                bool rem, wait;
                look(g0.x[0], g0.t[0], rem, wait);
                const uint64_t before = U;
                U &= ~wave_rows(rem, g0.t[0] & 63);
                decide(wave_rows(wait, g0.t[0] & 63));
                if (U == 0) break;
                if (U == before) __builtin_amdgcn_s_sleep(1);
            }
        } else {
            bool fetched = false;   // grp holds the next block's first words
            for (int e0 = 0; e0 < cur.total && U != 0; e0 += 64 * kGroup) {
                const Group g = grp;
                const bool more = e0 + 64 * kGroup < cur.total;
                load(more ? cur : nxt, more ? e0 + 64 * kGroup : 0, grp);
                fetched = !more;
#pragma unroll
                for (int u = 0; u < kGroup; ++u) {
                    if (e0 + 64 * u >= cur.total) continue;
                    while (waiting > kNmsWaiting - 64) sweep();
                    bool rem, wait;
                    look(g.x[u], g.t[u], rem, wait);
                    U &= ~wave_rows(rem, g.t[u] & 63);
                    waiting += put(g.x[u], g.t[u], wait, waiting);
                }
            }
            if (!fetched) load(nxt, 0, grp);
            for (;;) {
                const uint64_t before = U;
                decide(waiting > 0 ? sweep() : 0);
                if (U == 0) break;
                if (U == before) __builtin_amdgcn_s_sleep(1);
            }
        }
        cur = nxt;
        own = own_next;
    }
    __syncthreads();
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
