// nms.hip -- greedy non-maximum suppression of scored boxes.
//
// The proposals a two-stage detector extracts RoI features for come out of NMS over
// the dense head's scored boxes; MMDetection runs such bbox operations on the GPU (§1).
// Definition (rank order, tie rules, binary32 IoU decision) in include/roi_extract.h.
//
// Three kernels on one stream:
//   nms_rank_kernel      a box's rank is the number of boxes before it in rank order, so
//                        every workgroup counts the ranks of 32 boxes against all keys in
//                        LDS (N^2 compares over the whole GPU instead of a sort in one
//                        workgroup) and writes them to their place
//   nms_overlap_kernel   each box's overlaps with the boxes of higher rank (nms.hpp)
//   nms_resolve_kernel   one workgroup decides every box (nms.hpp) and writes the kept
//                        indices in rank order
//
// 8192 boxes of two categories: 82 (bitonic sort) -> 11 us, 42 -> 23 us, 461 (blocks
// walked in order) -> 22 us; the call 585 -> 53 us.
#include "nms.hpp"

namespace rex {

constexpr int kNmsRankThreads = 1024;
constexpr int kNmsRankBoxes = 32;   // per workgroup

// Lane = (box, half): the two halves of a wave take alternate groups of four keys of the
// wave's sixteenth of all keys.  Before the workgroup's own boxes equal keys rank first,
// after them last; only among them are indices compared.
__global__ __launch_bounds__(kNmsRankThreads) void nms_rank_kernel(NmsArgs a) {
    __shared__ __align__(16) uint32_t keys[kNmsMaxBoxes];
    __shared__ int32_t part[kNmsRankThreads / 64][kNmsRankBoxes];
    const int N = a.N;
    constexpr int kWaves = kNmsRankThreads / 64;
    const int chunk = ((N + kWaves - 1) / kWaves + 7) & ~7;
    const int padded = min(chunk * kWaves, kNmsMaxBoxes);
    for (int j = threadIdx.x; j < padded; j += kNmsRankThreads)
        keys[j] = j < N ? nms_key(a.scores[j]) : 0xffffffffu;   // padding precedes no box
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = uniform_i(threadIdx.x >> 6);
    const int half = lane >> 5;
    const int I0 = static_cast<int>(blockIdx.x) * kNmsRankBoxes;
    const int i = I0 + (lane & 31);
    const uint32_t ki = i < N ? keys[i] : 0u;
    const int c0 = min(wave * chunk, padded), c1 = min(c0 + chunk, padded);
    int cnt = 0;
    const int e0 = min(c1, I0);
    for (int j = c0; j < e0; j += 8) {
        const uint4 k = *reinterpret_cast<const uint4 *>(&keys[j + 4 * half]);
        cnt += (k.x <= ki) + (k.y <= ki) + (k.z <= ki) + (k.w <= ki);
    }
    const int e1 = min(c1, I0 + kNmsRankBoxes);
    for (int j = max(c0, I0); j < e1; j += 8) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jj = j + 4 * half + u;
            const uint32_t k = keys[jj];
            cnt += (k < ki || (k == ki && jj < i)) ? 1 : 0;
        }
    }
    for (int j = max(c0, I0 + kNmsRankBoxes); j < c1; j += 8) {
        const uint4 k = *reinterpret_cast<const uint4 *>(&keys[j + 4 * half]);
        cnt += (k.x < ki) + (k.y < ki) + (k.z < ki) + (k.w < ki);
    }
    cnt += __shfl_xor(cnt, 32);
    if (half == 0) part[wave][lane] = cnt;
    __syncthreads();
    if (threadIdx.x < kNmsRankBoxes && i < N) {
        int r = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) r += part[w][lane];
        a.order[r] = i;
        const float *b = a.boxes + 4 * static_cast<int64_t>(i);
        a.sboxes[r] = make_float4(b[0], b[1], b[2], b[3]);
        a.scats[r] = a.categories ? a.categories[i] : 0;
    }
}

__global__ __launch_bounds__(kNmsOverlapThreads) void nms_overlap_kernel(NmsArgs a, float share) {
    __shared__ int32_t count;
    overlap_rows(a.sboxes, a.scats, a.N, a.threshold, share, a.mask,
                 static_cast<int>(blockIdx.x) >> kNmsSplitLog,
                 static_cast<int>(blockIdx.x) & ((1 << kNmsSplitLog) - 1), kNmsSplitLog, &count);
}

template <int M>
__global__ __launch_bounds__(kNmsResolveThreads) void nms_resolve_kernel(NmsArgs a) {
    __shared__ ResolveSmem<M> sm;
    resolve_rows<M, kNmsSplitLog>(a.mask, a.N, sm);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nb = (a.N + 63) >> 6;
    const int limit = static_cast<int>(min<int64_t>(a.max_keep, a.N));
    // a block's first rank is the kept count of the blocks before it
    for (int b = wave; b < nb; b += kNmsResolveThreads / 64) {
        const int before = kept_before(sm.kept, b, lane);
        const uint64_t kept = sm.kept[b];
        if ((kept >> lane) & 1) {
            const int rank = before + __popcll(kept & ((uint64_t(1) << lane) - 1));
            if (rank < limit) a.keep[rank] = a.order[b * 64 + lane];
        }
    }
    const int n = min(kept_before(sm.kept, nb, lane), limit);
    for (int r = n + static_cast<int>(threadIdx.x); r < limit; r += kNmsResolveThreads) a.keep[r] = -1;
    if (threadIdx.x == 0) a.num_keep[0] = n;
}

hipError_t launch_nms(NmsArgs a, hipStream_t stream) {
    if (a.N > 0) {
        nms_rank_kernel<<<static_cast<uint32_t>((a.N + kNmsRankBoxes - 1) / kNmsRankBoxes),
                          kNmsRankThreads, 0, stream>>>(a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        nms_overlap_kernel<<<static_cast<uint32_t>(a.nw << kNmsSplitLog), kNmsOverlapThreads, 0, stream>>>(
            a, nms_share(a.threshold));
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // blocks per wave; no boxes: the count only
    if (a.nw <= 16) nms_resolve_kernel<1><<<1, kNmsResolveThreads, 0, stream>>>(a);
    else if (a.nw <= 48) nms_resolve_kernel<3><<<1, kNmsResolveThreads, 0, stream>>>(a);
    else nms_resolve_kernel<8><<<1, kNmsResolveThreads, 0, stream>>>(a);
    return hipGetLastError();
}

}  // namespace rex
