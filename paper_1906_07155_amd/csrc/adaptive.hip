// adaptive.hip -- RoIAlign with any sampling ratio on the 7x7 and 14x14 grids: the
// adaptive grid (sampling_ratio 0: ceil(bin) samples per bin and axis) and fixed ratios
// other than 2, on channels-last levels (forward) and on any levels the tile gather
// addresses (backward).
//
// The sample positions of a RoI are separable whatever their number, so its output is
//     out[ph][pw] = 1/count * sum_y sum_x Wy[ph][y] * Wx[pw][x] * F[y][x]
// over the pixel rows y and columns x its samples tap, Wy and Wx the summed bilinear
// weights of the bin's samples.  The number of samples then only enters the weights: the
// kernels load (or write) every footprint pixel once, as the two-samples kernels do, and
// not once per sample and corner.
//
//   fwd_any_kernel         (RoI, slice of channels) per workgroup, lanes over channels
//   bwd_gather_any_kernel  the tile gather: (bin-tile, 64 channels) per workgroup
//   bwd_stray_kernel       scatter of the RoIs whose level is not the plan's (normally
//                          none): the tile lists do not hold them
//
// Batch of 3 x 171 RoIs, 256 binary32 channels, 608 x 1056 images, adaptive grid, against
// one thread per output element with four taps (atomics) per sample:
//   forward 618 -> 44 us, backward 24 (clearing) + 9996 -> 58 + 4 us (stray pass).
#include <algorithm>

#include "gather.hpp"

namespace rex {

constexpr int kAnyGrid = kGridCap;   // samples per bin and axis at most (RE_MAX_SAMPLING)

// Position of sample i of bin p after the cut and the clamp: -2 marks a sample off the
// map, anything else is in [0, size - 1] and its taps are (int)v and, unless that is the
// last pixel, the next one with weight v - (int)v (the steps of axis_tap).
__device__ __forceinline__ float any_position(const Axis &a, int p, int i, int size) {
    const float t1 = static_cast<float>(p) * a.bin;
    const float t2 = a.start + t1;
    const float t3 = static_cast<float>(i) + 0.5f;
    const float t4 = t3 * a.bin;
    const float t5 = t4 / static_cast<float>(a.grid);
    float v = t2 + t5;
    if (v < -1.0f || v > static_cast<float>(size)) return -2.0f;
    v = fmaxf(v, 0.0f);
    return static_cast<int>(v) >= size - 1 ? static_cast<float>(size - 1) : v;
}

// The samples i0..i1 of bin p that can tap pixel X of the axis: only those whose position
// before the clamp is within a pixel of X and, for X <= 1, all those clamped up to 0.  The
// positions are evenly spaced, so they are an index range, widened by one and by what the
// rounding of a position and of `rel` comes to in units of the spacing: at most 8 units of
// 2^-24 of the coordinate (samples closer than that round to one position) and of the box,
// whose part the widening by one covers.  A box without extent takes all samples.
__device__ __forceinline__ void any_window(const Axis &a, int p, int X, int &i0, int &i1) {
    const float g = static_cast<float>(a.grid);
    i0 = 0;
    i1 = a.grid - 1;
    if (a.bin > 0.0f) {
        const float inv = g * __builtin_amdgcn_rcpf(a.bin);
        const float rel = (static_cast<float>(X) - a.start) - static_cast<float>(p) * a.bin;
        const float slack = (static_cast<float>(X) + 2.0f) * inv * 0x1p-21f;
        const float lo = (rel - 1.0f) * inv - (1.5f + slack);   // floor - 1 of the first index
        const float hi = (rel + 1.0f) * inv + (0.5f + slack);   // ceil + 1 of the last
        if (X > 1 && lo > 0.0f) i0 = static_cast<int>(fminf(lo, g));
        if (hi < g - 1.0f) i1 = static_cast<int>(fmaxf(hi, -1.0f));
    }
}

// Summed weight the samples of bin p put on pixel X, and whether any of them taps it (also
// with weight zero).  pos holds the bin's positions.
__device__ __forceinline__ float any_weight(const float *pos, const Axis &a, int p, int X, int size,
                                            bool &hit) {
    int i0, i1;
    any_window(a, p, X, i0, i1);
    float w = 0.0f;
    hit = false;
#pragma unroll 1
    for (int i = i0; i <= i1; ++i) {
        const float v = pos[i];
        const int l = static_cast<int>(v);
        const float f = v - static_cast<float>(l);
        const bool a0 = v >= 0.0f && l == X;
        const bool a1 = v >= 0.0f && l + 1 == X && l < size - 1;
        w += a0 ? 1.0f - f : 0.0f;
        w += a1 ? f : 0.0f;
        hit = hit || a0 || a1;
    }
    return w;
}

// Positions of every sample of both axes into pos ([bin][sample] of the rows, then of the
// columns at kAnyGrid * P), by the whole workgroup.
template <int P, int NT = 256>
__device__ __forceinline__ void any_positions(const Axis &ay, const Axis &ax, int H, int W,
                                              float *pos) {
    const int ny = P * ay.grid, n = ny + P * ax.grid;
    for (int e = threadIdx.x; e < n; e += NT) {
        const bool row = e < ny;
        const int u = row ? e : e - ny;
        const int g = row ? ay.grid : ax.grid;
        const int p = small_div_exact(u, g);
        Axis a;
        a.start = row ? ay.start : ax.start;
        a.bin = row ? ay.bin : ax.bin;
        a.grid = g;
        pos[(row ? 0 : kAnyGrid * P) + u] = any_position(a, p, u - p * g, row ? H : W);
    }
}

// ---------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------
//
// As the two-samples kernel (fwd.hip): wave w owns bin rows [w * RPW, (w + 1) * RPW) and
// loads the pixel rows they tap times the RoI's columns, in chunks of CX columns with D
// units (chunk, row) in flight; each row is weighted into the wave's bin rows, and at the
// end of a chunk its columns are reduced into the bin columns that tap them.  Rows and columns
// are walked in panels of kAnyRows (per wave) and kAnyCols slots, each with its own weights (a
// box may span the whole map).  A slot is a pixel row or column of the run from the first
// tapped to the last, or, where the run is longer than the samples have taps (few samples in
// wide bins: most of the run is not tapped), one tap of one sample.  (One 200 x 336 level, boxes
// of 200 to 800 pixels at stride 4, 7x7, S = 1 / 3 / 4: 14 / 66 / 105 us, runs always: 253 /
// 478 / 514, one thread per output element: 57 / 585 / 1120.)
constexpr int kAnyCols = 64;
constexpr int kAnyRows = 32;

template <typename T, int CPL>
struct AnyPix {
    static constexpr int W = (static_cast<int>(sizeof(T)) * CPL + 3) / 4;
    uint32_t w[W];
};

template <typename T, int CPL>
__device__ __forceinline__ void any_load(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff,
                                         AnyPix<T, CPL> &p) {
    static_assert(sizeof(T) * CPL <= 4, "one 32-bit register per lane and pixel");
    if constexpr (sizeof(T) * CPL == 4) p.w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0);
    else p.w[0] = __builtin_amdgcn_raw_buffer_load_b16(r, off, soff, 0);
}

template <typename T, int CPL>
__device__ __forceinline__ float any_value(const AnyPix<T, CPL> &p, int j) {
    if constexpr (sizeof(T) == 4) return __uint_as_float(p.w[0]);
    else if constexpr (CPL == 1) return __uint_as_float(p.w[0] << 16);
    else return __uint_as_float(j == 0 ? (p.w[0] << 16) : (p.w[0] & 0xffff0000u));
}

template <int P, int CHK, int NW>
struct AnyFwdSmem {
    float pos[2 * P * kAnyGrid];
    __align__(16) float wx[P][kAnyCols];
    __align__(16) float wy[NW][kAnyRows][NW == 4 ? 4 : 1];   // [wave][row][bin row of the wave]
    __align__(16) uint32_t xoff[kAnyCols];    // byte offsets of the panel's columns
    uint64_t hit[P];                          // columns of the panel a bin column taps
    __align__(16) float stile[CHK * P * P];
};

// Tap j of the samples at pos: sample j / 2, its lower pixel for even j, the upper one (the same
// on the last pixel, with weight zero) for odd j; false for a sample off the map.
__device__ __forceinline__ bool any_tap(const float *pos, int j, int size, int &pixel, float &w) {
    const float v = pos[j >> 1];
    const int l = static_cast<int>(v);
    const float f = v - static_cast<float>(l);
    pixel = (j & 1) ? min(l + 1, size - 1) : l;
    w = (j & 1) ? f : 1.0f - f;
    return v >= 0.0f;
}

// Column offsets come from an LDS table and not from registers kept over a chunk's rows (the
// registers cost a wave per SIMD: 70 us against 44 us on the batch above); five waves per
// SIMD by spilling 12 registers is slower too (50 us).
template <typename T, typename TO, int P, int CX, int CHK, int CPL, int D, int NW>
__global__ __launch_bounds__(64 * NW) void fwd_any_kernel(FwdArgs args) {
    constexpr int NB = P * P;
    constexpr int RPW = (P + NW - 1) / NW;    // bin rows per wave
    static_assert(NW == 4 || RPW == 1, "AnyFwdSmem::wy");
    constexpr int SLICE = 64 * CPL;
    static_assert(RPW <= 4 && 64 % kAnyRows == 0 && kAnyCols == 64 && kAnyCols % CX == 0, "tables");
    __shared__ AnyFwdSmem<P, CHK, NW> sm;
    (void)args;
    const FwdArgs &a = *(const FwdArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    const LevelTable &lv = a.lv;
    const uint32_t lid = xcd_remap(blockIdx.x, gridDim.x);
    const int slot = static_cast<int>(lid / static_cast<uint32_t>(a.wg_per_roi));
    const int sub = static_cast<int>(lid) - slot * a.wg_per_roi;
    const int slice0 = sub * a.spw;
    const int slice1 = min(a.nslices, slice0 + a.spw);
    int k = uniform_i(a.perm ? a.perm[slot] : slot);
    const bool kvalid = k >= 0 && k < a.K;
    if (!kvalid) k = 0;
    const float *r = a.rois + 5 * static_cast<int64_t>(k);
    const float rb = r[0], x1 = r[1], y1 = r[2], x2 = r[3], y2 = r[4];
    const int lvl = uniform_i(a.roi_levels ? a.roi_levels[k] : 0);
    const bool lvalid = lvl >= 0 && lvl < lv.num;
    const LevelArg L = level_at(lv, lvalid ? lvl : 0);
    const int b = roi_batch(rb, lv.N);
    Axis ax = axis_setup(x1, x2, L.scale, a.aligned, P, a.S);
    Axis ay = axis_setup(y1, y2, L.scale, a.aligned, P, a.S);
    ax.grid = uniform_i(ax.grid);
    ay.grid = uniform_i(ay.grid);
    // an adaptive grid may be empty (a box without extent): every output is zero
    const bool active = kvalid && lvalid && b >= 0 && ax.grid > 0 && ay.grid > 0;

    const int t = threadIdx.x;
    const int wave = uniform_i(t >> 6);
    const int lane = t & 63;
    const int p0 = min(P, wave * RPW);
    const int p1 = min(P, p0 + RPW);
    const uint32_t sh_b = static_cast<uint32_t>(L.sh * int64_t(sizeof(T)));
    const uint32_t sw_b = static_cast<uint32_t>(L.sw * int64_t(sizeof(T)));
    const float *const ypos = sm.pos;
    const float *const xpos = sm.pos + kAnyGrid * P;

    if (active) any_positions<P, 64 * NW>(ay, ax, L.H, L.W, sm.pos);
    __syncthreads();
    // The wave's tapped rows and the RoI's tapped columns (every wave finds them itself).
    int ya = 0, ny = 0, xa = 0, xb = 0, nx = 0;
    if (active) {
        float ylo = 3e38f, yhi = -1.0f, xlo = 3e38f, xhi = -1.0f;
        for (int u = p0 * ay.grid + lane; u < p1 * ay.grid; u += 64) {
            const float v = ypos[u];
            if (v >= 0.0f) {
                ylo = fminf(ylo, v);
                yhi = fmaxf(yhi, v);
            }
        }
        for (int u = lane; u < P * ax.grid; u += 64) {
            const float v = xpos[u];
            if (v >= 0.0f) {
                xlo = fminf(xlo, v);
                xhi = fmaxf(xhi, v);
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            ylo = fminf(ylo, __shfl_xor(ylo, o));
            yhi = fmaxf(yhi, __shfl_xor(yhi, o));
            xlo = fminf(xlo, __shfl_xor(xlo, o));
            xhi = fmaxf(xhi, __shfl_xor(xhi, o));
        }
        if (yhi >= 0.0f) {
            ya = uniform_i(static_cast<int>(ylo));
            ny = uniform_i(min(static_cast<int>(yhi) + 1, L.H - 1)) - ya + 1;
        }
        if (xhi >= 0.0f) {
            xa = uniform_i(static_cast<int>(xlo));
            xb = uniform_i(min(static_cast<int>(xhi) + 1, L.W - 1));
            nx = xb - xa + 1;
        }
    }
    // slots: the run's pixels or, if fewer, the samples' taps
    const bool xtaps = nx > 2 * P * ax.grid;                // the same in every wave
    const bool ytaps = ny > 2 * (p1 - p0) * ay.grid;        // the wave's own, as its rows
    const int nxs = xtaps ? 2 * P * ax.grid : nx;
    const int nys = ytaps ? 2 * (p1 - p0) * ay.grid : ny;
    const int npx = (nxs + kAnyCols - 1) / kAnyCols;
    const int npy = (nys + kAnyRows - 1) / kAnyRows;
    const float inv_count = 1.0f / static_cast<float>(max(ay.grid * ax.grid, 1));

    uint32_t cmask = 0;
    int yoff = 0;   // byte offset of the panel's row `lane` (the lower half's lanes)
    for (int slice = slice0; slice < slice1; ++slice) {
        if (slice > slice0) __syncthreads();   // the previous slice's output tile is stored
        const int c = slice * SLICE + lane * CPL;
        const bool lane_on = active && c < lv.C;
        const char *img = static_cast<const char *>(L.data) +
                          (active ? static_cast<int64_t>(b) * L.sn * int64_t(sizeof(T)) : 0);
        const __amdgpu_buffer_rsrc_t res = make_rsrc(img, L.img_bytes);
        const uint32_t vbase = lane_on ? static_cast<uint32_t>(c) * uint32_t(sizeof(T)) : kBufOOB;

        float acc[CPL][RPW][P];
#pragma unroll
        for (int j = 0; j < CPL; ++j)
#pragma unroll
            for (int p = 0; p < RPW; ++p)
#pragma unroll
                for (int q = 0; q < P; ++q) acc[j][p][q] = 0.0f;

        for (int px = 0; px < npx; ++px) {
            const int X0 = px * kAnyCols;
            // column weights of the panel: a wave takes whole bin columns, lane = column
            if (slice == slice0 || npx > 1) {
                if (px > 0 || slice > slice0) __syncthreads();   // the last panel is consumed
                // columns past the last slot repeat the last pixel (their weights are zero)
                int X = min(xa + X0 + lane, xb), xq = 0;
                float xw = 0.0f;
                bool xon = X0 + lane < nxs;
                if (xtaps && xon) {
                    xon = any_tap(xpos, X0 + lane, L.W, X, xw);
                    xq = small_div_exact((X0 + lane) >> 1, ax.grid);
                }
                if (wave == 3) sm.xoff[lane] = xtaps && !xon ? kBufOOB : static_cast<uint32_t>(X) * sw_b;
                for (int q = wave; q < P; q += NW) {
                    bool h = xon && xq == q;
                    float w = h ? xw : 0.0f;
                    if (!xtaps) {
                        h = false;
                        if (xon) w = any_weight(xpos + q * ax.grid, ax, q, X, L.W, h);
                    }
                    sm.wx[q][lane] = w;
                    const uint64_t m = __ballot(h);
                    if (lane == 0) sm.hit[q] = m;
                }
                __syncthreads();
                // bin columns each chunk of CX columns reaches, lane = chunk
                cmask = 0;
                if (lane < kAnyCols / CX) {
#pragma unroll
                    for (int q = 0; q < P; ++q)
                        cmask |= ((sm.hit[q] >> (lane * CX)) & ((1u << CX) - 1u)) ? 1u << q : 0u;
                }
            }
            const int nch = (min(kAnyCols, nxs - X0) + CX - 1) / CX;
            for (int py = 0; py < npy; ++py) {
                const int Y0 = py * kAnyRows;
                const int rows = min(kAnyRows, nys - Y0);
                // row weights of the panel (the wave's own): lanes over (bin row, row)
                if ((slice == slice0 && px == 0) || npy > 1) {
                    wave_sync();   // the last panel's are consumed
#pragma unroll
                    for (int pp = 0; pp < (RPW * kAnyRows + 63) / 64; ++pp) {
                        const int u = pp * 64 + lane;
                        const int p = u / kAnyRows, y = u % kAnyRows;
                        int Y = ya + Y0 + y;
                        float w = 0.0f;
                        bool h = false;
                        if (ytaps && y < rows) {
                            h = any_tap(ypos + p0 * ay.grid, Y0 + y, L.H, Y, w);
                            if (!h || small_div_exact((Y0 + y) >> 1, ay.grid) != p) w = 0.0f;
                        } else if (p < RPW && p0 + p < p1 && y < rows) {
                            w = any_weight(ypos + (p0 + p) * ay.grid, ay, p0 + p, Y, L.H, h);
                        }
                        if (p < RPW) sm.wy[wave][y][p] = w;
                        if (pp == 0) yoff = static_cast<int>(ytaps && !h ? kBufOOB : static_cast<uint32_t>(Y) * sh_b);
                    }
                    wave_sync();
                }
                float H[CPL][CX][RPW];
#pragma unroll
                for (int j = 0; j < CPL; ++j)
#pragma unroll
                    for (int x = 0; x < CX; ++x)
#pragma unroll
                        for (int p = 0; p < RPW; ++p) H[j][x][p] = 0.0f;

                auto issue = [&](int ch, int yi, AnyPix<T, CPL> (&v)[CX]) {
                    const uint32_t rowb = vbase + static_cast<uint32_t>(__builtin_amdgcn_readlane(yoff, yi));
                    const uint32_t *xo = sm.xoff + ch * CX;
#pragma unroll
                    for (int x = 0; x < CX; ++x) any_load<T, CPL>(res, rowb + xo[x], 0, v[x]);
                };
                auto consume = [&](int ch, int yi, const AnyPix<T, CPL> (&v)[CX]) {
                    const float *wy = sm.wy[wave][yi];
#pragma unroll
                    for (int x = 0; x < CX; ++x)
#pragma unroll
                        for (int j = 0; j < CPL; ++j) {
                            const float f = any_value<T, CPL>(v[x], j);
#pragma unroll
                            for (int p = 0; p < RPW; ++p) H[j][x][p] = fmaf(wy[p], f, H[j][x][p]);
                        }
                    if (yi == rows - 1) {
                        // the chunk's columns into the bin columns that tap them
                        const uint32_t m = __builtin_amdgcn_readlane(cmask, ch);
#pragma unroll
                        for (int q = 0; q < P; ++q) {
                            if (!((m >> q) & 1u)) continue;
                            float wq[CX];
#pragma unroll
                            for (int x4 = 0; x4 < CX; x4 += 4) {
                                const float4 w4 =
                                    *reinterpret_cast<const float4 *>(&sm.wx[q][ch * CX + x4]);
                                wq[x4] = w4.x;
                                wq[x4 + 1] = w4.y;
                                wq[x4 + 2] = w4.z;
                                wq[x4 + 3] = w4.w;
                            }
#pragma unroll
                            for (int x = 0; x < CX; ++x)
#pragma unroll
                                for (int j = 0; j < CPL; ++j)
#pragma unroll
                                    for (int p = 0; p < RPW; ++p)
                                        acc[j][p][q] = fmaf(wq[x], H[j][x][p], acc[j][p][q]);
                            __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                        for (int x = 0; x < CX; ++x)
#pragma unroll
                            for (int j = 0; j < CPL; ++j)
#pragma unroll
                                for (int p = 0; p < RPW; ++p) H[j][x][p] = 0.0f;
                    }
                };

                constexpr int NBUF = D + 1;
                AnyPix<T, CPL> v[NBUF][CX];
                const int units = rows * nch;
                int ic = 0, iy = 0, cc = 0, cy = 0;   // next unit to issue, to consume
                auto issue_next = [&](AnyPix<T, CPL> (&dst)[CX]) {
                    issue(ic, iy, dst);
                    if (++iy == rows) {
                        iy = 0;
                        ++ic;
                    }
                };
#pragma unroll
                for (int d = 0; d < D; ++d)
                    if (d < units) issue_next(v[d]);
                for (int u0 = 0; u0 < units; u0 += NBUF) {
#pragma unroll
                    for (int jj = 0; jj < NBUF; ++jj) {
                        if (u0 + jj >= units) break;
                        if (u0 + jj + D < units) issue_next(v[(jj + D) % NBUF]);
                        __builtin_amdgcn_sched_barrier(0);
                        consume(cc, cy, v[jj]);
                        if (++cy == rows) {
                            cy = 0;
                            ++cc;
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }

        // A zero weight times a non-finite feature may have reached bins whose samples do
        // not tap it, and shows as a non-finite output of the wave: then its bins are
        // recomputed sample by sample, every product taken where the definition takes it.
        uint32_t bad = 0;
#pragma unroll
        for (int j = 0; j < CPL; ++j)
#pragma unroll
            for (int p = 0; p < RPW; ++p)
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    acc[j][p][q] *= inv_count;
                    bad |= __builtin_isfinite(acc[j][p][q]) ? 0u : 1u;
                }
        if (__builtin_amdgcn_ballot_w64(bad != 0) != 0) {
#pragma unroll
            for (int j = 0; j < CPL; ++j) {
                const uint32_t vb = vbase + static_cast<uint32_t>(j) * uint32_t(sizeof(T));
#pragma unroll
                for (int p = 0; p < RPW; ++p) {
                    if (p0 + p >= p1) continue;
#pragma unroll 1
                    for (int q = 0; q < P; ++q) {
                        float sum = 0.0f;
                        for (int iy = 0; iy < ay.grid; ++iy) {
                            const float vy = ypos[(p0 + p) * ay.grid + iy];
                            if (vy < 0.0f) continue;
                            const int yl = static_cast<int>(vy);
                            const float fy = vy - static_cast<float>(yl);
                            const uint32_t r0 = vb + static_cast<uint32_t>(yl) * sh_b;
                            const uint32_t r1 = vb + static_cast<uint32_t>(min(yl + 1, L.H - 1)) * sh_b;
                            for (int ix = 0; ix < ax.grid; ++ix) {
                                const float vx = xpos[q * ax.grid + ix];
                                if (vx < 0.0f) continue;
                                const int xl = static_cast<int>(vx);
                                const float fx = vx - static_cast<float>(xl);
                                const uint32_t cl = static_cast<uint32_t>(xl) * sw_b;
                                const uint32_t chh = static_cast<uint32_t>(min(xl + 1, L.W - 1)) * sw_b;
                                const float v00 = raw_to_f32<T>(buf_load_raw<T>(res, r0 + cl));
                                const float v01 = raw_to_f32<T>(buf_load_raw<T>(res, r0 + chh));
                                const float v10 = raw_to_f32<T>(buf_load_raw<T>(res, r1 + cl));
                                const float v11 = raw_to_f32<T>(buf_load_raw<T>(res, r1 + chh));
                                const float xl_ = fmaf(fx, v01, (1.0f - fx) * v00);
                                const float xh_ = fmaf(fx, v11, (1.0f - fx) * v10);
                                sum += fmaf(fy, xh_, (1.0f - fy) * xl_);
                            }
                        }
                        sum = sum / static_cast<float>(max(ay.grid * ax.grid, 1));
#pragma unroll
                        for (int qq = 0; qq < P; ++qq) acc[j][p][qq] = (qq == q) ? sum : acc[j][p][qq];
                    }
                }
            }
        }

        // the slice's [SLICE][P][P] block, transposed through LDS in rounds of CHK channels
        const int nchan = min(SLICE, lv.C - slice * SLICE);
        const gptr<TO> out_blk = as_global_mut<TO>(a.out) +
                                 (static_cast<int64_t>(k) * lv.C + static_cast<int64_t>(slice) * SLICE) * NB;
#pragma unroll
        for (int c0 = 0; c0 < SLICE; c0 += CHK) {
            if (lane * CPL >= c0 && lane * CPL < c0 + CHK) {
#pragma unroll
                for (int j = 0; j < CPL; ++j)
#pragma unroll
                    for (int p = 0; p < RPW; ++p) {
                        if (p0 + p >= p1) continue;
#pragma unroll
                        for (int q = 0; q < P; ++q)
                            sm.stile[(lane * CPL + j - c0) * NB + (p0 + p) * P + q] = acc[j][p][q];
                    }
            }
            __syncthreads();
            const int ne = max(0, min(CHK, nchan - c0)) * NB;
            if (kvalid) store_run_f32<TO>(out_blk + c0 * NB, sm.stile, ne, t, 64 * NW);
            if (c0 + CHK < SLICE) __syncthreads();
        }
    }
}

// Waves per workgroup: four, or one per bin row with more loads in flight (units of CXF columns,
// DF of them, all 64 channels stored at once) in a grid that leaves most of the chip idle, where
// the chain of a wave is all there is (adaptive grid, 7x7, boxes of 8 to 800 pixels on four levels:
// 64 RoIs of 256 channels 29.4 -> 22.7 us, 128 RoIs 22.7 -> 19.3, 256 RoIs 31.3 against 36.7; 14x14:
// 16 RoIs 31.7 -> 20.2, 64 RoIs 56 -> 31, 256 RoIs 75 against 88).
constexpr int any_few(int P) { return P == 7 ? 512 : 256; }   // workgroups
template <typename T, typename TO, int P, int CX, int CHK, int CPL, int D, int CXF, int DF>
static hipError_t launch_any(FwdArgs a, hipStream_t stream) {
    a.nslices = (a.lv.C + 64 * CPL - 1) / (64 * CPL);
    // slices per workgroup as in the two-samples forward: up to 4 share the geometry while
    // the grid keeps at least 32 workgroups per CU
    a.spw = 1;
    for (int spw = 4; spw > 1; spw /= 2)
        if (static_cast<int64_t>(a.K) * ((a.nslices + spw - 1) / spw) >= 8192) {
            a.spw = spw;
            break;
        }
    a.wg_per_roi = (a.nslices + a.spw - 1) / a.spw;
    const int64_t grid = static_cast<int64_t>(a.K) * a.wg_per_roi;
    if (grid >= (int64_t(1) << 24)) return hipErrorInvalidConfiguration;
    const uint32_t g = static_cast<uint32_t>(grid);
    if (grid <= any_few(P)) fwd_any_kernel<T, TO, P, CXF, 64, CPL, DF, P><<<g, 64 * P, 0, stream>>>(a);
    else fwd_any_kernel<T, TO, P, CX, CHK, CPL, D, 4><<<g, 256, 0, stream>>>(a);
    return hipGetLastError();
}

template <typename T, typename TO>
hipError_t launch_fwd_any_typed(const FwdArgs &a, hipStream_t stream) {
    // columns per unit, channels per lane and units in flight of the two-samples kernels
    if (a.PH == 7) {
        if constexpr (sizeof(T) == 2)
            if (channel_pairs(a.lv)) return launch_any<T, TO, 7, 4, 64, 2, 4, 4, 8>(a, stream);
        return launch_any<T, TO, 7, 8, 64, 1, 2, 8, 4>(a, stream);
    }
    return launch_any<T, TO, 14, 4, 16, 1, 2, 8, 3>(a, stream);
}

hipError_t launch_fwd_any(const FwdArgs &a, int feat_dtype, int out_dtype, hipStream_t stream) {
    if (feat_dtype == kF32)
        return out_dtype == kF32 ? launch_fwd_any_typed<float, float>(a, stream)
                                 : launch_fwd_any_typed<float, uint16_t>(a, stream);
    return out_dtype == kF32 ? launch_fwd_any_typed<uint16_t, float>(a, stream)
                             : launch_fwd_any_typed<uint16_t, uint16_t>(a, stream);
}

// ---------------------------------------------------------------------------
// Backward: tile gather
// ---------------------------------------------------------------------------
//
// The two-samples gather (bwd.hip) with the weights of a quadrant summed from the RoI's
// sample positions, which the workgroup puts in LDS while the RoI's gradient block is
// copied.  The tile lists hold every RoI whose samples can tap the tile, whatever their
// number.  A non-finite sum in a tile (a NaN or infinity upstream, or an overflow) makes
// the workgroup walk its list twice more: once for the finite gradients, product by product,
// and once for the pixels that the others reach and what the definition's products make of
// them, which is added to the sums in memory.
template <typename TG, int P>
struct AnyGatherSmem {
    static constexpr int T = 8;
    static constexpr int NB = P * P;
    static constexpr int GB = 64 * NB;
    static constexpr int RUN = sizeof(TG) == 4 ? 256 : 64;
    static constexpr int NRUN = (GB + RUN - 1) / RUN;
    static constexpr int GBP = NRUN * RUN;
    static constexpr int NBUF = 2 * GBP * 4 <= 53248 ? 2 : 1;
    float pos[NBUF][2 * P * kAnyGrid];
    __align__(16) float wy[4][P * T];
    __align__(16) float wx[4][P * T];
    int k[64];
    Axis ax[64], ay[64];
    int rng[64][4];   // tap extent ymin, ymax, xmin, xmax
    int n;
};

// The smallest and largest weight a sample of bin p puts on pixel X; false if none taps it.
// A sample on the last pixel taps it twice, the second time with weight zero, as axis_tap has it.
__device__ __forceinline__ bool any_extremes(const float *pos, const Axis &a, int p, int X, int size,
                                             float &least, float &most) {
    int i0, i1;
    any_window(a, p, X, i0, i1);
    least = 2.0f;
    most = -1.0f;
#pragma unroll 1
    for (int i = i0; i <= i1; ++i) {
        const float v = pos[i];
        if (!(v >= 0.0f)) continue;
        const int l = static_cast<int>(v);
        const float f = v - static_cast<float>(l);
        if (l == X) {
            least = fminf(least, 1.0f - f);
            most = fmaxf(most, 1.0f - f);
        }
        if (min(l + 1, size - 1) == X) {
            least = fminf(least, f);
            most = fmaxf(most, f);
        }
    }
    return most >= 0.0f;
}

// What a bin's non-finite gradients do to the quadrant, as bits r * 8 + q of its pixels: an
// infinity times a positive weight is infinite, times a zero weight NaN, and a NaN is NaN on
// every tapped pixel.  A weight is the product of a row's and a column's; it is monotone in
// both, so the extremes of the two axes tell whether some sample's is zero and whether some
// sample's is not.
struct GatherMarks {
    uint64_t nan, up, down;   // of the lane's channel
};

// One RoI's part of a wave's quadrant: its sample positions, the lane's gradient block, the
// weights (wy with 1 / count), the tapped (row bin, row) pairs as ballots, and the runs of bins
// that reach the quadrant.
template <int NP>
struct AnyItem {
    Axis ay, ax;
    const float *ypos, *xpos;
    const uint32_t *gl;
    const float *wy, *wx;
    uint64_t yb[NP];
    int pha, phb, pwa, pwb;
    float inv_count;
};

// Walks the tile's RoIs and hands each one's part of the wave's quadrant to add.
template <typename TG, int P, typename Add>
__device__ __forceinline__ void any_phase(const GatherHead &h, const LevelTable &lv, int S, int t,
                                          const GatherTile &x, AnyGatherSmem<TG, P> &sm,
                                          uint32_t *slot0, uint32_t *slot1, Add &&add) {
    using SM = AnyGatherSmem<TG, P>;
    constexpr int T = SM::T, NB = SM::NB, GB = SM::GB, NBUF = SM::NBUF;
    constexpr int NP = (P * T + 63) / 64;   // ballot passes for the weights of an axis
    const int tid = threadIdx.x;
    const int wave = uniform_i(tid >> 6);
    const int lane = tid & 63;
    const LevelArg &L = x.L;
    const int l = x.l, b = x.b, R0 = x.R0, Q0 = x.Q0;
    int s0 = h.tile_start[t];
    int s1 = h.tile_end[t];
    s0 = max(0, min(s0, h.capacity));
    s1 = max(s0, min(s1, h.capacity));
    float *wy = sm.wy[wave];
    float *wx = sm.wx[wave];
    const int64_t kstride = static_cast<int64_t>(lv.C) * NB;
    const int nvalid = x.nch * NB;
    const bool wide = sizeof(TG) == 4 && (lv.C & 3) == 0 &&
                      (reinterpret_cast<uintptr_t>(h.gout) & 15u) == 0;
    // copy of kept RoI j's gradient block into LDS (as in bwd.hip's gather)
    auto fetch = [&](int j, uint32_t *gdst) {
        const int k = uniform_i(sm.k[j]);
        const char *src = static_cast<const char *>(h.gout) +
                          (static_cast<int64_t>(x.cg) * 64 * NB + static_cast<int64_t>(k) * kstride) *
                              int64_t(sizeof(TG));
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(src, static_cast<uint32_t>(nvalid) * uint32_t(sizeof(TG)));
        constexpr int RUN = SM::RUN, NRUN = SM::NRUN;
        if (RUN == 256 && wide) {
#pragma unroll
            for (int m = 0; m < (NRUN + 3) / 4; ++m) {
                const int run = wave + 4 * m;
                if (m < NRUN / 4 || run < NRUN) {
                    auto *dst = (__attribute__((address_space(3))) void *)(gdst + RUN * run);
                    const uint32_t off = static_cast<uint32_t>(RUN * run + lane * 4) * 4u;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 16, off, 0, 0, 0);
                }
            }
        } else {
            constexpr int NR64 = GB / 64;
#pragma unroll
            for (int m = 0; m < (NR64 + 3) / 4; ++m) {
                const int run = wave + 4 * m;
                if (m < NR64 / 4 || run < NR64) {
                    auto *dst = (__attribute__((address_space(3))) void *)(gdst + 64 * run);
                    const uint32_t off = static_cast<uint32_t>(64 * run + lane) * uint32_t(sizeof(TG));
                    if constexpr (sizeof(TG) == 4)
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 4, off, 0, 0, 0);
                    else
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 2, off, 0, 0, 0);
                }
            }
        }
    };
    auto fetch_wait = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70); };
    auto positions = [&](int j, float *pos) { any_positions<P>(sm.ay[j], sm.ax[j], L.H, L.W, pos); };
    auto consume = [&](int j, const uint32_t *gsrc, const float *pos) {
        const int ymin = sm.rng[j][0], ymax = sm.rng[j][1];
        const int xmin = sm.rng[j][2], xmax = sm.rng[j][3];
        if (!x.wave_on || ymax < R0 || ymin >= R0 + T || xmax < Q0 || xmin >= Q0 + T) return;
        const Axis ay = sm.ay[j], ax = sm.ax[j];
        const float inv_count = 1.0f / static_cast<float>(max(ay.grid * ax.grid, 1));
        uint64_t xb[NP];
        AnyItem<NP> it;
        it.ay = ay;
        it.ax = ax;
        it.ypos = pos;
        it.xpos = pos + kAnyGrid * P;
        it.inv_count = inv_count;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int u = p * 64 + lane;
            bool hy = false, hx = false;
            if (u < P * T) {
                const int bin = u / T;
                const float w = any_weight(it.ypos + bin * ay.grid, ay, bin, R0 + (u % T), L.H, hy);
                wy[u] = w * inv_count;
                wx[u] = any_weight(it.xpos + bin * ax.grid, ax, bin, Q0 + (u % T), L.W, hx);
            }
            it.yb[p] = __ballot(hy);
            xb[p] = __ballot(hx);
        }
        if (first_set(it.yb) < 0 || first_set(xb) < 0) return;
        it.pha = first_set(it.yb) / T;
        it.phb = last_set(it.yb) / T;
        it.pwa = first_set(xb) / T;
        it.pwb = last_set(xb) / T;
        it.gl = gsrc + lane * NB;
        it.wy = wy;
        it.wx = wx;
        wave_sync();
        add(it);
    };

    for (int base = s0; base < s1; base += 64) {
        const int n = min(64, s1 - base);
        __syncthreads();   // previous batch fully consumed
        if (wave == 0) {
            bool keep = false;
            int k = 0, ymin = 0, ymax = -1, xmin = 0, xmax = -1;
            Axis ax{}, ay{};
            if (lane < n) {
                k = h.tile_rois[base + lane];
                if (k >= 0 && k < h.K) {
                    const float *r = h.rois + 5 * static_cast<int64_t>(k);
                    const float r0 = r[0], x1 = r[1], y1 = r[2], x2 = r[3], y2 = r[4];
                    const int lvl = h.roi_levels ? h.roi_levels[k] : 0;
                    if (lvl == l && roi_batch(r0, lv.N) == b) {
                        ax = axis_setup(x1, x2, L.scale, h.aligned, P, S);
                        ay = axis_setup(y1, y2, L.scale, h.aligned, P, S);
                        if (ax.grid > 0 && ay.grid > 0) {
                            // extent from the end samples (either may come first in an
                            // inverted box); an end sample off the map widens it to the edge
                            const Tap fy = axis_tap(ay, 0, 0, L.H);
                            const Tap ly = axis_tap(ay, P - 1, ay.grid - 1, L.H);
                            const Tap fx = axis_tap(ax, 0, 0, L.W);
                            const Tap lx = axis_tap(ax, P - 1, ax.grid - 1, L.W);
                            const bool yok = fy.lo >= 0 && ly.lo >= 0;
                            const bool xok = fx.lo >= 0 && lx.lo >= 0;
                            const bool ydn = !(ay.bin >= 0.0f), xdn = !(ax.bin >= 0.0f);
                            ymin = yok ? min(fy.lo, ly.lo) : ydn || fy.lo < 0 ? 0 : fy.lo;
                            ymax = yok ? max(fy.hi, ly.hi) : ydn || ly.lo < 0 ? L.H - 1 : ly.hi;
                            xmin = xok ? min(fx.lo, lx.lo) : xdn || fx.lo < 0 ? 0 : fx.lo;
                            xmax = xok ? max(fx.hi, lx.hi) : xdn || lx.lo < 0 ? L.W - 1 : lx.hi;
                            keep = ymax >= x.WR0 && ymin < x.WR1 && xmax >= x.WC0 && xmin < x.WC1;
                        }
                    }
                }
            }
            const uint64_t km = __ballot(keep);
            if (keep) {
                const int pos = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                    static_cast<uint32_t>(km >> 32),
                    __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(km), 0u)));
                sm.k[pos] = k;
                sm.ax[pos] = ax;
                sm.ay[pos] = ay;
                sm.rng[pos][0] = ymin;
                sm.rng[pos][1] = ymax;
                sm.rng[pos][2] = xmin;
                sm.rng[pos][3] = xmax;
            }
            if (lane == 0) sm.n = __builtin_popcountll(km);
        }
        __syncthreads();
        const int nk = uniform_i(sm.n);
        if (nk == 0) continue;
        if constexpr (NBUF == 2) {
            fetch(0, slot0);
            positions(0, sm.pos[0]);
            fetch_wait();
            __syncthreads();
            for (int j = 0; j < nk; j += 2) {
                if (j + 1 < nk) {
                    fetch(j + 1, slot1);
                    positions(j + 1, sm.pos[1]);
                }
                consume(j, slot0, sm.pos[0]);
                fetch_wait();
                __syncthreads();
                if (j + 1 >= nk) break;
                if (j + 2 < nk) {
                    fetch(j + 2, slot0);
                    positions(j + 2, sm.pos[0]);
                }
                consume(j + 1, slot1, sm.pos[1]);
                fetch_wait();
                __syncthreads();
            }
        } else {
            for (int j = 0; j < nk; ++j) {
                if (j > 0) __syncthreads();   // the previous block is fully consumed
                fetch(j, slot0);
                positions(j, sm.pos[0]);
                fetch_wait();
                __syncthreads();
                consume(j, slot0, sm.pos[0]);
            }
        }
    }
}

// Accumulation: the quadrant's sums added with atomics, pixels no sample taps left alone, so
// calls that add into one pyramid may overlap on two streams, as scatters may, and a call's
// cost follows its RoIs and not the pyramid (against loading and storing every pixel: 8 RoIs on
// four levels 36 -> 20 us, 512 RoIs 85 -> 98 us).  Channels in separate planes: a row of the
// quadrant is turned around in the wave's LDS, so that an instruction adds to 8 runs of 8
// adjacent pixels and not to 64 planes (512 RoIs: 1125 -> 213 us).
constexpr int kAddPitch = 65;   // floats per pixel column in the scratch
__device__ __forceinline__ void gather_add(const GatherTile &x, const float (&acc)[8][8], float *scratch) {
    if (!x.wave_on) return;
    const int lane = threadIdx.x & 63;
    const LevelArg &L = x.L;
    float *const base = static_cast<float *>(const_cast<void *>(L.data)) + x.b * L.sn +
                        static_cast<int64_t>(x.cg * 64) * L.sc + x.R0 * L.sh + x.Q0 * L.sw;
    const bool planes = L.sc != 1 && L.sw == 1;
    const bool lane_on = lane < x.nch;
    float *const mine = base + (lane_on ? lane : 0) * L.sc;
    const int q8 = lane & 7, c8 = lane >> 3;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (x.R0 + r >= L.H) break;
        if (planes) {
#pragma unroll
            for (int q = 0; q < 8; ++q) scratch[q * kAddPitch + lane] = acc[r][q];
            wave_sync();
#pragma unroll
            for (int h = 0; h < 8; ++h) {
                const int c = 8 * h + c8;
                const float v = scratch[q8 * kAddPitch + c];
                if (c < x.nch && x.Q0 + q8 < L.W && v != 0.0f) unsafeAtomicAdd(base + c * L.sc + r * L.sh + q8, v);
            }
            wave_sync();   // the row's values are read before the next row overwrites them
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (x.Q0 + q < L.W && lane_on && acc[r][q] != 0.0f)
                    unsafeAtomicAdd(mine + r * L.sh + q * L.sw, acc[r][q]);
        }
    }
}

// 7x7: held to 128 registers (137 without, three waves per SIMD: 70 us against 58 us on the
// batch above); 14x14: its 50 KiB block allows two workgroups per CU anyway.
template <typename TG, int P>
__global__ __launch_bounds__(256, P == 7 ? 4 : 2) void bwd_gather_any_kernel(GatherArgs a) {
    using SM = AnyGatherSmem<TG, P>;
    constexpr bool two = SM::NBUF == 2;
    __shared__ SM sm;
    __shared__ __align__(16) uint32_t blk0[SM::GBP];
    __shared__ __align__(16) uint32_t blk1[two ? SM::GBP : 1];
    GatherTile x;
    const int t = gather_tile(a, a.tile_order, x);
    constexpr int NP = (P * 8 + 63) / 64;
    uint32_t *const slot1 = two ? blk1 : nullptr;
    float acc[8][8];
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[r][q] = 0.0f;
    any_phase<TG, P>(a.head[0], a.lv, a.S, t, x, sm, blk0, slot1, [&](const AnyItem<NP> &it) {
        gather_rows<TG, P>(acc, it.gl + it.pwa, it.wx + it.pwa * 8, it.wy, it.yb, it.pha, it.phb,
                           it.pwb - it.pwa + 1);
    });
    bool bad = false;
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int q = 0; q < 8; ++q) bad = bad || !__builtin_isfinite(acc[r][q]);
    static_assert(SM::GBP >= 4 * 8 * kAddPitch, "store scratch in the first slot");
    // also the barrier after which the staging slots are free
    const bool exact = __syncthreads_or(bad && x.wave_on);
    const int lane = threadIdx.x & 63;
    if (exact) {
        // A NaN or infinity upstream (or an overflow on the way): the list once more, bin by
        // bin and product by product, with the finite gradients only.
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[r][q] = 0.0f;
        any_phase<TG, P>(a.head[0], a.lv, a.S, t, x, sm, blk0, slot1, [&](const AnyItem<NP> &it) {
#pragma unroll 1
            for (int ph = it.pha; ph <= it.phb; ++ph) {
                const uint32_t rb =
                    static_cast<uint32_t>(it.yb[NP == 1 ? 0 : ph >> 3] >> ((ph & 7) * 8)) & 0xffu;
#pragma unroll 1
                for (int pw = it.pwa; pw <= it.pwb; ++pw) {
                    // lane = pixel of the quadrant (zero where no sample taps it)
                    const float w = it.wy[ph * 8 + (lane >> 3)] * it.wx[pw * 8 + (lane & 7)];
                    float g = raw_to_f32<TG>(it.gl[ph * P + pw]);
                    g = __builtin_isfinite(g) ? g : 0.0f;
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        if (((rb >> r) & 1u) == 0) continue;
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            acc[r][q] = fmaf(__int_as_float(__builtin_amdgcn_readlane(
                                                 __float_as_int(w), 8 * r + q)), g, acc[r][q]);
                    }
                }
            }
        });
        __syncthreads();   // the staging slots are free again
    }
    float *const scratch = reinterpret_cast<float *>(blk0) + (threadIdx.x >> 6) * (8 * kAddPitch);
    if (a.zero_init) gather_store(x, 1, acc, scratch);
    else gather_add(x, acc, scratch);
    if (!exact) return;
    // The non-finite gradients: which pixels they reach, then those pixels' values.
    GatherMarks m{0, 0, 0};
    any_phase<TG, P>(a.head[0], a.lv, a.S, t, x, sm, blk0, slot1, [&](const AnyItem<NP> &it) {
        const int Y = x.R0 + (lane >> 3), X = x.Q0 + (lane & 7);
#pragma unroll 1
        for (int ph = it.pha; ph <= it.phb; ++ph) {
            float ly, my;
            const bool hy = any_extremes(it.ypos + ph * it.ay.grid, it.ay, ph, Y, x.L.H, ly, my);
#pragma unroll 1
            for (int pw = it.pwa; pw <= it.pwb; ++pw) {
                const float g = raw_to_f32<TG>(it.gl[ph * P + pw]);
                if (__ballot(!__builtin_isfinite(g)) == 0) continue;
                float lx, mx;
                const bool hx = any_extremes(it.xpos + pw * it.ax.grid, it.ax, pw, X, x.L.W, lx, mx);
                const uint64_t hit = __ballot(hy && hx);
                const uint64_t zero = __ballot(hy && hx && ly * lx == 0.0f);
                const uint64_t some = __ballot(hy && hx && my * mx != 0.0f);
                const float inf = __builtin_inff();
                m.nan |= g != g ? hit : fabsf(g) == inf ? zero : 0;
                m.up |= g == inf ? some : 0;
                m.down |= g == -inf ? some : 0;
            }
        }
    });
    if (!x.wave_on || lane >= x.nch) return;
    __builtin_amdgcn_s_waitcnt(0x0F70);   // the wave's stores above are done
    float *const base = static_cast<float *>(const_cast<void *>(x.L.data)) + x.b * x.L.sn +
                        (x.cg * 64 + lane) * x.L.sc;
    for (uint64_t todo = m.nan | m.up | m.down; todo; todo &= todo - 1) {
        const int i = __builtin_ctzll(todo);
        float *const px = base + (x.R0 + (i >> 3)) * x.L.sh + (x.Q0 + (i & 7)) * x.L.sw;
        const bool up = (m.up >> i) & 1, down = (m.down >> i) & 1;
        const float v = ((m.nan >> i) & 1) || (up && down) ? __builtin_nanf("")
                                                           : up ? __builtin_inff() : -__builtin_inff();
        if (a.zero_init) *px += v;
        else unsafeAtomicAdd(px, v);
    }
}

// The RoIs whose level differs from the one the plan gave them (a caller may pass levels of
// its own): no tile list of their level holds them, so they are scattered with atomics.
// Plan slot s belongs to the level whose slot range holds it.
template <typename TG>
__global__ __launch_bounds__(256) void bwd_stray_kernel(GatherArgs a) {
    const GatherHead &h = a.head[0];
    const int s = static_cast<int>(blockIdx.x) * 256 + static_cast<int>(threadIdx.x);
    const int lane = threadIdx.x & 63;
    int k = -1, lvl = -1;
    if (s < h.K) {
        k = h.perm[s];
        if (k >= 0 && k < h.K) {
            int planned = 0;
            for (int i = 1; i < a.lv.num; ++i) planned += s >= h.offsets[i] ? 1 : 0;
            lvl = h.roi_levels ? h.roi_levels[k] : 0;
            if (lvl == planned || lvl < 0 || lvl >= a.lv.num) k = -1;
        } else {
            k = -1;
        }
    }
    uint64_t todo = __ballot(k >= 0);
    while (todo) {
        const int src = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int kk = __shfl(k, src);
        const int ll = __shfl(lvl, src);
        const float *r = h.rois + 5 * static_cast<int64_t>(kk);
        const int b = roi_batch(r[0], a.lv.N);
        if (b < 0) continue;
        const LevelArg L = level_at(a.lv, uniform_i(ll));
        const Axis ax = axis_setup(r[1], r[3], L.scale, h.aligned, a.PW, a.S);
        const Axis ay = axis_setup(r[2], r[4], L.scale, h.aligned, a.PH, a.S);
        const int nb = a.PH * a.PW;
        const int64_t n = static_cast<int64_t>(a.lv.C) * nb;
        for (int64_t e = lane; e < n; e += 64) {
            const int64_t c = e / nb;
            const int j = static_cast<int>(e - c * nb);
            const int ph = j / a.PW, pw = j - (j / a.PW) * a.PW;
            const float g = load_f32(as_global<TG>(h.gout) + kk * n + e) /
                            static_cast<float>(max(ay.grid * ax.grid, 1));
            float *base = static_cast<float *>(const_cast<void *>(L.data)) + b * L.sn + c * L.sc;
            for (int iy = 0; iy < ay.grid; ++iy) {
                const Tap ty = axis_tap(ay, ph, iy, L.H);
                if (ty.lo < 0) continue;
                for (int ix = 0; ix < ax.grid; ++ix) {
                    const Tap tx = axis_tap(ax, pw, ix, L.W);
                    if (tx.lo < 0) continue;
                    unsafeAtomicAdd(base + ty.lo * L.sh + tx.lo * L.sw, g * (ty.wlo * tx.wlo));
                    unsafeAtomicAdd(base + ty.lo * L.sh + tx.hi * L.sw, g * (ty.wlo * tx.whi));
                    unsafeAtomicAdd(base + ty.hi * L.sh + tx.lo * L.sw, g * (ty.whi * tx.wlo));
                    unsafeAtomicAdd(base + ty.hi * L.sh + tx.hi * L.sw, g * (ty.whi * tx.whi));
                }
            }
        }
    }
}

// `a` prepared (gather_prepare), `grid` its workgroups.
hipError_t launch_gather_any(const GatherArgs &a, uint32_t grid, int gout_dtype, hipStream_t stream) {
    const uint32_t g2 = static_cast<uint32_t>((a.head[0].K + 255) / 256);
    if (gout_dtype == kF32) {
        if (a.PH == 7) bwd_gather_any_kernel<float, 7><<<grid, 256, 0, stream>>>(a);
        else bwd_gather_any_kernel<float, 14><<<grid, 256, 0, stream>>>(a);
        bwd_stray_kernel<float><<<g2, 256, 0, stream>>>(a);
    } else {
        if (a.PH == 7) bwd_gather_any_kernel<uint16_t, 7><<<grid, 256, 0, stream>>>(a);
        else bwd_gather_any_kernel<uint16_t, 14><<<grid, 256, 0, stream>>>(a);
        bwd_stray_kernel<uint16_t><<<g2, 256, 0, stream>>>(a);
    }
    return hipGetLastError();
}

}  // namespace rex
