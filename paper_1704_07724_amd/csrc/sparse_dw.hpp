// Weight-gradient kernel (declarations and, for the per-filter-size
// translation units that define ISC_DW_INSTANTIATE, the kernel and its
// launchers).
//
// Weight gradient with zero skipping, for training.  The paper measures the
// sparsity of rectified inputs during training (Sec. "Sparsity of ReLUs");
// the gradient of Eq. 1 with respect to the filter,
//   dw[k,c,r,s] = sum_{n,i,j} dy[n,k,i,j] * X^[n, c, i+r-P, j+s-P]   (stride 1),
// multiplies every input by output gradients, so a zero input contributes
// nothing and the work scales with the nonzeros as in ISC (Sec. "Sparse
// Convolution").  This is ISC step 2 with the roles of the filter and the
// output exchanged: a nonzero x at window row wy, shifted column xp meets the
// K-contiguous vector of output gradients dy[n, :, oy0 + wy - r, ox0 + xp - s]
// for every tap (r, s) whose output lies in the tile, and adds x times it to
// the K-contiguous gradient vector dw[:, c, r, s].
//
// A wavefront owns 64 output maps (lanes over maps, as in the forward
// kernels), CH input channels and a contiguous range of output tiles (TH x TW
// outputs of one image each), and keeps its CH*R*S gradient sums in registers
// for the whole range.  Per tile it holds the tile's output gradients of its
// maps in registers and walks, channel by channel, the nonzeros of the
// window that reaches the tile by computed jumps (AsmGradWalk, the forward
// walk with accumulators and operands exchanged).  The four wavefronts of a
// workgroup share maps and tile range and differ in channels: the tile's
// gradients come into LDS once, by direct global->LDS loads, a map's
// positions consecutive at an odd pitch, so that 64 lanes reading one position
// of their maps meet 64 banks.  Between two barriers a wavefront reads its
// gradients and windows into registers; the next tile's loads then land in
// the same LDS while this one is walked.  Sums are taken per tile and then
// added (shorter chains of rounding than one chain per range).  Each
// wavefront finally stores its sums for its range, maps fastest; a second launch adds the ranges in a fixed order and
// transposes (deterministic, no atomics).
//
// A position past the map's last row or column has gradient zero, so it adds
// nothing to a finite product; where an infinite or NaN input met one, the
// range's sum is not finite, and the second launch takes it again over the
// outputs alone.
//
// Before, one-row tiles under a static scan met 1.9 nonzeros per channel
// and tile with 2.2 FMAs each at 3x3; 7 x 13 tiles meet 4.9 with 7.2.
#pragma once

#include "sparse_tile.hpp"

namespace isc {
namespace dwk {

using tile::kLanes;
constexpr int kDwWaves = 4;
// Range of the buffers a tile is read through: past the offsets of every row
// a tile or its window spans (at most 13 of 65535 columns); a load outside the
// map has tile::kPastPlane for an offset and reads zero.
constexpr int kWindowBytes = 1 << 30;

struct DwArgs {
    const float *x;    // N x C x H x W
    const float *dy;   // N x K x Ho x Wo
    float *part;       // [splits][C*R*S][Kp]: sums of each tile range
    int N, C, H, W, K, P, Ho, Wo;
    int Kp;            // K rounded up to 64
    int ctiles;        // column tiles per row band
    int bands;         // groups of TH output rows
    int cgroups;       // groups of kDwWaves * CH channels
    int splits, per;   // tile ranges, tiles per range
    int ntiles;        // N * bands * ctiles
    int th, tw;        // outputs of a tile
};

// Tiles (TH x TW outputs; same: which window positions the walk visits, as in
// gen_dispatch.py) and the channels per wavefront: the tile's gradients and the
// sums leave three wavefronts per SIMD (168 registers), and a tile's
// gradients, read from LDS by every wavefront, serve as many channels as that
// allows.
struct DwTile {
    int th, tw, same, ch;
};
constexpr DwTile kDwTiles3[] = {{7, 7, 2, 4}, {7, 13, 1, 4}, {7, 14, 1, 3}, {7, 14, 0, 2}, {4, 16, 0, 4}, {2, 16, 0, 4}};
constexpr DwTile kDwTiles5[] = {{7, 7, 2, 2}, {9, 9, 0, 1}, {4, 14, 0, 2}, {2, 14, 0, 2}};
constexpr DwTile kDwTiles1[] = {{7, 7, 0, 8}, {7, 14, 0, 8}, {2, 14, 0, 8}};

struct DwPlan {
    DwTile t;
    int ctiles, bands, kgroups, cgroups, splits, per, ntiles;
};

// Launchers of the kernels of one filter size (sparse_dw_r{1,3,5}.hip).
hipError_t launch_r1(const DwArgs &a, const DwPlan &p, hipStream_t s);
hipError_t launch_r3(const DwArgs &a, const DwPlan &p, hipStream_t s);
hipError_t launch_r5(const DwArgs &a, const DwPlan &p, hipStream_t s);

}  // namespace dwk
}  // namespace isc

#ifdef ISC_DW_INSTANTIATE
namespace isc {
namespace dwk {
namespace {

template <int RS_, int TH, int TW, int SAME, int CH>
__global__ __launch_bounds__(kDwWaves * kLanes, 3)
void sparse_dw_kernel(DwArgs a) {
    using Walk = tile::AsmGradWalk<RS_, TH, TW, SAME>;
    constexpr int RS2 = RS_ * RS_, EPL = Walk::kChunks, NQ = Walk::kPositions;
    constexpr int WCH = tile::kWalkChunk, TP = TH * TW, PITCH = TP | 1;
    constexpr int NL = (TP + kLanes - 1) / kLanes;   // loads of one map's positions
    constexpr int MPW = kLanes / kDwWaves;           // maps each wavefront loads
    // a tile's gradients, [map][position], then the wavefronts' windows
    __shared__ float lds[kLanes * PITCH + kDwWaves * CH * EPL * kLanes];

    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    int b = blockIdx.x;
    const int cg = b % a.cgroups;
    b /= a.cgroups;
    const int split = b % a.splits;
    const int kg = b / a.splits;
    const int c0 = (cg * kDwWaves + wave) * CH;
    const int kbase = kg * kLanes;
    const int C = a.C, H = a.H, W = a.W, K = a.K, P = a.P, Ho = a.Ho, Wo = a.Wo;
    float *win = lds + kLanes * PITCH + wave * CH * EPL * kLanes;

    float acc[CH][RS2];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch)
#pragma unroll
        for (int t = 0; t < RS2; ++t) acc[ch][t] = 0.0f;

    const int t0 = split * a.per;
    const int t1 = min(a.ntiles, t0 + a.per);
    // the tile loaded next, counted on from t0: column tile, band, image
    int ct = t0 % a.ctiles, band = t0 / a.ctiles % a.bands, n = t0 / a.ctiles / a.bands;

    // the loads of one tile into LDS: its gradients (zero past the map; maps
    // past K repeat the last one, their sums are dropped) and this
    // wavefront's windows (position q * WCH + lane of the walk; lanes without
    // one read zero)
    auto load_tile = [&]() {
        const int oy0 = band * TH, ox0 = ct * TW;
        const int rows = Ho - oy0, cols = Wo - ox0;  // outputs from the tile's corner
        int goff[NL];
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int p = j * kLanes + lane;
            const int r = p / TW, c = p - r * TW;
            goff[j] = r < rows && c < cols ? (r * Wo + ox0 + c) * static_cast<int>(sizeof(float)) : tile::kPastPlane;
        }
        // offsets count from the tile's first row: a plane may exceed 2^31 bytes
        const float *gp = a.dy + (static_cast<size_t>(n) * K + kbase) * Ho * Wo + static_cast<size_t>(oy0) * Wo;
        const int mlast = K - 1 - kbase;
        gp += static_cast<size_t>(min(wave * MPW, mlast)) * (Ho * Wo);
#pragma unroll
        for (int i = 0; i < MPW; ++i) {
            const int m = wave * MPW + i;
            const __amdgpu_buffer_rsrc_t g =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(gp), 0, kWindowBytes, tile::kBufferFormat);
#pragma unroll
            for (int j = 0; j < NL; ++j)
                if (j * kLanes + lane < TP) tile::buffer_lds4(g, lds + m * PITCH + j * kLanes, goff[j]);
            gp += m < mlast ? Ho * Wo : 0;
        }
        const int y0 = max(0, oy0 - P);
        int xoff[EPL];
#pragma unroll
        for (int q = 0; q < EPL; ++q) {
            const int e = q * WCH + lane;
            const int wy = e / Walk::kCols + Walk::kRow0, xp = e % Walk::kCols + Walk::kCol0;
            const int y = oy0 - P + wy, xx = ox0 - P + xp;
            const bool in = lane < WCH && e < NQ && wy < rows + RS_ - 1 && xp < cols + RS_ - 1 && y >= 0 && y < H &&
                            xx >= 0 && xx < W;
            xoff[q] = in ? ((y - y0) * W + xx) * static_cast<int>(sizeof(float)) : tile::kPastPlane;
        }
        const float *xp = a.x + (static_cast<size_t>(n) * C + min(c0, C - 1)) * H * W + static_cast<size_t>(y0) * W;
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            const __amdgpu_buffer_rsrc_t x =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(xp), 0, kWindowBytes, tile::kBufferFormat);
#pragma unroll
            for (int q = 0; q < EPL; ++q) tile::buffer_lds4(x, win + (ch * EPL + q) * kLanes, xoff[q]);
            xp += c0 + ch + 1 < C ? H * W : 0;
        }
        if (++ct == a.ctiles) {
            ct = 0;
            if (++band == a.bands) {
                band = 0;
                ++n;
            }
        }
    };

    if (t0 < t1) load_tile();
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
        tile::wait_vm_and_barrier<0>();  // everyone's loads of this tile have landed
        float cur[CH][EPL], g[TP];
#pragma unroll
        for (int p = 0; p < TP; ++p) g[p] = lds[lane * PITCH + p];
#pragma unroll
        for (int ch = 0; ch < CH; ++ch)
#pragma unroll
            for (int q = 0; q < EPL; ++q) cur[ch][q] = win[(ch * EPL + q) * kLanes + lane];
        tile::wait_vm_and_barrier<0>();  // and been read
        if (t + 1 < t1) load_tile();
        tile::static_for<0, CH>([&](auto chc) {
            constexpr int ch = decltype(chc)::value;
            unsigned long long mask[EPL];
#pragma unroll
            for (int q = 0; q < EPL; ++q) {
                constexpr int kLast = NQ - (EPL - 1) * WCH;  // positions of the last ballot
                mask[q] = __ballot((__float_as_uint(cur[ch][q]) & 0x7fffffffu) != 0u) |
                          (1ull << (q + 1 < EPL ? WCH : kLast));
            }
            float sum[RS2];
#pragma unroll
            for (int i = 0; i < RS2; ++i) sum[i] = 0.0f;
            Walk::run(mask, cur[ch], g, sum);
#pragma unroll
            for (int i = 0; i < RS2; ++i) acc[ch][i] += sum[i];
        });
    }

    // this range's sums
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
        if (c0 + ch >= C) break;
        float *dst = a.part + (static_cast<size_t>(split) * C + c0 + ch) * RS2 * a.Kp + kbase + lane;
#pragma unroll
        for (int t = 0; t < RS2; ++t) dst[static_cast<size_t>(t) * a.Kp] = acc[ch][t];
    }
}

// The launcher of table entry I when it is the chosen tile, else the next's.
template <int RS_, const DwTile *TILES, int I, int NT>
hipError_t launch_dw_table(const DwArgs &a, const DwPlan &p, hipStream_t s) {
    if constexpr (I >= NT) {
        return hipErrorInvalidValue;
    } else {
        constexpr DwTile t = TILES[I];
        if (p.t.th != t.th || p.t.tw != t.tw || p.t.same != t.same) return launch_dw_table<RS_, TILES, I + 1, NT>(a, p, s);
        const int64_t grid = static_cast<int64_t>(p.kgroups) * a.splits * a.cgroups;
        sparse_dw_kernel<RS_, t.th, t.tw, t.same, t.ch><<<static_cast<unsigned>(grid), kDwWaves * kLanes, 0, s>>>(a);
        return hipGetLastError();
    }
}

}  // namespace
}  // namespace dwk
}  // namespace isc
#endif
