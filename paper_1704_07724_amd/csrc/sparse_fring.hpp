// Filter-ring kernel (declarations and, for the per-filter-size translation
// units that define ISC_FRING_INSTANTIATE, the kernel and its launchers).
//
// ISC steps 1-3 (Sec. "Sparse Convolution") in one launch for stride-1
// convolutions with square 1x1, 3x3 or 5x5 filters whose output is wider than
// 16 columns or whose filter does not fit in LDS (AlexNet conv2, an
// inception 3x3 branch): the input is compacted on the fly as in the
// register-weight kernel (sparse_fused.hpp), and the filter is streamed
// through LDS.
//
// The output of every image is cut into TH x TW tiles, numbered image by
// image, row band by row band, and each tile's input channels are dealt to
// `phases` wavefronts of one workgroup.  A wavefront holds 64*KPL output maps
// of its tile in registers and is on its own until the end: its LDS slot
// takes the next channel's R*S*64*KPL weights (from the K-contiguous repacked
// filter) and its window of that channel by direct global->LDS loads while
// it walks the current channel, whose weights and window it has read into
// registers; no barrier per channel, so a wavefront with many nonzeros
// delays nobody.  The walk is AsmWalk's: from nonzero to nonzero by computed
// jumps.  At the end the phases' tiles are summed through LDS in order and
// stored to NCHW (step 3) a few rows at a time, consecutive lanes on
// consecutive columns.
//
// Before, the four wavefronts of a workgroup shared each channel's stage of
// an LDS ring behind a barrier and scanned their windows statically, at two
// wavefronts per SIMD (100 weights and 108 accumulators): AlexNet conv2, 510
// us, spent most of them waiting for the slowest wavefront of each channel
// and for the weights' LDS reads.  One map per lane on a large tile reads a
// quarter of the weights per nonzero (9 x 9: 16 nonzeros a channel, 15 FMAs
// each) at four wavefronts per SIMD, and the workgroup's L1 serves the
// wavefronts' separate reads.  Kernel alone: AlexNet conv2 at batch 128 510 ->
// 243 us (43 TFLOP/s on nonzero MACs of 78.6), batch 1 163 -> 28; the
// inception 3x3 branch 204 -> 93, batch 1 114 -> 17; 64 -> 192 maps of 56 x 56,
// 3x3, batch 32 260 -> 102.
// Summation order per output is fixed (channels in
// order within a phase, window order within a channel, phases in order), so
// results are deterministic.
#pragma once

#include "sparse_tile.hpp"

namespace isc {
namespace fring {

using tile::kLanes;
// Range of the buffers a window is read through: past the offsets of every row
// it spans (at most 13 of 65535 columns); a position outside the map has
// tile::kPastPlane for an offset and reads zero.
constexpr int kWindowBytes = 1 << 30;

struct FringArgs {
    const float *x;   // N x C x H x W
    const float *wt;  // [C][R][S][Kp], K contiguous, zero past K
    float *y;         // N x K x Ho x Wo
    int N, C, H, W, K, Kp, P, Ho, Wo;
    int ctiles;       // column tiles per row band, ceil(Wo / TW)
    int rtiles;       // row bands per image, ceil(Ho / TH)
    int ntiles;       // N * rtiles * ctiles
    int kgroups;      // groups of 64 * KPL output maps
    int phases;       // wavefronts that share a tile's channels (1, 2 or 4)
    int T;            // stride, 1 or 2
    Decision dec;
    Epilogue epi;     // rectifier and census of y
};

// A register tile: KPL maps per lane, TH x TW outputs, so TH * TW * KPL
// accumulators and R*S*KPL weights per lane; NW wavefronts per workgroup.
struct TileChoice {
    int kpl, th, tw, nw;
};

// Wavefronts a SIMD holds of a tile's kernel: accumulators, weights and about
// 18 registers of window values, offsets and addresses, of 512.
constexpr int fring_waves_per_simd(int RS, int KPL, int TH, int TW) {
    const int regs = TH * TW * KPL + RS * RS * KPL + 18;
    return regs <= 64 ? 8 : (regs <= 80 ? 6 : (regs <= 96 ? 5 : (regs <= 128 ? 4 : (regs <= 170 ? 3 : 2))));
}

// The tiles compiled for each filter size, the choice's candidates.
constexpr TileChoice kTiles5[] = {{1, 9, 9, 4}, {1, 7, 14, 4}, {1, 5, 14, 4}, {1, 3, 14, 4}, {2, 1, 28, 4}};
constexpr TileChoice kTiles3[] = {{1, 7, 14, 4}, {1, 4, 14, 4}, {1, 2, 14, 4}, {2, 4, 14, 4}};
constexpr TileChoice kTiles1[] = {{1, 7, 14, 4}, {1, 4, 14, 4}, {1, 2, 14, 4}, {2, 4, 14, 4}};

// At stride 2 (where isc_conv2d's sparse path takes the kernel for shapes no
// other on-the-fly kernel does): a nonzero meets a quarter of the taps, so
// the tiles are small and their windows are not.
constexpr TileChoice kStrided[] = {{1, 4, 7, 4}, {2, 4, 7, 4}, {1, 2, 7, 4}};   // 3x3 and 5x5
constexpr TileChoice kStrided1[] = {{1, 4, 14, 4}, {2, 4, 14, 4}, {1, 2, 14, 4}};

// Launchers of the kernels of one filter size (sparse_fring_r{1,3,5}.hip).
hipError_t launch_r1(const FringArgs &a, const TileChoice &tc, hipStream_t s);
hipError_t launch_r3(const FringArgs &a, const TileChoice &tc, hipStream_t s);
hipError_t launch_r5(const FringArgs &a, const TileChoice &tc, hipStream_t s);

}  // namespace fring
}  // namespace isc

#ifdef ISC_FRING_INSTANTIATE
namespace isc {
namespace fring {
namespace {

template <int RS_, int KPL, int TH, int TW, int NW, int ST>
struct FringShape {
    using Walk = tile::AsmWalk<RS_, TH, TW, 0, KPL, ST>;
    static constexpr int RS2 = RS_ * RS_, KW = kLanes * KPL;
    static constexpr int CHF = RS2 * KW;           // floats of one channel's weights
    static constexpr int NDW = (CHF + 255) / 256;  // 1 KB direct-to-LDS blocks
    static constexpr int EPL = Walk::kChunks;
    // a wavefront's slot (floats): the channel's weights [R*S][KW] padded to
    // whole blocks, then its window, one word per lane and ballot; at the end
    // RC rows of its tile, [position][map] with a padded pitch
    static constexpr int PITCH = KW + 1;
    static constexpr int LOADF = NDW * 256 + EPL * kLanes;
    static constexpr int RFIT = LOADF / (TW * PITCH) < kLanes / TW ? LOADF / (TW * PITCH) : kLanes / TW;
    static constexpr int RC = RFIT < 1 ? 1 : (RFIT < TH ? RFIT : TH);
    static constexpr int SLOTF = ((LOADF > RC * TW * PITCH ? LOADF : RC * TW * PITCH) + 3) / 4 * 4;
    static constexpr size_t lds = sizeof(float) * SLOTF * NW;
};

template <int RS_, int KPL, int TH, int TW, int NW, int ST>
__global__ __launch_bounds__(NW * kLanes, fring_waves_per_simd(RS_, KPL, TH, TW))
void sparse_conv_fring_kernel(FringArgs a) {
    using SH = FringShape<RS_, KPL, TH, TW, NW, ST>;
    using Walk = typename SH::Walk;
    constexpr int RS2 = SH::RS2, KW = SH::KW, NDW = SH::NDW, EPL = SH::EPL, TP = TH * TW;
    constexpr int CH = tile::kWalkChunk, NQ = Walk::kPositions;
    __shared__ __align__(16) float slots[NW][SH::SLOTF];

    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const int kg = blockIdx.x % a.kgroups;
    const int phase = wave % a.phases;
    // this wavefront's tile (past the last one: nothing walked, nothing stored)
    const int tile = static_cast<int>(blockIdx.x / a.kgroups) * (NW / a.phases) + wave / a.phases;
    const bool has = tile < a.ntiles;
    int t = has ? tile : 0;
    const int ct = t % a.ctiles;
    t /= a.ctiles;
    const int band = t % a.rtiles;
    const int n = t / a.rtiles;
    const int oy0 = band * TH;
    const int ox0 = ct * TW;
    const int kbase = kg * KW;
    const int C = a.C, H = a.H, W = a.W, P = a.P;
    const size_t HW = static_cast<size_t>(H) * W;
    const int y0 = max(0, oy0 * ST - P);  // the window's first row in the map
    const float *x_n = a.x + static_cast<size_t>(n) * C * HW + static_cast<size_t>(y0) * W;
    const int ncw = has && phase < C ? (C - 1 - phase) / a.phases + 1 : 0;
    float *slot = slots[wave];

    // byte offset from row y0 (a plane may exceed 2^31 bytes) of position
    // q * CH + lane of the walk; lanes without one (padding, and lane CH of a
    // ballot, whose bit is the walk's sentinel) an offset past the buffer, which
    // reads as zero
    int xoff[EPL];
#pragma unroll
    for (int q = 0; q < EPL; ++q) {
        const int e = q * CH + lane;
        const int wy = e / Walk::kCols;
        const int y = oy0 * ST - P + wy * Walk::kStep, xx = ox0 * ST - P + (e - wy * Walk::kCols) * Walk::kStep;
        const bool in = lane < CH && e < NQ && y >= 0 && y < H && xx >= 0 && xx < W;
        xoff[q] = in ? ((y - y0) * W + xx) * static_cast<int>(sizeof(float)) : tile::kPastPlane;
    }
    // byte offset in a channel's weights of this lane's 16 bytes of block d
    // (blocks past the last tap repeat it)
    int woff[NDW];
#pragma unroll
    for (int d = 0; d < NDW; ++d) {
        const int f = d * 256 + lane * 4;
        const int tap = min(f / KW, RS2 - 1);
        woff[d] = (tap * a.Kp + min(kbase + f % KW, a.Kp - 4)) * static_cast<int>(sizeof(float));
    }
    const int chan_bytes = RS2 * a.Kp * static_cast<int>(sizeof(float));

    // channel i of this wavefront into its slot
    auto issue = [&](int i) {
        const int c = phase + i * a.phases;
        const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(a.wt) + static_cast<size_t>(c) * RS2 * a.Kp, 0, chan_bytes, tile::kBufferFormat);
#pragma unroll
        for (int d = 0; d < NDW; ++d) tile::buffer_lds16(wres, slot + d * 256, woff[d]);
        const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(x_n) + static_cast<size_t>(c) * HW, 0, kWindowBytes, tile::kBufferFormat);
#pragma unroll
        for (int q = 0; q < EPL; ++q) tile::buffer_lds4(xres, slot + NDW * 256 + q * kLanes, xoff[q]);
    };
    if (ncw > 0) issue(0);
    const bool run = decision_gate(a.dec, 1u);
    if (!run) {
        __builtin_amdgcn_s_waitcnt(0);  // no load into LDS may outlive the workgroup
        return;
    }

    float acc[TP * KPL];
#pragma unroll
    for (int p = 0; p < TP * KPL; ++p) acc[p] = 0.0f;

#pragma unroll 1
    for (int i = 0; i < ncw; ++i) {
        float cur[EPL], w[RS2 * KPL];
        tile::wait_vm<0, true>();  // this channel's loads into the slot have landed
        asm volatile("" ::: "memory");
#pragma unroll
        for (int q = 0; q < EPL; ++q) cur[q] = slot[NDW * 256 + q * kLanes + lane];
#pragma unroll
        for (int r = 0; r < RS2; ++r)
#pragma unroll
            for (int j = 0; j < KPL; ++j) w[r * KPL + j] = slot[r * KW + lane * KPL + j];
        // read into registers before the next channel's loads overwrite them
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + 1 < ncw) issue(i + 1);
        unsigned long long mask[EPL];
#pragma unroll
        for (int q = 0; q < EPL; ++q) {
            constexpr int kLast = NQ - (EPL - 1) * CH;  // positions of the last ballot
            mask[q] = __ballot((__float_as_uint(cur[q]) & 0x7fffffffu) != 0u) | (1ull << (q + 1 < EPL ? CH : kLast));
        }
        Walk::run(mask, cur, acc, w);
    }

    // step 3: RC rows at a time, every wavefront writes them to its slot as
    // [position][map] and the tile's wavefronts share the sums and stores:
    // consecutive lanes on consecutive positions of one map
    constexpr int RC = SH::RC, PITCH = SH::PITCH;
    const size_t plane_out = static_cast<size_t>(a.Ho) * a.Wo;
    const int cols = min(TW, a.Wo - ox0);
    const int kcnt = min(KW, a.K - kbase);
    const int w0 = wave - phase;  // the tile's first wavefront
    const int relu = a.epi.relu;
    uint32_t cnt = 0;
    tile::static_for<0, (TH + RC - 1) / RC>([&](auto pc) {
        constexpr int R0 = decltype(pc)::value * RC, R1 = R0 + RC < TH ? R0 + RC : TH;
        if (a.phases > 1) {
            if constexpr (R0 > 0) __syncthreads();  // the previous rows are read
        } else {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
#pragma unroll
        for (int p = R0 * TW; p < R1 * TW; ++p)
#pragma unroll
            for (int j = 0; j < KPL; ++j) slot[(p - R0 * TW) * PITCH + lane * KPL + j] = acc[p * KPL + j];
        if (a.phases > 1) __syncthreads();
        else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int rows = min(R1 - R0, a.Ho - oy0 - R0);
        if (!has || rows <= 0) return;
        // lane i of the tile's phases * 64: position i % npos of the rows,
        // every ostep-th map from i / npos
        const int npos = rows * cols;
        const int id = phase * kLanes + lane;
        const int ostep = a.phases * kLanes / npos;
        const int k0 = id / npos;
        const int pos = id - k0 * npos;
        const int oy = pos / cols, ox = pos - oy * cols;
        const float *src = slots[w0] + (oy * TW + ox) * PITCH;
        float *dst = a.y + (static_cast<size_t>(n) * a.K + kbase) * plane_out +
                     static_cast<size_t>(oy0 + R0 + oy) * a.Wo + ox0 + ox;
        for (int k = k0 < ostep ? k0 : kcnt; k < kcnt; k += ostep) {
            float sum = src[k];
            for (int p = 1; p < a.phases; ++p) sum += src[p * SH::SLOTF + k];
            sum = epilogue_value(sum, relu);
            cnt += nonzero_bit(sum);
            dst[static_cast<size_t>(k) * plane_out] = sum;
        }
    });
    if (a.epi.census) {
        __syncthreads();  // every wavefront is done with the slots
        census_commit(a.epi, cnt, reinterpret_cast<uint32_t *>(&slots[0][0]));
    }
}

template <int RS_, int KPL, int TH, int TW, int NW, int ST>
hipError_t launch_fring_t(const FringArgs &a, hipStream_t s) {
    using SH = FringShape<RS_, KPL, TH, TW, NW, ST>;
    static_assert(SH::lds <= 64 * 1024, "static LDS of a workgroup");
    const int64_t grid = static_cast<int64_t>((a.ntiles + NW / a.phases - 1) / (NW / a.phases)) * a.kgroups;
    if (a.epi.census && census_slots_for(grid) > a.epi.cap) return hipErrorInvalidValue;
    sparse_conv_fring_kernel<RS_, KPL, TH, TW, NW, ST><<<static_cast<unsigned>(grid), NW * kLanes, 0, s>>>(a);
    return hipGetLastError();
}

// The launcher of table entry I of TILES when it is the chosen tile, else
// the next entry's.
template <int RS_, int ST, const TileChoice *TILES, int I, int NT>
hipError_t launch_fring_table(const FringArgs &a, const TileChoice &tc, hipStream_t s) {
    if constexpr (I >= NT) {
        return hipErrorInvalidValue;
    } else {
        constexpr TileChoice t = TILES[I];
        if (tc.kpl == t.kpl && tc.th == t.th && tc.tw == t.tw && tc.nw == t.nw)
            return launch_fring_t<RS_, t.kpl, t.th, t.tw, t.nw, ST>(a, s);
        return launch_fring_table<RS_, ST, TILES, I + 1, NT>(a, tc, s);
    }
}

template <int RS_>
hipError_t launch_fring_rs(const FringArgs &a, const TileChoice &tc, hipStream_t s) {
    constexpr int n1 = sizeof(kTiles1) / sizeof(TileChoice), n3 = sizeof(kTiles3) / sizeof(TileChoice);
    constexpr int n5 = sizeof(kTiles5) / sizeof(TileChoice);
    constexpr int ns1 = sizeof(kStrided1) / sizeof(TileChoice), ns = sizeof(kStrided) / sizeof(TileChoice);
    if constexpr (RS_ == 5) {
        return a.T == 2 ? launch_fring_table<5, 2, kStrided, 0, ns>(a, tc, s)
                        : launch_fring_table<5, 1, kTiles5, 0, n5>(a, tc, s);
    } else if constexpr (RS_ == 3) {
        return a.T == 2 ? launch_fring_table<3, 2, kStrided, 0, ns>(a, tc, s)
                        : launch_fring_table<3, 1, kTiles3, 0, n3>(a, tc, s);
    } else {
        return a.T == 2 ? launch_fring_table<1, 2, kStrided1, 0, ns1>(a, tc, s)
                        : launch_fring_table<1, 1, kTiles1, 0, n1>(a, tc, s);
    }
}

}  // namespace
}  // namespace fring
}  // namespace isc
#endif
