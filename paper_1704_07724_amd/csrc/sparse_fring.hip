// Filter-ring kernel (sparse_fring.hpp): the choice of tile and the launch.
#include "sparse_fring.hpp"

#include <algorithm>
#include <cstring>

namespace isc {
namespace fring {
namespace {

// The compiled tiles of a filter size and stride.
template <int N>
int tiles_of(const TileChoice (&table)[N], const TileChoice **t) {
    *t = table;
    return N;
}
int tiles_for(int R, int T, const TileChoice **t) {
    if (T == 2) return R == 1 ? tiles_of(kStrided1, t) : tiles_of(kStrided, t);
    return R == 5 ? tiles_of(kTiles5, t) : (R == 3 ? tiles_of(kTiles3, t) : tiles_of(kTiles1, t));
}

// Modelled cycles of the kernel on a tile with its channels over `phases`
// wavefronts, at an input density: the larger of two lines.  A CU's w
// workgroups put a wavefront on each SIMD.  They are bound by issue (per
// wavefront and channel 33 cycles, 50 a ballot, 3.5 a weight; per nonzero its
// FMAs at 4 cycles and 4 more, at least its scalar chain's 28) or by one
// wavefront's chain of jumps (96 cycles a nonzero beside its FMAs), and
// part of a workgroup's duration passes at the end with CUs running dry, which
// is what more phases, hence more and shorter workgroups, are for (AlexNet
// conv2 on 9 x 9 tiles: 286 / 250 / 243 us on 1 / 2 / 4 phases, the inception
// 3x3 branch at batch 1 on 2 x 14: 48 / 28 / 17).  Fitted to the kernel timed on
// 43 shapes at sparsities 0.3 to 0.95: 8 % rms, 21 % at most.
struct RingCost {
    double issue0, issue1, chain0, chain1;  // issue0 + issue1 * density, chain0 + chain1 * density
    double at(double d) const { return std::max(issue0 + issue1 * d, chain0 + chain1 * d); }
};

RingCost ring_cost(const SparseShape &sh, const TileChoice &t, int phases) {
    const int64_t bands = (sh.Ho + t.th - 1) / t.th, ctiles = (sh.Wo + t.tw - 1) / t.tw;
    const int64_t kw = static_cast<int64_t>(kLanes) * t.kpl;
    const int64_t per = t.nw / phases;
    const int64_t wgs = (sh.N * bands * ctiles + per - 1) / per * ((sh.K + kw - 1) / kw);
    const double w = std::max(1.0, static_cast<double>(wgs) / 256.0);
    const int occ = fring_waves_per_simd(sh.R, t.kpl, t.th, t.tw);
    const double resident = std::min<double>(occ, std::ceil(w));
    // input rows and columns a tile's window holds on average: all but the
    // padding and what the last tile reaches past the map
    const int wr = (t.th - 1) * sh.T + sh.R, wc = (t.tw - 1) * sh.T + sh.R;  // the window's extent
    const int64_t inr = bands * wr - sh.P - ((bands * t.th - sh.Ho) * sh.T + sh.P);
    const int64_t inc = ctiles * wc - sh.P - ((ctiles * t.tw - sh.Wo) * sh.T + sh.P);
    const double rows = std::min<double>(sh.H, std::max(1.0, static_cast<double>(inr) / bands));
    const double cols = std::min<double>(sh.W, std::max(1.0, static_cast<double>(inc) / ctiles));
    const double seen = sh.R < sh.T ? 1.0 / (sh.T * sh.T) : 1.0;  // share of the window's positions visited
    const double fmas = t.kpl * taps_inside(sh.P, sh.R, sh.Ho) * taps_inside(sh.P, sh.R, sh.Wo) *
                        static_cast<double>(std::min(t.th, sh.Ho)) * std::min(t.tw, sh.Wo) * sh.R * sh.R /
                        (rows * cols * seen);
    const int chunks = static_cast<int>((wr * wc * seen + tile::kWalkChunk - 1) / tile::kWalkChunk);
    const double chan = (sh.C + phases - 1) / phases;
    const double i0 = 33.0 + 50.0 * chunks + 3.5 * sh.R * sh.R * t.kpl;
    const double i1 = rows * cols * seen * std::max(28.0, 4.1 + 4.0 * fmas);
    const double c0 = 382.0 + 50.0 * chunks, c1 = rows * cols * seen * (96.0 + 4.0 * fmas);
    const double fixed = 15720.0 + 106.0 * w * t.th * t.tw * t.kpl;
    const double iw = chan * (w + (w > 1.0 ? 0.76 * resident : 0.0)), cw = chan * std::max(1.0, w / occ);
    return {iw * i0 + fixed, iw * i1, cw * c0 + fixed, cw * c1};
}

constexpr double kPlanDensity = 0.1;  // the paper's layers are 0.9 to 0.95 sparse

// The cheapest compiled tile and number of phases, restricted to a caller's
// maps_per_lane / rows / cols / waves when those name a compiled tile, and
// to a caller's phases (1, 2 or 4; 1 where only the tile is named).
bool choose(const SparseShape &sh, TileChoice *tc, int *phases) {
    if (!(sh.T == 1 || sh.T == 2) || sh.R != sh.S || !(sh.R == 1 || sh.R == 3 || sh.R == 5)) return false;
    // the kernel addresses a channel's weights by 31-bit byte offsets
    const int64_t kp = (sh.K + kLanes - 1) / kLanes * static_cast<int64_t>(kLanes);
    if (kp * sh.R * sh.S * 4 >= (1ll << 31)) return false;
    const TileChoice *tiles;
    const int n = tiles_for(sh.R, sh.T, &tiles);
    for (int pass = 0; pass < 2; ++pass) {
        const bool forced = pass == 0;
        if (forced && sh.tu.maps_per_lane <= 0 && sh.tu.rows <= 0 && sh.tu.cols <= 0 && sh.tu.waves <= 0) continue;
        const bool named = sh.tu.phases == 1 || sh.tu.phases == 2 || sh.tu.phases == 4;
        const int fix = named ? sh.tu.phases : (forced ? 1 : 0);
        bool found = false;
        double best = 0.0;
        for (int i = 0; i < n; ++i) {
            const TileChoice &t = tiles[i];
            if (forced && ((sh.tu.maps_per_lane > 0 && t.kpl != sh.tu.maps_per_lane) ||
                           (sh.tu.rows > 0 && t.th != sh.tu.rows) || (sh.tu.cols > 0 && t.tw != sh.tu.cols) ||
                           (sh.tu.waves > 0 && t.nw != sh.tu.waves)))
                continue;
            for (int ph : {1, 2, 4}) {
                if (fix > 0 && fix != ph) continue;
                const double c = ring_cost(sh, t, ph).at(kPlanDensity);
                if (!found || c < best) {
                    *tc = t;
                    *phases = ph;
                    best = c;
                    found = true;
                }
            }
        }
        if (found) return true;
    }
    return false;
}

// The choice of a shape, asked for several times in the course of one call:
// the calling thread's last answer is kept beside the shape and the
// overrides it was computed from.
bool fring_choose(const SparseShape &sh, TileChoice *tc, int *phases) {
    struct Last {
        SparseShape sh;
        TileChoice tc;
        int phases;
        int ok = -1;
    };
    static thread_local Last last;
    if (last.ok < 0 || std::memcmp(&last.sh, &sh, sizeof sh) != 0) {
        last.ok = choose(sh, &last.tc, &last.phases);
        last.sh = sh;
    }
    if (last.ok) {
        *tc = last.tc;
        *phases = last.phases;
    }
    return last.ok != 0;
}

int64_t ring_groups(const SparseShape &sh, const TileChoice &t, int phases) {
    const int64_t ntiles = static_cast<int64_t>(sh.N) * ((sh.Ho + t.th - 1) / t.th) * ((sh.Wo + t.tw - 1) / t.tw);
    const int per = t.nw / phases;
    return (ntiles + per - 1) / per * ((sh.K + kLanes * t.kpl - 1) / (kLanes * t.kpl));
}

}  // namespace
}  // namespace fring

bool sparse_fring_applies(const SparseShape &sh) {
    fring::TileChoice tc;
    int phases;
    return sh.T == 1 && fring::fring_choose(sh, &tc, &phases);
}

bool sparse_strided_applies(const SparseShape &sh) {
    fring::TileChoice tc;
    int phases;
    return sh.T == 2 && (sh.tu.kernel == 0 || sh.tu.kernel == ISC_KERNEL_FUSED_RING) &&
           list_kernel_for(sh) == kListGeneric && fring::fring_choose(sh, &tc, &phases);
}

int64_t sparse_fring_max_groups(const SparseShape &sh) {
    using namespace fring;
    const TileChoice *tiles;
    const int n = tiles_for(sh.R, sh.T, &tiles);
    int64_t most = 0;
    for (int i = 0; i < n; ++i) most = std::max(most, ring_groups(sh, tiles[i], 4));
    return most;
}

bool sparse_ring_time_model(const SparseShape &sh, KernelTime *t) {
    using namespace fring;
    TileChoice tc;
    int phases;
    if (!fring_choose(sh, &tc, &phases)) return false;
    const RingCost c = ring_cost(sh, tc, phases);
    constexpr double kMs = 1.0 / 2.4e6;  // a cycle at 2.4 GHz
    *t = KernelTime{{c.issue0 * kMs, c.chain0 * kMs}, {c.issue1 * kMs, c.chain1 * kMs}};
    return true;
}

bool sparse_fring_plan_info(const SparseShape &sh, isc_plan *out) {
    using namespace fring;
    TileChoice tc;
    int phases;
    if (!fring_choose(sh, &tc, &phases)) return false;
    *out = isc_plan{ISC_KERNEL_FUSED_RING, tc.th, tc.tw, tc.kpl, phases, tc.nw, ring_groups(sh, tc, phases)};
    return true;
}

hipError_t launch_sparse_fring(const SparseShape &sh, const float *x, const float *wt, float *y, const Decision &dec,
                               hipStream_t s, const Epilogue &epi) {
    using namespace fring;
    TileChoice tc;
    int phases;
    if (!fring_choose(sh, &tc, &phases)) return hipErrorInvalidValue;
    FringArgs a{};
    a.x = x;
    a.wt = wt;
    a.y = y;
    a.N = sh.N; a.C = sh.C; a.H = sh.H; a.W = sh.W; a.K = sh.K;
    a.Kp = (sh.K + kLanes - 1) / kLanes * kLanes;
    a.P = sh.P; a.Ho = sh.Ho; a.Wo = sh.Wo;
    a.ctiles = (sh.Wo + tc.tw - 1) / tc.tw;
    a.rtiles = (sh.Ho + tc.th - 1) / tc.th;
    const int64_t ntiles = static_cast<int64_t>(sh.N) * a.rtiles * a.ctiles;
    if (ntiles >= (1ll << 31) - tc.nw) return hipErrorInvalidValue;
    a.ntiles = static_cast<int>(ntiles);
    a.kgroups = (sh.K + kLanes * tc.kpl - 1) / (kLanes * tc.kpl);
    a.phases = phases;
    a.T = sh.T;
    a.dec = dec;
    a.epi = epi;
    switch (sh.R) {
    case 1: return launch_r1(a, tc, s);
    case 3: return launch_r3(a, tc, s);
    default: return launch_r5(a, tc, s);
    }
}

}  // namespace isc
