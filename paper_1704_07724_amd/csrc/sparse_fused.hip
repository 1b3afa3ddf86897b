// Filter-resident kernel (sparse_fused.hpp): the plan, the launch, and the
// choice between it and the filter-ring kernel.
#include "sparse_fused.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace isc {
namespace fused {
namespace {

int fused_tw(int Wo) { return Wo <= 8 ? 8 : (Wo <= 16 ? 16 : 28); }

// Whether the register-weight kernel is compiled for the tile.
template <int R>
bool reg_tile_compiled_r(RegTile t) {
    bool ok = false;
    tile::static_for<0, kRegTiles>([&](auto ic) {
        constexpr RegTile c = kRegTile[decltype(ic)::value];
        if (c.th == t.th && c.tw == t.tw && c.same == t.same) ok = tile::AsmWalk<R, c.th, c.tw, c.same>::kReg;
    });
    return ok;
}
bool reg_tile_compiled(int R, RegTile t) {
    return R == 1 ? reg_tile_compiled_r<1>(t) : (R == 3 ? reg_tile_compiled_r<3>(t) : reg_tile_compiled_r<5>(t));
}

// Whether the register-weight kernel may run the shape on the tile: one
// column tile holds the output, and the positions its walk leaves out are
// padding.
bool reg_tile_takes(const SparseShape &sh, RegTile t) {
    if (sh.Wo > t.tw || !reg_tile_compiled(sh.R, t)) return false;
    if (t.same >= 1 && (sh.P != sh.R / 2 || sh.W > t.tw)) return false;
    return t.same < 2 || sh.H <= t.th;
}

// Modelled cycles of the register-weight kernel on a tile at an input
// density, which choose the tile and stand for the kernel in AUTO's crossover.
// The CU with most workgroups (w of them, two wavefronts per SIMD each, `occ`
// resident) is bound either by issue (per wavefront and channel 90 cycles and
// 9.2 a weight, per nonzero its FMAs at 4 cycles and 5 more, at least its
// scalar chain's 28) or, with few wavefronts, by the latency of one
// wavefront's jumps (73 cycles a nonzero beside its FMAs).  Each round also
// pays its reduction, each launch its start.  Fitted to the kernel timed on 51
// shapes (this repository's layers and log-uniform sizes) at sparsities 0.3 to
// 0.95: 11 % rms, 33 % at most.
constexpr double kPlanDensity = 0.1;  // the paper's layers are 0.9 to 0.95 sparse

struct RegCost {
    // cycles at density d: max(issue0 + issue1 * d, chain0 + chain1 * d)
    double issue0, issue1, chain0, chain1;
    double at(double d) const { return std::max(issue0 + issue1 * d, chain0 + chain1 * d); }
};

RegCost reg_cost(const SparseShape &sh, RegTile t) {
    const int64_t bands = (sh.Ho + t.th - 1) / t.th;
    // the tile's registers: accumulators, two sets of weights, addresses
    const int vgprs = t.th * t.tw + 2 * sh.R * sh.R + 14;
    const int occ = vgprs <= 64 ? 4 : (vgprs <= 80 ? 3 : 2);
    const int64_t wgs = sh.N * bands * ((sh.K + kLanes - 1) / kLanes);
    const int64_t w = (wgs + 255) / 256;
    const double rounds = static_cast<double>((w + occ - 1) / occ);
    const double cols = std::min(t.tw + sh.R - 1, sh.W);
    // input rows a band's window holds on average: all but the padding above
    // the first band and what the last one reaches past the map
    const int64_t in = bands * (t.th + sh.R - 1) - sh.P - (bands * t.th - sh.Ho + sh.P);
    const double rows = std::min<double>(sh.H, std::max(1.0, static_cast<double>(in) / bands));
    const double fmas = taps_inside(sh.P, sh.R, sh.Ho) * taps_inside(sh.P, sh.R, sh.Wo) *
                        static_cast<double>(std::min(t.th, sh.Ho)) * t.tw * sh.R * sh.R / (rows * cols);
    const double chan = (sh.C + kWaves - 1) / kWaves;
    const double fixed = 15840.0 + 48.6 * rounds * t.th * t.tw + 32.0 * w * t.th * t.tw;
    return {fixed + 2.0 * w * chan * (90.0 + 9.2 * sh.R * sh.R),
            2.0 * w * chan * rows * cols * std::max(28.0, 5.3 + 4.0 * fmas), fixed + rounds * chan * 95.0,
            rounds * chan * rows * cols * (73.0 + 4.0 * fmas)};
}

size_t fused_lds(int crs, int th, int tw) {
    return std::max(sizeof(float) * crs * kWPitch, sizeof(float) * kWaves * th * tw * kRPad);
}

// Plans whose wavefronts share no channel (every wavefront its own phase)
// gain nothing from the filter in LDS: with the weights streamed to
// registers, LDS holds only the reduction's tiles (LeNet conv2: 13.2 -> 9.5
// us).  The filter need not fit in LDS at all, and one workgroup per group of
// 64 maps takes any K (AlexNet-ImageNet conv4 of Tab. 2 at batch 128: 259 us
// on the filter-ring kernel, 43 here).  Taken wherever eligible: stride 1,
// square 1x1, 3x3 and 5x5 filters, at most 16 output columns; the tile is the
// cheapest by reg_cost's model (tall ones on full grids, short ones where a
// small batch leaves CUs idle: inception 4e.3 at batch 1 takes 10.9 us on 1 x
// 16 and 22.2 on 7 x 14, at batch 128 182 and 69).  A caller's tuning kernel
// FUSED or FUSED_RING keeps the filter in LDS, or in the ring beyond 64 maps;
// rows and cols name a tile.
bool fused_wreg_plan(const SparseShape &sh, FusedPlan *plan) {
    if (sh.tu.kernel == ISC_KERNEL_FUSED || sh.tu.kernel == ISC_KERNEL_FUSED_RING) return false;
    if (sh.T != 1 || sh.Wo > 16) return false;
    // the kernel addresses the repacked filter with 32-bit byte offsets
    const int64_t kp = (sh.K + kLanes - 1) / kLanes * kLanes;
    if (static_cast<int64_t>(sh.C) * sh.R * sh.S * kp * static_cast<int64_t>(sizeof(float)) >= (1ll << 31))
        return false;
    RegTile best{0, 0, 0};
    double best_c = 0.0;
    for (const RegTile &t : kRegTile) {
        if (!reg_tile_takes(sh, t)) continue;
        if (t.th == sh.tu.rows && (sh.tu.cols == 0 || sh.tu.cols == t.tw)) {
            best = t;
            break;
        }
        const double c = reg_cost(sh, t).at(kPlanDensity);
        if (best.th == 0 || c < best_c) {
            best = t;
            best_c = c;
        }
    }
    *plan = FusedPlan{best.th, best.tw, kWaves,
                      sizeof(float) * kRegSlots * reg_chunk_rows(best.th, best.tw) * best.tw * kRPad, 1, true, best.same};
    return true;
}

// The filter must fit in LDS; stride 1, or stride 2 with 3x3 or 5x5 filters
// and at most 8 output columns.  Tile height and channel phases: the tallest
// tile (up to kMaxTile accumulators per lane), then the fewest phases that
// leave no row group of a workgroup idle (rg <= ceil(Ho / TH)), preferring
// plans with at least kMinGroups workgroups; else the plan with most
// workgroups.  A caller's tuning rows caps the tile height and phases fixes
// the phases; tuning kernel FUSED_RING leaves the shape to the filter-ring
// kernel.
bool make_fused_plan(const SparseShape &sh, FusedPlan *plan) {
    if (sh.tu.kernel == ISC_KERNEL_FUSED_RING && sparse_fring_applies(sh)) return false;
    if (sh.R != sh.S || !(sh.R == 1 || sh.R == 3 || sh.R == 5)) return false;
    if (!(sh.T == 1 || (sh.T == 2 && sh.R > 1 && sh.Wo <= 8))) return false;
    if (sh.Wo > 28) return false;
    // beyond 64 maps only the register-weight kernel (one wavefront per 64
    // maps and channel phase), where it takes the shape and the caller does
    // not ask for the filter-ring kernel: at 13 x 13 and sparsity 0.95
    // (AlexNet conv3-5) it beat every tile of the filter-ring kernel by
    // 12-30 %, the ring's tiles of up to 384 maps leaving CUs idle or
    // waiting on each channel's stage
    if (sh.K > kLanes) return fused_wreg_plan(sh, plan);
    const int crs = sh.C * sh.R * sh.S;
    // a filter too large for LDS: only the register-weight kernel, which
    // keeps none of it there, takes it (one phase per wavefront)
    if (static_cast<size_t>(crs) * kWPitch * sizeof(float) > kLdsMax) return fused_wreg_plan(sh, plan);
    const int tw = fused_tw(sh.Wo);
    const int th_cap = sh.tu.rows > 0 ? sh.tu.rows : 8;
    const int cs_fix = sh.tu.phases == 1 || sh.tu.phases == 2 || sh.tu.phases == 4 || sh.tu.phases == 8 ? sh.tu.phases : 0;
    bool found = false, done = false;
    int64_t best_groups = 0;
    for (int th : {8, 4, 2, 1}) {
        if (th * tw > kMaxTile || th > th_cap) continue;
        const int rows_need = (sh.Ho + th - 1) / th;
        for (int cs : {1, 2, 4, 8}) {
            if (cs_fix > 0 && cs != cs_fix) continue;
            const int rg = kWaves / cs;
            if (cs_fix == 0 && rg > rows_need && cs < kWaves) continue;  // idle row groups
            const int64_t groups = static_cast<int64_t>(sh.N) * ((sh.Ho + rg * th - 1) / (rg * th));
            const size_t lds = fused_lds(crs, th, tw);
            if (lds > kLdsMax) continue;
            if (!found || groups > best_groups) {
                *plan = FusedPlan{th, tw, cs, lds, sh.T, false, 0};
                best_groups = groups;
                found = true;
            }
            done = groups >= kMinGroups;
            break;  // more phases only add partial tiles
        }
        if (done) break;
    }
    if (found && plan->cs == kWaves) fused_wreg_plan(sh, plan);
    return found;
}

// The plan of a shape, asked for several times in the course of one call
// (workspace layout, crossover, launch): the calling thread's last answer is
// kept beside the shape and the overrides it was computed from.
bool fused_plan(const SparseShape &sh, FusedPlan *plan) {
    struct Last {
        SparseShape sh;
        FusedPlan plan;
        int ok = -1;
    };
    static_assert(sizeof(SparseShape) == 11 * sizeof(int) + sizeof(isc_tuning), "SparseShape has no padding");
    static thread_local Last last;
    if (last.ok < 0 || std::memcmp(&last.sh, &sh, sizeof sh) != 0) {
        last.ok = make_fused_plan(sh, &last.plan);
        last.sh = sh;
    }
    if (last.ok) *plan = last.plan;
    return last.ok != 0;
}

// Shapes of the filter-resident plan that the filter-ring kernel's walk runs:
// at stride 1 those wider than 16 columns (narrower ones keep the order of sums
// they share with the register-weight kernel), unless the caller names the
// kernel or a part of its plan.
// Streaming the filter through each wavefront's slot costs less than one
// resident copy that leaves a CU eight wavefronts (inception 5x5 at batch 128:
// 46 -> 25 us, 32 -> 64 maps of 20 x 20, 3x3, batch 64: 44 -> 22, 256 -> 64 maps
// of 28 x 28, 1x1, batch 2: 106 -> 20).
bool fused_walks(const SparseShape &sh, const FusedPlan &p) {
    const isc_tuning &tu = sh.tu;
    return !p.wreg && sh.T == 1 && sh.Wo > 16 && tu.kernel == 0 && tu.rows == 0 && tu.cols == 0 && tu.phases == 0 &&
           sparse_fring_applies(sh);
}

}  // namespace
}  // namespace fused

// The filter-resident kernel launches N * bands <= N * Ho workgroups; its
// register-weight variant N * bands * map groups, with bands <= Ho; the
// filter-ring kernel at most what its largest grid over its compiled tiles
// is (sparse_fring_max_groups).
int64_t sparse_fused_max_groups(const SparseShape &sh) {
    const int64_t reg = static_cast<int64_t>(sh.N) * sh.Ho * ((sh.K + 63) / 64);  // register-weight kernel
    return std::max(reg, sparse_fring_max_groups(sh));
}

bool sparse_fused_applies(const SparseShape &sh) {
    fused::FusedPlan p;
    return fused::fused_plan(sh, &p) || sparse_fring_applies(sh);
}

int sparse_fused_kernel(const SparseShape &sh) {
    fused::FusedPlan p;
    if (fused::fused_plan(sh, &p)) return p.wreg ? 6 : 1;
    return sparse_fring_applies(sh) ? 5 : 0;
}

bool sparse_reg_time_model(const SparseShape &sh, KernelTime *t) {
    using namespace fused;
    FusedPlan p;
    if (!fused_plan(sh, &p) || !p.wreg) return false;
    const RegCost c = reg_cost(sh, RegTile{p.th, p.tw, p.same});
    constexpr double kMs = 1.0 / 2.4e6;  // a cycle at 2.4 GHz
    *t = KernelTime{{c.issue0 * kMs, c.chain0 * kMs}, {c.issue1 * kMs, c.chain1 * kMs}};
    return true;
}

bool sparse_fused_plan_info(const SparseShape &sh, isc_plan *out) {
    using namespace fused;
    FusedPlan p;
    if (!fused_plan(sh, &p)) return sparse_fring_applies(sh) && sparse_fring_plan_info(sh, out);
    if (fused_walks(sh, p)) return sparse_fring_plan_info(sh, out);
    const int rg = kWaves / p.cs;
    const int64_t bands = (sh.Ho + rg * p.th - 1) / (rg * p.th);
    const int64_t kgroups = p.wreg ? (sh.K + kLanes - 1) / kLanes : 1;
    *out = isc_plan{p.wreg ? ISC_KERNEL_FUSED_REG : ISC_KERNEL_FUSED, p.th, p.tw, 1, p.cs, kWaves,
                    static_cast<int64_t>(sh.N) * bands * kgroups};
    return true;
}

// The filter-resident kernel when the filter fits in LDS, else the
// filter-ring kernel.
hipError_t launch_sparse_fused(const SparseShape &sh, const float *x, const float *wt, float *y, const Decision &dec,
                               hipStream_t s, const Epilogue &epi) {
    using namespace fused;
    FusedPlan p;
    if (!fused_plan(sh, &p) || fused_walks(sh, p)) return launch_sparse_fring(sh, x, wt, y, dec, s, epi);
    FusedArgs a{};
    a.x = x;
    a.wt = wt;
    a.y = y;
    a.N = sh.N; a.C = sh.C; a.H = sh.H; a.W = sh.W; a.K = sh.K; a.P = sh.P; a.Ho = sh.Ho; a.Wo = sh.Wo;
    a.cs = p.cs;
    a.rg = kWaves / p.cs;
    a.bands = (sh.Ho + a.rg * p.th - 1) / (a.rg * p.th);
    a.Kp = (sh.K + kLanes - 1) / kLanes * kLanes;
    a.kgroups = p.wreg ? a.Kp / kLanes : 1;
    a.wide = a.kgroups > 1 || sh.tu.wide_loads == 1;
    a.dec = dec;
    a.epi = epi;
    switch (sh.R) {
    case 1: return launch_r1(a, p, s);
    case 3: return launch_r3(a, p, s);
    default: return launch_r5(a, p, s);
    }
}

}  // namespace isc
