// Weight-gradient kernel (sparse_dw.hpp): the plan, the ordered sum of the
// ranges and the launch.
#include "sparse_dw.hpp"

#include <algorithm>

namespace isc {
namespace dwk {
namespace {

// One range's sums for (c, r, s) = e and the 64 maps of a wavefront's lanes
// (map k, at most K - 1), over the outputs alone and the nonzero inputs in
// order: 64 inputs are tested at a time, each nonzero meets the maps' gradients.
// Ends early where every wanted lane has its NaN.
__device__ float dw_range_again(const DwArgs &a, int R, int range, int e, int k, bool wanted) {
    const int lane = threadIdx.x & (kLanes - 1);
    const int c = e / (R * R), rs = e - c * R * R;
    const int dyr = rs / R - a.P, dxs = rs % R - a.P;
    float sum = 0.0f;
    const int t1 = min(a.ntiles, (range + 1) * a.per);
    for (int t = range * a.per; t < t1; ++t) {
        const int ox0 = t % a.ctiles * a.tw, oy0 = t / a.ctiles % a.bands * a.th, n = t / a.ctiles / a.bands;
        const int rows = min(a.th, a.Ho - oy0), cols = min(a.tw, a.Wo - ox0);
        const float *x = a.x + (static_cast<size_t>(n) * a.C + c) * a.H * a.W;
        const float *g = a.dy + ((static_cast<size_t>(n) * a.K + k) * a.Ho + oy0) * a.Wo + ox0;
        for (int p0 = 0; p0 < rows * cols; p0 += kLanes) {
            const int p = p0 + lane, i = p / cols, j = p - i * cols;
            const int y = oy0 + i + dyr, xx = ox0 + j + dxs;
            float v = 0.0f;
            if (i < rows && y >= 0 && y < a.H && xx >= 0 && xx < a.W) v = x[static_cast<size_t>(y) * a.W + xx];
            for (unsigned long long nz = __ballot(v != 0.0f); nz; nz &= nz - 1) {
                const int l = __builtin_ctzll(nz), q = p0 + l;
                const float vl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
                sum = __builtin_fmaf(vl, g[static_cast<size_t>(q / cols) * a.Wo + q % cols], sum);
            }
            if (!__any(wanted && !__builtin_isnan(sum))) return sum;
        }
    }
    return sum;
}

// dw[k][e] = sum over ranges of part[range][e][k] (e = (c, r, s)): a block
// takes 8 values of e times 64 maps; wavefront w adds the ranges w, w + 4, ...
// in order, consecutive lanes on consecutive maps, eight loads and more in
// flight, then the four sums are added in order and written with consecutive
// lanes on consecutive e.  Where a sum is not finite, its ranges are added again,
// those that are not finite themselves summed anew (AlexNet conv3 with one NaN
// 178 us in all, 141 without, conv2 497 and 351; a thread per entry over all its
// outputs took 5600 and 27500).
constexpr int kRedE = 8, kRedWaves = 4;

__global__ __launch_bounds__(kRedWaves * kLanes)
void dw_reduce_kernel(DwArgs a, int R, float *__restrict__ dw) {
    __shared__ float turn[kRedWaves][kRedE][kLanes + 1];
    const int crs = a.C * R * R;
    const int e0 = blockIdx.x * kRedE, k0 = blockIdx.y * kLanes;
    const int lane = threadIdx.x & (kLanes - 1), wave = threadIdx.x / kLanes;
    const size_t stride = static_cast<size_t>(crs) * a.Kp;
    const float *src = a.part + static_cast<size_t>(e0) * a.Kp + k0 + lane;
    const int last = min(kRedE, crs - e0) - 1;  // rows past it load it again and are dropped
    float sum[kRedE];
#pragma unroll
    for (int i = 0; i < kRedE; ++i) sum[i] = 0.0f;
#pragma unroll 4
    for (int sp = wave; sp < a.splits; sp += kRedWaves)
#pragma unroll
        for (int i = 0; i < kRedE; ++i) sum[i] += src[sp * stride + static_cast<size_t>(min(i, last)) * a.Kp];
#pragma unroll
    for (int i = 0; i < kRedE; ++i) turn[wave][i][lane] = sum[i];
    __syncthreads();
    const int col = threadIdx.x & (kRedE - 1);
    float finite = 0.0f;  // NaN where a sum is not finite
    if (e0 + col < crs) {
        for (int m = threadIdx.x / kRedE; m < kLanes; m += kRedWaves * kLanes / kRedE) {
            const int k = k0 + m;
            if (k >= a.K) break;
            float s = turn[0][col][m];
            for (int w = 1; w < kRedWaves; ++w) s += turn[w][col][m];
            finite = __builtin_fmaf(s, 0.0f, finite);
            dw[static_cast<size_t>(k) * crs + e0 + col] = s;
        }
    }
    if (!__syncthreads_or(!(finite == 0.0f))) return;
    for (int i = wave; i <= last; i += kRedWaves) {
        float s = turn[0][i][lane];
        for (int w = 1; w < kRedWaves; ++w) s += turn[w][i][lane];
        const bool odd = k0 + lane < a.K && !__builtin_isfinite(s);
        if (!__any(odd)) continue;
        float all = 0.0f;
        for (int sp = 0; sp < a.splits; ++sp) {
            float v = src[sp * stride + static_cast<size_t>(i) * a.Kp];
            const bool again = odd && !__builtin_isfinite(v);
            if (__any(again)) {
                const float r = dw_range_again(a, R, sp, e0 + i, min(k0 + lane, a.K - 1), again);
                v = again ? r : v;
            }
            all += v;
        }
        if (odd) dw[static_cast<size_t>(k0 + lane) * crs + e0 + i] = all;
    }
}

// Workgroups the ranges are cut for: one round of three per CU.  More ranges
// would write and read more partial sums (AlexNet conv3: 3.5 MB each).
constexpr int64_t kDwGroups = 768;

// The tiles compiled for a filter size.
int dw_tiles(int R, const DwTile **tiles) {
    *tiles = R == 1 ? kDwTiles1 : (R == 3 ? kDwTiles3 : kDwTiles5);
    return static_cast<int>(R == 1 ? sizeof(kDwTiles1) : (R == 3 ? sizeof(kDwTiles3) : sizeof(kDwTiles5))) /
           static_cast<int>(sizeof(DwTile));
}

// Whether a tile takes the shape: the positions its walk leaves out are padding.
bool dw_tile_takes(const SparseShape &sh, const DwTile &t) {
    if (t.same >= 1 && (sh.P != sh.R / 2 || sh.W > t.tw)) return false;
    return t.same < 2 || sh.H <= t.th;
}

// The first tile that takes the shape and that a caller's rows and cols name;
// else the cheapest among those that take it: a wavefront's cycles per
// tile (reading the gradients, and per channel a fixed part and the window's
// nonzeros at a tenth of its positions) times the tiles of all workgroups, or
// of one round where the tiles do not fill it (small batches, where short
// tiles give more workgroups).
bool dw_plan(const SparseShape &sh, DwPlan *p) {
    if (sh.T != 1 || sh.R != sh.S || !(sh.R == 1 || sh.R == 3 || sh.R == 5)) return false;
    const DwTile *tiles;
    const int n = dw_tiles(sh.R, &tiles);
    int named = -1;
    for (int i = 0; i < n && named < 0 && (sh.tu.rows > 0 || sh.tu.cols > 0); ++i)
        if (dw_tile_takes(sh, tiles[i]) && (sh.tu.rows <= 0 || tiles[i].th == sh.tu.rows) &&
            (sh.tu.cols <= 0 || tiles[i].tw == sh.tu.cols))
            named = i;
    p->kgroups = (sh.K + kLanes - 1) / kLanes;
    double best = -1.0;
    int64_t ntiles = 0;
    for (int i = 0; i < n; ++i) {
        const DwTile &t = tiles[i];
        if (named >= 0 ? i != named : !dw_tile_takes(sh, t)) continue;
        const int64_t bands = (sh.Ho + t.th - 1) / t.th, ctiles = (sh.Wo + t.tw - 1) / t.tw;
        const int64_t cgroups = (sh.C + kDwWaves * t.ch - 1) / (kDwWaves * t.ch);
        const int64_t nt = sh.N * bands * ctiles;
        const double rows = std::min(t.same == 2 ? t.th : t.th + sh.R - 1, sh.H);
        const double cols = std::min(t.same ? t.tw : t.tw + sh.R - 1, sh.W);
        const double fmas = std::min<double>(t.th, sh.Ho) * std::min(t.tw, sh.Wo) * sh.R * sh.R / (rows * cols);
        const double per = 400.0 + 8.0 * t.th * t.tw +
                           t.ch * (150.0 + 8.0 * sh.R * sh.R + 0.1 * rows * cols * (15.0 + 4.0 * fmas));
        const double cost = std::max<double>(static_cast<double>(nt) * cgroups * p->kgroups, kDwGroups) * per;
        if (best < 0.0 || cost < best) {
            best = cost;
            ntiles = nt;
            p->t = t;
            p->bands = static_cast<int>(bands);
            p->ctiles = static_cast<int>(ctiles);
            p->cgroups = static_cast<int>(cgroups);
        }
    }
    if (ntiles > (1ll << 30)) return false;
    p->ntiles = static_cast<int>(ntiles);
    const int64_t base = static_cast<int64_t>(p->kgroups) * p->cgroups;
    const int64_t splits = std::max<int64_t>(1, std::min<int64_t>(ntiles, kDwGroups / base));
    p->per = static_cast<int>((ntiles + splits - 1) / splits);
    p->splits = static_cast<int>((ntiles + p->per - 1) / p->per);
    return base * p->splits < (1ll << 31);
}

}  // namespace
}  // namespace dwk

bool sparse_dw_applies(const SparseShape &sh) {
    dwk::DwPlan p;
    return dwk::dw_plan(sh, &p);
}

bool sparse_dw_plan_info(const SparseShape &sh, DwPlanInfo *out) {
    dwk::DwPlan p;
    if (!dwk::dw_plan(sh, &p)) return false;
    *out = DwPlanInfo{p.t.th, p.t.tw, p.t.same, p.t.ch, p.splits};
    return true;
}

// The largest partial-sum buffer of any tile a caller may name, so that one
// workspace size holds for every plan.
size_t sparse_dw_workspace_floats(const SparseShape &sh) {
    using namespace dwk;
    DwPlan p;
    if (!dw_plan(sh, &p)) return 0;
    int most = p.splits;
    const DwTile *tiles;
    const int n = dw_tiles(sh.R, &tiles);
    SparseShape v = sh;
    v.tu = isc_tuning{};
    for (int i = 0; i < n; ++i) {
        v.tu.rows = tiles[i].th;
        v.tu.cols = tiles[i].tw;
        if (dw_plan(v, &p)) most = std::max(most, p.splits);
    }
    return static_cast<size_t>(most) * sh.C * sh.R * sh.S * p.kgroups * kLanes;
}

hipError_t launch_sparse_dw(const SparseShape &sh, const float *x, const float *dy, float *dw, float *part,
                            hipStream_t s) {
    using namespace dwk;
    DwPlan p;
    if (!dw_plan(sh, &p)) return hipErrorInvalidValue;
    DwArgs a{};
    a.x = x;
    a.dy = dy;
    a.part = part;
    a.N = sh.N; a.C = sh.C; a.H = sh.H; a.W = sh.W; a.K = sh.K; a.P = sh.P; a.Ho = sh.Ho; a.Wo = sh.Wo;
    a.Kp = p.kgroups * kLanes;
    a.ctiles = p.ctiles;
    a.bands = p.bands;
    a.cgroups = p.cgroups;
    a.splits = p.splits;
    a.per = p.per;
    a.ntiles = p.ntiles;
    a.th = p.t.th;
    a.tw = p.t.tw;
    hipError_t e = sh.R == 1 ? launch_r1(a, p, s) : sh.R == 3 ? launch_r3(a, p, s) : launch_r5(a, p, s);
    if (e != hipSuccess) return e;
    const int crs = sh.C * sh.R * sh.S;
    const dim3 grid(static_cast<unsigned>((crs + kRedE - 1) / kRedE), static_cast<unsigned>(p.kgroups));
    dw_reduce_kernel<<<grid, kRedWaves * kLanes, 0, s>>>(a, sh.R, dw);
    return hipGetLastError();
}

}  // namespace isc
