// AUTO's per-shape crossover between the zero-skipping path and the dense
// path: the dispatcher of the paper's ISC (Sec. "Sparse Convolution")
// against the matrix-multiplication formulation of Fig. 3, decided by the
// measured sparsity of the input.  The paper's CPU experiments put the
// crossover near a sparsity of 0.9 (Abstract); on this GPU it depends on the
// shape: from below 0.5 (LeNet conv2, 5x5 filters at batch 256) to never
// (1x1 filters at batch 128, which the matrix cores run faster at any
// sparsity).
//
// Both paths' times are modelled from the plan the launch would run.  The
// register-weight and filter-ring kernels' models, which also choose their
// tiles, are the larger of two lines in the input's density (sparse_fused.hip,
// sparse_fring.hip); the filter-resident kernel's is one line, below.  The
// dense path's model is in dense_conv.hip.  The limit handed to the device
// is the largest nonzero count whose modelled sparse time does not exceed
// the modelled dense time; the device compares integers only.
#include "isc_internal.hpp"

#include <algorithm>
#include <cmath>

namespace isc {
namespace {

constexpr double kShortCall = 0.04;       // ms
constexpr double kShortSlower = 1.2;
constexpr double kChoiceLaunches = 0.009; // ms: the count's launch and the gated ones
constexpr double kGatedLaunches = 0.004;  // ms: the gated ones alone
constexpr double kCountPerInput = 1e-9;  // ms: 4 bytes at 4 TB/s

// The largest count whose density does not exceed dstar, where the dense path takes
// `dense` ms and the sparse path `no_zeros` on an input without any.
long long limit_for(double dstar, int64_t total, double dense, double no_zeros) {
    // a crossover past 0.95 sparsity counts as none: keeping the choice open
    // (the count, and the gated launch of the path not taken) costs more on
    // every call than the sparse path could save on the rare inputs past it
    // (Tab. 2's inception 4a.1 at batch 128: modelled crossover 0.97-0.99,
    // measured none up to 0.99; AUTO 18 % over the dense path at 0.9 while
    // it kept the choice)
    if (dstar < 0.05) return -1;
    // and on a short call, where the gated launches are a fifth, every input
    // counts as sparse if one without zeros takes the sparse path at most
    // kShortSlower times what the open choice costs it (inception 4e.3 at batch
    // 1: 16 us against 19 at 0.9, 25 against 29 at 0.6, 34 against 28 at 0.3 and 42
    // against 28 without zeros; 64 -> 192 maps of 56 x 56, 3x3, one image, left
    // open: 20 against 23, 32 against 31, 44 and 56 against 31)
    if (dstar >= 1.0 || (dense < kShortCall && no_zeros < kShortSlower * (dense + kChoiceLaunches)))
        return static_cast<long long>(total);
    // the kernels' models are those of rectified inputs: past a density of
    // 0.69 the two paths are within a tenth of each other where they cross
    return static_cast<long long>(std::floor(std::min(dstar, 0.69) * static_cast<double>(total)));
}

}  // namespace

long long crossover_nnz_limit(const SparseShape &sh) {
    const int64_t total = static_cast<int64_t>(sh.N) * sh.C * sh.H * sh.W;
    isc_plan p{};
    if (!sparse_fused_plan_info(sh, &p)) {
        // the kernels over compacted lists have no model, and the filter-ring
        // kernel's at stride 2 was not held against AUTO: the paper's 0.9
        return static_cast<long long>(std::floor(0.1 * static_cast<double>(total)));
    }
    const double dense = dense_time_model(sh.K, static_cast<int64_t>(sh.N) * sh.Ho * sh.Wo,
                                          static_cast<int64_t>(sh.C) * sh.R * sh.S);
    KernelTime rt;
    if (p.kernel == ISC_KERNEL_FUSED_REG ? sparse_reg_time_model(sh, &rt)
                                         : p.kernel == ISC_KERNEL_FUSED_RING && sparse_ring_time_model(sh, &rt)) {
        // kept open only where the sparse path, with its count, is the faster
        // one on a 0.95 sparse input: the count reads every input (12 us of
        // inception 4a.1's 54 at batch 128), and where the whole call is short
        // the count's launch and the gated ones weigh in (32 -> 64 maps of 20 x
        // 20, 3x3, batch 64: 19 us dense alone, 28 with the choice open)
        const double at95 = std::max(rt.base[0] + 0.05 * rt.slope[0], rt.base[1] + 0.05 * rt.slope[1]);
        const double launches = dense < kShortCall ? kChoiceLaunches : 0.0;
        if (at95 + launches + static_cast<double>(total) * kCountPerInput > dense) return -1;
        // the density where the first of the kernel's two bounds meets the
        // dense path, leaning a tenth to the sparse path, whose model is that
        // much too slow where the largest layer crosses (AlexNet conv2 at 0.6:
        // 720 us measured, 790 modelled)
        const double meet = 1.1 * dense;
        return limit_for(std::min((meet - rt.base[0]) / rt.slope[0], (meet - rt.base[1]) / rt.slope[1]), total, dense,
                         std::max(rt.base[0] + rt.slope[0], rt.base[1] + rt.slope[1]));
    }
    // the filter-resident kernel, with the count and repack before it: per round
    // of workgroups over the CUs and per channel of a wavefront a fixed part, the
    // static scan of its window and the window's nonzeros, and the filter's copy
    // into LDS.  Fitted to the sparse path timed on 90 shapes at sparsities 0.3 to
    // 0.95 (9 % rms, 36 % at most).
    const int wrows = (p.rows - 1) * sh.T + sh.R, wcols = (p.cols - 1) * sh.T + sh.S;
    const double pin = static_cast<double>(std::min(wrows, sh.H)) * std::min(wcols, sh.W);
    const double useful = static_cast<double>(std::min(p.rows, sh.Ho)) * std::min(p.cols, sh.Wo);
    const double taps = std::min<double>(sh.R * sh.S, useful * sh.R * sh.S / pin);
    const double rounds = std::ceil(static_cast<double>(p.workgroups) / 256.0);
    const double channels = (sh.C + std::max(1, p.phases) - 1) / std::max(1, p.phases);
    const double fixed = 0.00763 + rounds * (channels * (0.000142 + 4.54e-6 * wrows * wcols) + 8.8e-7 * sh.C * sh.R * sh.S);
    const double per_density = 3.05e-6 * rounds * channels * pin * (10.0 + taps);
    // as above, the count being in the time
    if (fixed + per_density <= dense) return static_cast<long long>(total);
    if (fixed + 0.05 * per_density + (dense < kShortCall ? kGatedLaunches : 0.0) > dense) return -1;
    return limit_for((dense - fixed) / per_density, total, dense, fixed + per_density);
}

}  // namespace isc
