"""The second pass of the dense GEMM's split reduction never has more
workgroups than a census has counts for (host-side, no GPU)."""
import os
import subprocess

import pytest

from paper_1704_07724_amd import build as B

SOURCE = r'''
#include "isc_internal.hpp"
#include <cstdio>
int main() {
    for (int64_t k = 0; k <= 24; ++k)
        for (int64_t e = k * 131072 - 1100; e <= k * 131072 + 1100; ++e) {
            if (e < 1 || e >= (1ll << 31)) continue;
            const int64_t per = isc::split_reduce_per(e), groups = (e + per - 1) / per;
            if (per < 256 || per > 2048 || per % 256 != 0 || (groups > isc::kRectifyGroups && per != 2048)) {
                std::printf("%lld elements: %lld each, %lld workgroups\n", (long long)e, (long long)per, (long long)groups);
                return 1;
            }
        }
    return 0;
}
'''


def test_second_pass_fits_every_census(tmp_path):
    """At most 1024 workgroups (kRectifyGroups, the counts of the smallest
    census), or 2048 outputs each, one 32 x 64 tile of the GEMM."""
    if not os.path.exists(B.HIPCC):
        pytest.skip("ROCm toolchain not available")
    src, exe = tmp_path / "reduce.hip", str(tmp_path / "reduce")
    src.write_text(SOURCE)
    subprocess.run([B.HIPCC, "--offload-arch=" + B.ARCH, "-std=c++17", "-I", B.INCLUDE, "-I", B.CSRC, str(src), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
