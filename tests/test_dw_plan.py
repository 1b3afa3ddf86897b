"""The weight gradient's choice of tile (host-side, no GPU): the cases of the
GPU tests run the tile they name, between them every compiled one, and the
workspace holds for every tile a caller may name."""
import os
import re
import subprocess

import pytest

import paper_1704_07724_amd as isc
from paper_1704_07724_amd import build as B
from test_gpu_dw import DW_TILES

SOURCE = r'''
#include "isc_internal.hpp"
#include <cstdio>
// N C H W K R P rows cols per line -> rows cols same channels ranges
int main() {
    isc::SparseShape s{};
    int rows, cols;
    s.T = 1;
    while (std::scanf("%d %d %d %d %d %d %d %d %d", &s.N, &s.C, &s.H, &s.W, &s.K, &s.R, &s.P, &rows, &cols) == 9) {
        s.S = s.R;
        s.Ho = s.H + 2 * s.P - s.R + 1;
        s.Wo = s.W + 2 * s.P - s.R + 1;
        s.tu.rows = rows;
        s.tu.cols = cols;
        isc::DwPlanInfo p{};
        if (!isc::sparse_dw_plan_info(s, &p)) return 1;
        std::printf("%d %d %d %d %d\n", p.rows, p.cols, p.same, p.channels, p.ranges);
    }
}
'''


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if not os.path.exists(B.HIPCC):
        pytest.skip("ROCm toolchain not available")
    isc.lib()
    d = tmp_path_factory.mktemp("dw")
    (d / "plan.hip").write_text(SOURCE)
    subprocess.run([B.HIPCC, "--offload-arch=" + B.ARCH, "-std=c++17", "-I", B.INCLUDE, "-I", B.CSRC, str(d / "plan.hip"),
                    "-o", str(d / "plan"), "-x", "none", B.LIB, "-Wl,-rpath," + os.path.dirname(B.LIB)], check=True, capture_output=True)

    def run(cases):
        text = "".join(" ".join(map(str, c)) + "\n" for c in cases)
        out = subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def compiled_tiles():
    text = open(os.path.join(B.CSRC, "sparse_dw.hpp")).read()
    return {(int(m[0]),) + tuple(int(v) for v in t)[:3]
            for m in re.findall(r"kDwTiles(\d)\[\] = \{(.*?)\};", text)
            for t in re.findall(r"\{(\d+), (\d+), (\d+), \d+\}", m[1])}


def test_named_tiles_run(plans):
    got = plans(DW_TILES)
    assert [p[:2] for p in got] == [c[7:] for c in DW_TILES]
    assert {(c[5],) + p[:3] for c, p in zip(DW_TILES, got)} == compiled_tiles()


def test_unfit_names_are_ignored_and_the_workspace_holds(plans):
    # 40 columns: neither 7 x 13 nor 8 x 8 is a tile of it, so the library's own choice runs
    wide = (4, 40, 21, 40, 130, 3, 1)
    assert plans([wide + (7, 13), wide + (8, 8)]) == plans([wide + (0, 0)]) * 2
    for c in DW_TILES + [(128, 256, 13, 13, 384, 3, 1, 0, 0), (128, 96, 27, 27, 256, 5, 2, 0, 0)]:
        N, C, H, W, K, R, P = c[:7]
        size = isc.isc_conv2d_dw_workspace_size(isc.make_desc(N, C, H, W, K, R, R, 1, P))
        tiles = [t[1:3] for t in compiled_tiles() if t[0] == R]
        most = max(p[4] for p in plans([c[:7] + t for t in tiles + [(0, 0)]]))
        assert size >= 4 * most * C * R * R * ((K + 63) // 64 * 64)


def test_conv3_takes_the_tall_tile(plans):
    """AlexNet conv3's gradient at batch 128 runs 7 x 13 tiles, in one round of
    three workgroups per CU: 6 groups of maps x 16 of channels x 8 ranges."""
    assert plans([(128, 256, 13, 13, 384, 3, 1, 0, 0)]) == [(7, 13, 1, 4, 8)]
