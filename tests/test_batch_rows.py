"""Rows per thread of a batch's reconstruction (CPU): 1, 2 and 8 hold for every
view as they are asked for, 4 stands for the height by pairing and display
size, and the kernel of a frame holds the heights of its views."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "vafr_internal.h"
using namespace vafr;
static ReconView view(int w, int h, bool pair, bool dense) {
    static float4 other;
    ReconView v{};
    v.width = w;
    v.height = h;
    v.mode = dense ? kModeLmfr : kModeVafr;
    v.lp2 = pair ? &other : nullptr;
    return v;
}
int main() {
    const ReconView kinds[5] = {view(640, 361, true, false), view(7680, 4320, true, false),
                                view(640, 361, false, false), view(7680, 4320, false, false),
                                view(7680, 4320, false, true)};
    for (int rows : {1, 2, 4, 8}) {
        ReconView v[5];
        for (int k = 0; k < 5; ++k) {
            v[k] = kinds[k];
            v[k].rows = recon_rows_of(v[k], rows);
            std::printf("%d %lld %d ", v[k].rows, (long long)recon_blocks_of(v[k], v[k].rows),
                        recon_launch_rows(v + k, 1, rows));
        }
        const ReconView pairs[2] = {v[0], v[1]}, small[2] = {v[2], v[4]}, mixed[2] = {v[0], v[2]};
        std::printf("%d %d %d\n", recon_launch_rows(pairs, 2, rows), recon_launch_rows(small, 2, rows),
                    recon_launch_rows(mixed, 2, rows));
    }
}
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    from paper_2503_23410_amd import build as B
    d = tmp_path_factory.mktemp("rows")
    src, exe = str(d / "rows.cpp"), str(d / "rows")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([B.hipcc(), "-x", "hip", "--cuda-host-only", "-std=c++17", "-I", B.INCLUDE, "-I", B.CSRC, src,
                    "-x", "none", B.LIB, f"-Wl,-rpath,{B.PKG}", "-o", exe], check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return {rows: [int(x) for x in line.split()] for rows, line in zip((1, 2, 4, 8), out.splitlines())}


def _blocks(w, h, rows):
    return -(-w // 64) * -(-h // (4 * rows))


SIZES = [(640, 361), (7680, 4320), (640, 361), (7680, 4320), (7680, 4320)]
MIXED = 0


@pytest.mark.parametrize("rows", [1, 2, 8])
def test_asked_rows_are_taken(table, rows):
    for k, (w, h) in enumerate(SIZES):
        assert table[rows][3 * k:3 * k + 3] == [rows, _blocks(w, h, rows), rows]
    assert table[rows][15:] == [rows, rows, rows]


def test_default_chooses_by_view(table):
    heights = [2, 2, 4, 8, 4]    # pairs, a small and a large view alone, a dense view
    kernels = [2, 2, 4, MIXED, 4]
    for k, (w, h) in enumerate(SIZES):
        assert table[4][3 * k:3 * k + 3] == [heights[k], _blocks(w, h, heights[k]), kernels[k]]
    assert table[4][15:] == [2, 4, MIXED]
