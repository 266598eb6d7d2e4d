"""How the network kernels' work items are dealt to blocks and dies, on the CPU: the
kernels' own functions, compiled with the host's compiler."""
import os
import shutil
import subprocess

import pytest

MAIN = r"""
#include "nps_internal.hpp"
#include <cstdio>
#include <vector>
using namespace nps;
// every item of nz x ny x nx once, over a grid of that many blocks; the largest share of a die over the mean
static double share(Grid g, int grid) {
    const Columns cl = march_columns(g);
    std::vector<int> seen(cl.count(), 0);
    double die[kXcds] = {0}, most = 0.0;
    for (int b = 0; b < grid; ++b) {
        const MarchItems m = march_items(cl, grid, b, march_slabs(cl, grid));
        for (int li = m.li; li < m.count; li += m.step) {
            const MarchItem it = march_item(m, li, cl);
            if (it.cx < 0 || it.cx >= cl.ncx || it.cy < 0 || it.cy >= cl.ncy || it.zc < 0 || it.zc >= cl.ncz) return -1.0;
            seen[(it.zc * cl.ncy + it.cy) * cl.ncx + it.cx] += 1;
            die[b % kXcds] += 1.0;
        }
    }
    for (int s : seen)
        if (s != 1) return -1.0;
    for (double d : die) most = d > most ? d : most;
    return most / (cl.count() / (double)kXcds);
}
int main() {
    int nz, ny, nx, grid;
    while (scanf("%d %d %d %d", &nz, &ny, &nx, &grid) == 4) {
        const Columns cl = march_columns(Grid{nz, ny, nx});
        printf("%d %.4f\n", cl.count(), share(Grid{nz, ny, nx}, tile_blocks(cl.count() < grid ? cl.count() : grid)));
    }
}
"""


@pytest.fixture(scope="module")
def program(repo_root, tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("items")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "items")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(repo_root, "paper_2310_00177_amd", "csrc"), str(d / "main.cpp"), "-o", exe], check=True)
    return exe


# chunk counts 1, 2, 4, 9, 17, 18, 33 and multiples of 8; a footprint of 2 columns; fewer items than blocks
SHAPES = [(2, 512, 512), (4, 512, 512), (8, 512, 512), (8, 256, 256), (36, 256, 256), (34, 38, 70), (36, 32, 32),
          (130, 130, 130), (64, 64, 64), (128, 128, 128), (256, 256, 256), (72, 64, 64), (4096, 64, 2), (2, 2, 2)]


def test_items_are_dealt_once_and_evenly(program):
    """Every item goes to one block, and no die gets more than a tenth (and an item) above the mean."""
    cases = [(*s, grid) for s in SHAPES for grid in (768, 1024, 1280)]
    out = subprocess.run([program], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True,
                         check=True).stdout.split()
    for case, count, share in zip(cases, map(int, out[::2]), map(float, out[1::2])):
        assert share > 0.0, case
        assert share <= 1.0 + 1.0 / 9.0 + 8.0 / count + 1e-3, (case, share)
