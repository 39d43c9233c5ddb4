"""The addresses the dense solve's two passes over the packed triangle read, for every
row bucket and workgroup size the step kernel is built for and every row count of
the bucket, against the regions of the workgroup's LDS.  The kernel's own index
functions, compiled for the host."""
import subprocess

from paper_2603_16536_amd import build

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "kamx_internal.h"
using namespace kamx;
int main() {
    int bad = 0;
    for (const BucketSizes &b : kBucketSizes)
        for (int v = 0; v < b.n; ++v)
            for (int m = 1; m <= b.mc; ++m) {
                const int mc = b.mc, nt = b.nt[v], Q = (m + 3) >> 2, tri = tri_row_offset(mc);
                int last = 0, last_t = 0, pairs = 0;
                for (int gg = 0; gg < nt / 16; ++gg) {
                    // t = X r: four rows of a first and of a second group, the
                    // column quads up to the diagonal's
                    for (int G : {pair_first(gg, mc), std::max(Q - 1 - gg, 0)})
                        last = std::max(last, tri_row_offset(4 * G) + 3 * 4 * (G + 1) + 4 * G + 3);
                    // a thread group within the world's pairs reads its own pair
                    const bool one = gg <= Q - 1 - gg;
                    pairs += one;
                    if (one && pair_first(gg, mc) != gg) ++bad;
                    // X^T t: t of a thread's slots
                    for (int kq = 0; kq < 16; ++kq) {
                        const int x1 = (mc + 63) / 64, x2 = (mc / 2 + 63) / 64, c2 = Q - 1 - gg;
                        last_t = std::max(last_t, 4 * (std::min(gg, mc / 8) + kq) + 64 * (x1 - 1) + 3);
                        last_t = std::max(last_t, 4 * (std::min(std::max(c2, 0), mc / 4) + kq) + 64 * (x2 - 1) + 3);
                    }
                }
                if (pairs != (Q + 1) / 2) ++bad;  // every pair has its threads
                if (last >= tri || last_t >= t_floats(mc)) {
                    if (bad < 20) std::printf("%d rows of %d on %d threads: triangle %d of %d, t %d of %d\n", m, mc, nt, last, tri, last_t, t_floats(mc));
                    ++bad;
                }
            }
    std::printf("%d out of range\n", bad);
    return bad != 0;
}
"""


def test_passes_over_the_triangle_stay_inside(tmp_path):
    src, exe = tmp_path / "ranges.hip", tmp_path / "ranges"
    src.write_text(PROGRAM)
    subprocess.run([build.hipcc(), "-std=c++17", "-O1", "--offload-host-only", "-I", build.CSRC, str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
