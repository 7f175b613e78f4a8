"""CPU check of the reads of the K-split tile product (gemm_splitk.h): its
descriptors are built from splitk_bytes, compiled here for the host, and replayed
over every order, tile shape and group of columns that its callers use.  Every
byte that a descriptor covers lies inside the matrix, and every element that a
tile needs lies inside its descriptor.  With sizes counted from the shifted base
(the oracle's planted mistake) the same replay finds reads past the end."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

REPLAY = r"""
#include <algorithm>
#include <cstdio>
#include "splitk_extent.h"

static unsigned shifted_base(int kn, int ld, int) { return kn > 0 ? (unsigned)kn * (unsigned)ld * 8u : 0u; }

// rows r0 .. r0 + tile - 1 of `rows` in K columns of a matrix with cols columns:
// whether a read leaves the matrix or misses an element
template <typename Size>
static bool bad(Size size, int rows, int ld, int cols, int K, int r0, int tile, int group) {
    for (int k0 = 0; k0 < K + 4 * group; k0 += group) {
        const int kn = std::max(0, std::min(group, K - k0));
        const long long bytes = size(kn, ld, r0), base = ((long long)k0 * ld + r0) * 8;
        // what the lanes ask for: kn columns, tile rows each
        const long long asked = kn ? ((long long)(group - 1) * ld + tile) * 8 : (long long)tile * 8;
        if (base + std::min(bytes, asked) > (long long)ld * cols * 8 && std::min(bytes, asked) > 0) return true;
        const int last = std::min(rows, r0 + tile) - 1;  // the last row that is used
        if (kn && ((long long)(kn - 1) * ld + last - r0 + 1) * 8 > bytes) return true;
    }
    return false;
}

// the first order at which one does, or 0
template <typename Size>
static int first_bad(Size size) {
    const int heights[3] = {32, 64, 96}, groups[5] = {8, 16, 20, 24, 32};
    for (int n = 3; n <= 6300; n += n < 1200 ? 1 : 3) {
        const int ld = (n + 63) / 64 * 64;
        for (int tile : heights)
            for (int g : groups) {
                const int r0 = (n - 1) / tile * tile;  // the last tile of rows
                if (bad(size, n, ld, n, n, r0, tile, g) || bad(size, n, ld, n, n, 0, tile, g)) return n;
                if (n % 2) continue;
                // an embedding of order n: rows of Re and of Im, K over the left block column or all
                const int h = n / 2, e0 = (h - 1) / tile * tile;
                for (int part = 0; part < 2; part++)
                    if (bad(size, n, ld, n, h, e0 + part * h, tile, g) || bad(size, n, ld, h, h, e0 + part * h, tile, g)) return n;
            }
    }
    return 0;
}

int main() {
    const int real = first_bad(splitk_bytes), planted = first_bad(shifted_base);
    std::printf("%d %d\n", real, planted);
    return 0;
}
"""


def test_reads_stay_inside(tmp_path):
    src, exe = tmp_path / "replay.cpp", tmp_path / "replay"
    src.write_text(REPLAY)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2308_03140_amd", "csrc"),
                           str(src), "-o", str(exe)])
    real, planted = map(int, subprocess.check_output([str(exe)]).split())
    assert real == 0, "order %d" % real
    assert planted > 0
