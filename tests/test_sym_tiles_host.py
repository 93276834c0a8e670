"""Tile numbering of the symmetric kick (csrc/sym_common.h, SymShape), compiled
for the host: every launch slot names one tile of its own, every storage number
its group, and a group's slices cover its columns once, for slices of one and of
two widths."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2201_10058_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

CHECK = r'''
#include "sym_common.h"
#include <cstdio>
#include <vector>
using namespace genga;
static int check(int64_t n, int W, int A, int M)
{
    const SymShape h = sym_shape(n, W, A, M);
    std::vector<char> seen(h.T, 0);
    int64_t count = 0;
    for (int64_t t = 0; t < h.blocks(); ++t) {
        int64_t g, s;
        sym_tile(h, t, g, s);
        if (s < 0) continue;
        if (g < 0 || g >= h.G || s >= h.ns(g)) return 1;
        const int64_t sid = h.tb(g) + s;
        if (sid < 0 || sid >= h.T || seen[sid]) return 2;
        seen[sid] = 1;
        ++count;
        if (sym_group_of(h, sid) != g) return 3;
    }
    if (count != h.T) return 4;
    for (int64_t g = 0; g < h.G; ++g) {
        int64_t at = g * SYM_RG;
        for (int64_t s = 0; s < h.ns(g); ++s) {
            int64_t c0, c1;
            h.cols(g, s, c0, c1);
            if (c0 != at || c1 <= c0 || (c0 & 63)) return 5;
            if ((s < h.d) != (c0 < (g + 1) * SYM_RG)) return 6;
            at = c1;
        }
        if (at != n) return 7;
    }
    return 0;
}
int main()
{
    for (int64_t n : {1, 64, 511, 512, 513, 1025, 4097, 8192, 8193, 12999, 13000, 20011, 39999, 40000,
                      65536, 131071, 131072})
        for (int W : {64, 128, 256, 512})
            for (int A : {0, 8, 16, 24, 48})
                for (int M : {1, 2, 4, 8}) {
                    const int d = SYM_RG / W;
                    if (A % d || (A && A < d) || d % M || (!A && M != 1)) continue;
                    if (const int e = check(n, W, A, M)) {
                        std::printf("n %ld W %d A %d M %d: %d\n", (long)n, W, A, M, e);
                        return 1;
                    }
                }
    return 0;
}
'''


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_tiles_cover_every_column_once(tmp_path):
    src = tmp_path / "check.hip"
    src.write_text(CHECK)
    exe = tmp_path / "check"
    subprocess.run([HIPCC, "--offload-host-only", "-O1", "-std=c++17",
                    f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
