"""Staging room of the symmetric kick's tiles (csrc/genga_internal.h, SymShape),
compiled for the host: the tiles' segments lie behind one another without gaps, and a
wide tile has as much room per column as its shape promises."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2201_10058_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

CHECK = r'''
#include "genga_internal.h"
#include <cstdio>
using namespace genga;
static int check(int64_t n, int W, int A, int M)
{
    const SymShape h = sym_shape(n, W, A, M);
    if (h.P > M || h.P > SYM_PMAX || h.P & (h.P - 1)) return 1;
    int64_t at = 0;
    for (int64_t g = 0; g < h.G; ++g)
        for (int64_t s = 0; s < h.ns(g); ++s) {
            if (h.room(g, s) != at) return 2;
            if (h.segs(g, s) != (h.wide(g, s) ? h.P : 1)) return 3;
            at += h.segs(g, s);
        }
    if (h.room(h.G, 0) != at) return 4;
    if (h.P > 1 && at > SYM_ROOM) return 5;
    if (M == 1 && h.room(h.G, 0) != h.T) return 6;
    return 0;
}
int main()
{
    for (int64_t n : {1, 511, 512, 513, 4097, 8192, 8193, 12999, 13000, 14499, 14500, 20011, 23000, 39999, 40000, 46000,
                      65536, 131071})
        for (int W : {64, 128, 256, 512})
            for (int A : {0, 8, 16, 24})
                for (int M : {1, 2, 4}) {
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
def test_segments_follow_one_another(tmp_path):
    src = tmp_path / "check.hip"
    src.write_text(CHECK)
    exe = tmp_path / "check"
    subprocess.run([HIPCC, "--offload-host-only", "-O1", "-std=c++17",
                    f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
