"""The groups of tiles that K-means bounds are kept for, over every split of 1 to 1024 clusters into partitions: they fit the tables a workgroup
keeps of them, and each tile of a partition lies in exactly the group that the tile's entry names."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2604_10060_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include "lloyd_groups.h"
using namespace mosaic;
static int check(int P, int C) {
    const int Cs = P ? C / P : 0;
    const LloydGroups g(P, Cs, C);
    if (g.span < 1 || g.span > kLloydTiles) return 1;
    if (g.lo(0) != 0 || g.lo(kLloydGroups) != g.span) return 2;
    for (int t = 0; t < g.span; ++t)
        if (g.of(t) < 0 || g.of(t) >= kLloydGroups || t < g.lo(g.of(t)) || t >= g.lo(g.of(t) + 1)) return 3;
    for (int p = 0; p < (P ? P : 1); ++p) {
        const int lo = P ? p * Cs : 0, hi = P ? lo + Cs : C, t0 = lo / 16, t1 = (hi - 1) / 16 + 1;
        if (t1 - t0 > g.span) return 4;
        unsigned long long all = 0;
        for (int i = 0; i < kLloydGroups; ++i) {
            const unsigned long long m = g.tiles(i, t0, t1);
            if (all & m) return 5;
            all |= m;
            for (int t = t0; t < t1; ++t)
                if (((m >> t) & 1) != (unsigned long long)(g.of(t - t0) == i)) return 6;
        }
    }
    return 0;
}
int main() {
    for (int P = 0; P <= 64; ++P)
        for (int C = 1; C <= 1024; ++C)
            if (P == 0 || C % P == 0)
                if (const int e = check(P, C)) { printf("P %d C %d: %d\n", P, C, e); return 1; }
    return 0;
}
"""


def test_groups_of_tiles(tmp_path):
    src = tmp_path / "groups.cpp"
    src.write_text(SOURCE)
    exe = str(tmp_path / "groups")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", CSRC, "-o", exe, str(src)])
    p = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr
