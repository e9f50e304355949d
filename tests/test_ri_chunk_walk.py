"""CPU replay of the column walk of the RI diagnostic: ri_chunk of
csrc/nh_ri.hip, compiled here for the host, run for every thread of every
workgroup.  Each lattice column of a level is visited once, with its own x and y
index, and no index handed to the per-column tables lies outside them."""
import os
import re
import subprocess

import pytest

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_2504_08157_amd", "csrc", "nh_ri.hip")

HOST = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#define __device__
#define __forceinline__ inline
struct { int x; } threadIdx;
struct RiParams { int nx, ny, nb, rg; };
%s
int main(int argc, char **argv)
{
    RiParams p;
    p.nx = atoi(argv[1]);
    p.ny = atoi(argv[2]);
    p.nb = atoi(argv[3]);
    p.rg = argc > 4 ? atoi(argv[4]) : ri_row_groups(p.nx, p.ny, p.nb);
    const long nxy = (long)p.nx * p.ny;
    std::vector<int> seen(nxy, 0);
    long out = 0, wrong = 0;
    for (int b = 0; b < p.nb; ++b)
        for (threadIdx.x = 0; threadIdx.x < kRiThreads; ++threadIdx.x) {
            int at = -1;
            ri_chunk(
                p, b,
                [&](int ix) {
                    at = ix;
                    out += ix < 0 || ix >= p.nx;
                },
                [&](long i, int iy, int n) {
                    for (int r = 0; r < n; ++r) {
                        const long j = i + (long)r * p.nx;
                        if (j < 0 || j >= nxy || iy + r >= p.ny) {
                            ++out;
                            continue;
                        }
                        ++seen[j];
                        wrong += at != j %% p.nx || iy + r != j / p.nx;
                    }
                },
                [] {});
        }
    long missed = 0;
    for (int s : seen) missed += s != 1;
    printf("%%ld %%ld %%ld\n", out, wrong, missed);
}
"""


def _walk():
    src = open(SRC).read()
    consts = re.findall(r"^constexpr int kRi(?:Threads|Rows) = \d+;", src, re.M)
    funs = [src[i:src.index("\n}\n", i) + 3] for i in (src.index("static int ri_row_groups("),
                                                       src.index("template <typename B, typename R, typename E>"))]
    return "\n".join(consts + funs)


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    d = tmp_path_factory.mktemp("ri")
    src, exe = d / "walk.cpp", d / "walk"
    src.write_text(HOST % _walk())
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(exe), str(src)], check=True)
    return str(exe)


# rows narrower than a wave, of a wave, a node more, ragged, several workgroup widths; chunks of whole
# rows and chunks that begin within a row; the workgroups per level the library would take and others
@pytest.mark.parametrize("nx,ny,nb", [(2, 3, 1), (12, 10, 1), (24, 24, 1), (63, 7, 1), (64, 140, 3), (65, 282, 5),
                                      (129, 165, 6), (260, 200, 13), (402, 100, 10), (512, 512, 64), (4104, 7, 8),
                                      (7, 2000, 4), (65, 2, 9)])
@pytest.mark.parametrize("rg", [None, 1, 2, 7, 4096])
def test_columns_visited_once_inside_the_tables(replay, nx, ny, nb, rg):
    """rg: the groups of rows, the library's own choice (None) and others, also more than rows."""
    out = subprocess.run([replay, str(nx), str(ny), str(nb)] + ([] if rg is None else [str(rg)]), check=True,
                         capture_output=True, text=True).stdout
    assert out.split() == ["0", "0", "0"], "indices outside, wrong coordinates, columns not visited once: " + out
