"""The decode's split of cached rows over workgroups, checked on the host by enumeration: a
small program over the library's own header and geometry walks head layouts, masks, batch
sizes, bounds and contexts (negative ones and ones past the bound among them) and asserts, for
each, that

  * the splits with rows cover a problem's visible rows once, are no more than the launch has
    and the workspace has room for, and do not depend on capacity or bound;
  * a context outside [0, bound] counts as the nearest one inside, so that no index leaves the
    grid, the workspace or the cache;
  * every (problem, split) has exactly one workgroup, neighbouring heads that share cache lines
    stay on one XCD, and the first splits alone - all that short contexts under a loose bound
    leave - spread over the XCDs to within one unit of heads.
"""
import os
import shutil
import subprocess

import pytest

import paper_2607_08186_amd as hd

CSRC = os.path.join(os.path.dirname(hd.__file__), "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "decode_internal.h"

using namespace hd;

#define CHECK(x) \
    do { \
        if (!(x)) { \
            std::printf("failed: %s (B=%d Lcap=%d n=%d Hq=%d Hkv=%d D=%d mode=%d window=%d bound=%d ctx=%d)\n", #x, \
                        g.B, g.Lcap, g.n, g.Hq, g.Hkv, g.D, g.mode, g.window, g.max_ctx, ctx); \
            std::exit(1); \
        } \
    } while (0)

static int used(const DecRows &r) { return (r.kvlen - r.klo + r.per - 1) / r.per; }

int main()
{
    const int heads[][2] = {{8, 8}, {32, 8}, {16, 4}, {12, 4}, {6, 3}, {64, 8}, {5, 1}};
    const int bounds[] = {0, 1, 255, 256, 384, 640, 700, 1023, 1024, 1025, 2500, 5000, 40000};
    long cases = 0;
    for (const auto &h : heads)
        for (int D : {32, 64, 128})
            for (int n : {1, 3, 4, 8})
                for (int B : {1, 2, 5, 8, 16, 17, 33, 80})
                    for (int mode : {0, 1, 2})
                        for (int window : {1, 100, 3000, 2147483647}) {
                            if (mode != 2 && window != 1) continue;
                            for (int bound : bounds) {
                                const DecGeom g = make_dec_geom(B, bound + 1, n, h[0], h[1], D, mode, window, 1.f, bound);
                                const DecGeom big = make_dec_geom(B, 50001, n, h[0], h[1], D, mode, window, 1.f, 50000);
                                int ctx = 0;
                                CHECK(g.nsplit >= 1 && g.nsplit <= g.nchunk);
                                for (int c : {-7, 0, 1, 30, 100, 255, 300, 383, 500, 640, 800, 1024, 1500, 2047, 2100, 4096, 9000, 39999, 60000}) {
                                    ctx = c;
                                    const DecRows r = dec_rows(g, c);
                                    CHECK(r.ctx == std::min(std::max(c, 0), bound));
                                    CHECK(r.klo >= 0 && r.klo < r.kvlen && r.kvlen <= (mode == 0 ? 1 : n) * (bound + 1));
                                    CHECK(r.per >= 1 && used(r) >= 1 && used(r) <= g.nsplit);
                                    CHECK(used(r) == 1 || r.per % kDecTile == 0);
                                    if (mode == 2) {
                                        const long lo = std::max(0L, (long)r.ctx * n - window + 1);
                                        CHECK(r.klo <= lo && lo - r.klo < kDecTile);
                                    } else {
                                        CHECK(r.klo == 0);
                                    }
                                    const DecRows rb = dec_rows(big, r.ctx);
                                    CHECK(rb.per == r.per && rb.klo == r.klo && rb.kvlen == r.kvlen);
                                    CHECK(g.waves == big.waves);
                                    ++cases;
                                }
                            }
                        }
    for (const auto &h : heads)
        for (int D : {32, 64, 128})
            for (int n : {1, 4})
                for (int B : {1, 3, 8, 40})
                    for (int mode : {0, 1})
                        for (int bound : {100, 2000, 20000}) {
                            const DecGeom g = make_dec_geom(B, bound + 1, n, h[0], h[1], D, mode, 0, 1.f, bound);
                            const int ctx = bound;
                            std::vector<int> seen((size_t)g.problems * g.nsplit);
                            std::vector<int> xcd((size_t)g.problems), load(8);
                            const int64_t grid = dec_grid(g);
                            CHECK(grid < (1LL << 31));
                            for (int64_t id = 0; id < grid; ++id) {
                                DecProblem p;
                                int split;
                                if (!dec_place(g, (int)id, p, split)) continue;
                                const int ix = dec_index(g, p);
                                CHECK(p.b >= 0 && p.b < B && p.hk >= 0 && p.hk < g.Hkv && p.gc >= 0 && p.gc < g.ngc);
                                CHECK(p.s >= 0 && p.s < (mode == 0 ? n : 1) && split >= 0 && split < g.nsplit);
                                CHECK(ix >= 0 && ix < g.problems);
                                ++seen[(size_t)ix * g.nsplit + split];
                                if (split == 0) {
                                    xcd[ix] = (int)(id & 7);
                                    ++load[id & 7];
                                }
                            }
                            for (int s : seen) CHECK(s == 1);
                            CHECK(*std::max_element(load.begin(), load.end()) -
                                      *std::min_element(load.begin(), load.end()) <= g.heads);
                            if (D == 32)  // two neighbouring heads' rows fill one 128-byte line
                                for (int b = 0; b < B; ++b)
                                    for (int hk = 0; hk + 1 < g.Hkv; hk += 2) {
                                        if (g.Hkv % 2) continue;
                                        CHECK(xcd[dec_index(g, DecProblem{b, hk, 0, 0})] ==
                                              xcd[dec_index(g, DecProblem{b, hk + 1, 0, 0})]);
                                    }
                            ++cases;
                        }
    std::printf("%ld cases\n", cases);
    return 0;
}
"""


def test_decode_splits_enumerated(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP headers")
    src, exe = tmp_path / "splits.cpp", tmp_path / "splits"
    src.write_text(PROGRAM)
    lib = hd.binding.LIB_PATH
    subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
                    os.path.join(ROCM, "include"), str(src), lib, f"-Wl,-rpath,{os.path.dirname(lib)}",
                    f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}", "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                    "-w", "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("cases"), r.stdout
