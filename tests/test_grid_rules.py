"""The rule by which small forward and dQ grids take 128-row blocks, on the host: the library's own
header over shapes on both sides of its lines.  A grid of more such blocks than compute units runs
them in two rounds, which short and windowed sweeps must not be made to do."""
import os
import shutil
import subprocess

import pytest

import paper_2607_08186_amd as hd

CSRC = os.path.join(os.path.dirname(hd.__file__), "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = r"""
#include <cstdio>

#include "hd_internal.h"

int main()
{
    int final, mode, B, L, n, Hq, Hkv, D, window;
    while (std::scanf("%d %d %d %d %d %d %d %d %d", &final, &mode, &B, &L, &n, &Hq, &Hkv, &D, &window) == 9) {
        const hd::SfaGeom g = final ? hd::make_geom_final(B, L, n, Hq, Hkv, D, mode, 1.f, window)
                                    : hd::make_geom(B, L, n, Hq, Hkv, D, mode, 1.f, window);
        std::printf("%d%d\n", hd::fwd_split(g), hd::dq_split(g));
    }
    return 0;
}
"""

INTRA, MIX, LOCAL = 0, 1, 2
# (final, mode, B, L, n, Hq, Hkv, D, window), forward split, dQ split
SHAPES = [
    ((0, MIX, 1, 129, 1, 8, 2, 128, 0), 1, 1),
    ((0, MIX, 1, 128, 1, 8, 2, 128, 0), 0, 1),        # one key tile per group
    ((0, MIX, 16, 256, 1, 8, 2, 128, 0), 1, 1),       # 128 blocks, 256 halves
    ((0, MIX, 17, 250, 1, 8, 2, 128, 0), 0, 0),       # 136 short blocks, 272 halves
    ((0, MIX, 17, 250, 1, 8, 2, 64, 0), 0, 0),
    ((0, MIX, 17, 250, 1, 8, 2, 32, 0), 1, 1),        # two blocks per CU
    ((0, MIX, 9, 300, 1, 8, 2, 128, 0), 1, 1),        # 144 blocks, but 216 halves
    ((0, INTRA, 1, 250, 4, 48, 8, 128, 0), 0, 0),
    ((0, MIX, 9, 500, 1, 8, 2, 128, 0), 0, 0),
    ((0, MIX, 6, 800, 1, 8, 2, 128, 0), 1, 1),        # 192 blocks, long causal sweeps
    ((0, MIX, 8, 800, 1, 8, 2, 128, 0), 0, 0),        # 256 blocks
    ((0, LOCAL, 3, 1231, 1, 12, 4, 128, 235), 0, 0),  # 180 blocks of one length
    ((0, LOCAL, 2, 1231, 1, 12, 4, 128, 235), 1, 1),
    ((0, LOCAL, 3, 2000, 1, 8, 2, 128, 1000), 1, 0),
    ((0, LOCAL, 3, 2000, 1, 8, 2, 128, 2000), 1, 1),
    ((1, MIX, 24, 250, 4, 8, 2, 128, 0), 1, 0),
    ((1, MIX, 25, 250, 4, 8, 2, 128, 0), 0, 0),
    ((1, MIX, 6, 800, 2, 8, 2, 128, 0), 1, 1),
    ((1, LOCAL, 3, 1800, 4, 8, 2, 128, 400), 1, 0),
    ((1, MIX, 8, 1, 8, 8, 2, 64, 0), 1, 1),
]


def test_split_of_small_grids(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP headers")
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(PROGRAM)
    lib = hd.binding.LIB_PATH
    subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
                    os.path.join(ROCM, "include"), str(src), lib, f"-Wl,-rpath,{os.path.dirname(lib)}",
                    f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}", "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                    "-w", "-o", str(exe)], check=True)
    text = "\n".join(" ".join(map(str, s)) for s, _, _ in SHAPES)
    r = subprocess.run([str(exe)], input=text, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    got = r.stdout.split()
    assert len(got) == len(SHAPES)
    for (shape, fwd, dq), have in zip(SHAPES, got):
        assert have == f"{fwd}{dq}", f"{shape}: forward and dQ split {have}, expected {fwd}{dq}"
