"""Which path rotates a sector, by its size (svd_path in csrc/svd.h): the sizes that
tests/test_gpu_svd_paths.py runs are those of the path it names."""
import os
import subprocess

import pytest

REG, LDS, ROUNDS = 0, 1, 2
# one workgroup's LDS: at least 257 rows and X within 128 KB, so at most 63 columns
LDS_SHAPES = {
    "Vh in LDS, 64 lanes a pair": [(257, 2), (400, 32), (31, 260), (1500, 10)],
    "Vh in LDS, 32 lanes a pair": [(257, 33), (40, 300), (280, 48)],
    "X alone in LDS, 64 lanes a pair": [(500, 32), (2045, 8), (20, 810)],
    "X alone in LDS, 32 lanes a pair": [(257, 60), (50, 320), (260, 63)],
    "one column": [(300, 1), (1, 17000)],
}
REG_SHAPES = [(30, 40), (256, 126), (110, 130), (208, 205), (5, 1)]
ROUNDS_SHAPES = [(257, 64), (300, 100), (209, 209)]


def test_sizes_and_paths(tmp_path):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src = tmp_path / "path.cpp"
    src.write_text('#include "svd.h"\n#include <cstdio>\n#include <cstdlib>\n'
                   "int main(int c, char** v) { for (int i = 1; i + 1 < c; i += 2)\n"
                   'std::printf("%d ", bst::svd_path(std::atoi(v[i]), std::atoi(v[i + 1]))); }\n')
    exe = tmp_path / "path"
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(root, "paper_2401_01921_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    if r.returncode != 0 and "hip_runtime.h" in r.stderr:
        pytest.skip("no HIP headers for the host compiler")
    assert r.returncode == 0, r.stderr

    def paths(shapes):
        out = subprocess.run([str(exe)] + [str(x) for s in shapes for x in s], capture_output=True, text=True)
        return [int(x) for x in out.stdout.split()]

    for name, shapes in LDS_SHAPES.items():
        assert paths(shapes) == [LDS] * len(shapes), name
        for a, b in shapes:
            p, n = max(a, b), min(a, b)
            assert name.startswith("Vh") == (n > 1 and p * n + n * n <= 16384), (a, b)
            assert "64 lanes" not in name or n <= 32
            assert "32 lanes" not in name or 32 < n
    assert paths(REG_SHAPES) == [REG] * len(REG_SHAPES)
    assert paths(ROUNDS_SHAPES) == [ROUNDS] * len(ROUNDS_SHAPES)
