"""The plan of a launch of large tiles (csrc/gemm_shape.h), asked on the host: which rows take which shape."""
import os
import subprocess

import pytest

from paper_2410_23608_amd import build as spa_build

ROCM = os.path.dirname(os.path.dirname(spa_build.HIPCC))
CLANGXX = os.path.join(ROCM, "lib", "llvm", "bin", "clang++")
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "gemm_shape.h"
int main(int c, char** v) {
  for (int i = 1; i + 4 < c; i += 5) {
    const int rows = std::atoi(v[i]), n = std::atoi(v[i + 1]), k = std::atoi(v[i + 2]), more = std::atoi(v[i + 3]), copy = std::atoi(v[i + 4]);
    const spa::LargePlan p = spa::large_plan(rows, n, more, spa::large_rule(n, k, copy != 0));
    std::printf("%d %d %d %d\n", (int)p.medium, p.wide_rows, p.rounds, p.rest);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not os.path.exists(CLANGXX):
        pytest.skip("needs ROCm's clang++")
    d = tmp_path_factory.mktemp("large_plan")
    (d / "main.cpp").write_text(MAIN)
    cmd = [CLANGXX, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I",
           os.path.join(ROCM, "include"), "-I", spa_build.CSRC, str(d / "main.cpp"), "-o", str(d / "main")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def ask(calls):
        out = subprocess.run([str(d / "main")] + [str(int(v)) for c in calls for v in c], capture_output=True, text=True, check=True)
        return [tuple(int(v) for v in line.split()) for line in out.stdout.splitlines()]

    return ask


def test_the_measured_launches(plan):
    """(rows, columns, contraction, rows to clear or copy, copied): the shapes that measured faster, as stated at the kernel and the rule."""
    medium, wide, narrow = (1, 0), lambda rows: (0, rows), (0, 0)
    sizes = {(11540, 768, 768, 0, 0): medium, (13500, 768, 768, 0, 0): narrow, (7526, 2304, 768, 0, 0): medium,
             (12544, 2304, 768, 0, 0): wide(7168), (15052, 2304, 768, 0, 0): narrow, (11540, 768, 2304, 11540, 0): medium,
             (12544, 768, 2304, 12544, 0): narrow, (13500, 768, 768, 13500, 1): wide(13500)}
    assert [p[:2] for p in plan(list(sizes))] == list(sizes.values())


def test_rows_are_whole_tiles_and_the_rounds_hold_them(plan):
    calls = [(rows, n, k, more, copy) for rows in (0, 1, 255, 256, 257, 4096, 4097, 12449, 16545, 65535, 1 << 20) for n in (8, 192, 200, 768, 2304, 8192)
             for k, more, copy in ((8, 0, 0), (768, 5000, 1), (4096, 1 << 30, 0))]
    for (rows, n, k, more, copy), (medium, wide, rounds, rest) in zip(calls, plan(calls)):
        assert 0 <= wide <= rows and (wide == rows or wide % 256 == 0), (rows, n)
        up = lambda a, b: (a + b - 1) // b
        first = up(rows, 192) * up(n, 192) if medium else up(wide, 256) * up(n, 256)
        assert up(first, 256) <= rounds, (rows, n)
        assert (wide, rest) == (0, 0) if medium else up(up(rows - wide, 256) * up(n, 192), 256) <= rest, (rows, n)


def test_the_shapes_of_the_two_shape_launch_are_two(plan):
    from test_gpu_gemm_mixed import SPLIT
    calls = [(T, n, k, more, copy) for cap, T, k, n in SPLIT for more, copy in ((0, 0), (cap - T, 1), (cap - T, 0))]
    got = plan(calls)
    assert all(not medium and 0 < wide < c[0] and rest > 0 for c, (medium, wide, _, rest) in zip(calls, got))
    assert {g[2:] for g in got} == {(1, 1), (1, 2), (2, 1)}
