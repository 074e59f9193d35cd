"""How the weight sides are cut (csrc/weight_shape.h), asked on the host."""
import os
import subprocess

import pytest

from paper_2410_23608_amd import build as spa_build

ROCM = os.path.dirname(os.path.dirname(spa_build.HIPCC))
CLANGXX = os.path.join(ROCM, "lib", "llvm", "bin", "clang++")
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "weight_shape.h"
int main() {
  int m, k, n, cfg, forced;
  while (std::scanf("%d %d %d %d %d", &m, &k, &n, &cfg, &forced) == 5) {
    const spa::WeightShape s = spa::weight_shape(m, k, n, cfg, forced);
    std::printf("%d %d %d %d\n", s.edge, s.splits, (int)s.fold, (int)spa::in_one_launch(m, k));
  }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    if not os.path.exists(CLANGXX):
        pytest.skip("needs ROCm's clang++")
    d = tmp_path_factory.mktemp("weight_shape")
    (d / "main.cpp").write_text(MAIN)
    cmd = [CLANGXX, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I",
           os.path.join(ROCM, "include"), "-I", spa_build.CSRC, str(d / "main.cpp"), "-o", str(d / "main")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def ask(calls):
        text = "\n".join(" ".join(str(v) for v in c) for c in calls)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]

    return ask


ROWS = [1, 98, 2048, 2049, 3136, 5096, 6272, 6800, 7840, 9408, 11000, 12544, 15680, 18816, 23999, 24001, 25088, 40000, 100000]
COLUMNS = [8, 64, 128, 192, 264, 384, 448, 512, 520, 640, 768, 896, 1024, 1536, 2048]


def _tiles(a, b, edge):
    return -(-a // edge) * -(-b // edge)


def _chunks_of_one_sum(m, c, n):
    """Chunks that fill the chip: 128 x 128 tiles two a unit and at least 256 rows each, or, from 2.4e10 multiplications of both sides of a
    block on, both sides' 256 x 256 tiles one a unit, at least 512 rows each, at most ten."""
    if 4.0 * m * c * c > 2.4e10:
        return max(1, min(256 // (_tiles(c, c, 256) + _tiles(3 * c, c, 256)), m // 512, 10))
    return 1 if m <= 2048 else max(1, min(512 // _tiles(n, c, 128), m // 256, 16))


@pytest.mark.parametrize("tiles", [0, 2, 8, 14])
def test_fewer_chunks_only_with_sums_apart(shapes, tiles):
    """A chunk that is longer than those that fill the chip sums every 256 rows apart, whatever tiles are forced; 256 x 256 tiles cannot."""
    calls = [(m, c, n, tiles, 0) for m in ROWS for c in COLUMNS for n in (c, 3 * c)]
    apart = 0
    for (m, c, n, *_), (edge, splits, fold, _) in zip(calls, shapes(calls)):
        assert fold or splits >= _chunks_of_one_sum(m, c, n), (m, c, n)
        assert not fold or edge == 128, (m, c, n)
        assert {2: 128, 8: 256}.get(tiles, edge) == edge
        apart += fold
    assert (apart > 100) == (tiles != 8)


def test_the_pass_and_the_kernels_draw_one_line(shapes):
    """BlockTrainPass forms the launch group where the weight sides have the chunks for it."""
    from paper_2410_23608_amd.pipeline import _one_launch
    calls = [(m, c, c, 0, 0) for c in COLUMNS for m in ROWS + [int(w // (c * c)) + d for w in (6e9, 7.3e9) for d in (0, 1)]
             if 0 < m < 2 ** 31]
    got = [s[3] for s in shapes(calls)]
    assert got == [int(_one_launch(m, c)) for m, c, *_ in calls] and {0, 1} == set(got)


def test_forced_chunks_are_one_sum_each(shapes):
    calls = [(m, c, 3 * c, 0, s) for m in ROWS for c in COLUMNS for s in (1, 7, 16)]
    assert all(got[1:3] == (c[4], 0) for c, got in zip(calls, shapes(calls)))
