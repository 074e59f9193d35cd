"""The rules that choose the tiles of the projection GEMMs, asked on the host (csrc/gemm_shape.h compiled alone)."""
import os
import subprocess

import pytest

from paper_2410_23608_amd import build as spa_build

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.path.dirname(os.path.dirname(spa_build.HIPCC))
CLANGXX = os.path.join(ROCM, "lib", "llvm", "bin", "clang++")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """(m_cap, counted, columns, contraction) -> (large, 192 x 192 rather than 256 x 256) for a list of such."""
    if not os.path.exists(CLANGXX):
        pytest.skip("needs ROCm's clang++")
    exe = str(tmp_path_factory.mktemp("tile_rule") / "driver")
    cmd = [CLANGXX, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", spa_build.CSRC,
           os.path.join(HERE, "tile_rule_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def ask(calls):
        out = subprocess.run([exe] + [str(int(v)) for c in calls for v in c], capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) != 0 for v in line.split()) for line in out.splitlines()]

    return ask


@pytest.mark.parametrize("ncols,kc", [(8, 8), (64, 64), (384, 384), (768, 768), (2304, 768), (3072, 1024), (768, 2304)])
def test_few_rows_take_small_tiles(rules, ncols, kc):
    """Up to 128 rows are one row of tiles of any shape, fewer of the large ones than the chip has units: small tiles, also
    for a capacity of one row of which half are expected live."""
    calls = [(m, counted, ncols, kc) for m in (1, 2, 3, 64, 128) for counted in (0, 1)]
    assert not any(large for large, _ in rules(calls))


def test_the_measured_sizes(rules):
    """The sizes stated at the rule, as live rows (columns, contraction): where each side measured faster, and the tie."""
    sizes = {(6272, 2304, 768): True, (6272, 768, 768): False, (12544, 768, 768): True, (12544, 1536, 512): False,
             (12544, 768, 2304): True, (9408, 2304, 768): True}
    assert [large for large, _ in rules([(m, 0, n, k) for m, n, k in sizes])] == list(sizes.values())
    assert [large for large, _ in rules([(2 * m, 1, n, k) for m, n, k in sizes])] == list(sizes.values())
    # rounds of the large tiles, as measured at the kernel: 192 x 192 | 256 x 256
    rounds = {(11540, 768): True, (15052, 768): False, (7526, 2304): True, (11540, 2304): False, (12544, 2304): False, (15052, 2304): True}
    assert [medium for _, medium in rules([(m, 0, n, 768) for m, n in rounds])] == list(rounds.values())
