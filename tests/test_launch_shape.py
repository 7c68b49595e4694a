"""The launch-shape rule (csrc/shape.h) on the host: no block is counted that a
CU does not hold, and the shape is the best of those left."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2111_04867_amd", "csrc")
LDS, STEP = 160 * 1024, 1280
MAIN = r"""
#include <cstdio>
#include "shape.h"
int main() {
  long shared, wave, n;
  int max_waves, per_simd, spread;
  while (scanf("%ld %ld %d %d %ld %d", &shared, &wave, &max_waves, &per_simd, &n, &spread) == 6) {
    const taccl::LaunchShape s = taccl::resident_shape(shared, wave, max_waves, per_simd);
    printf("%d %d %d\n", s.waves, s.per_cu, taccl::wave_grid(s, n, 256, spread != 0));
  }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ is not installed")
    d = tmp_path_factory.mktemp("shape")
    src, exe = str(d / "main.cpp"), str(d / "shape")
    with open(src, "w") as f:
        f.write(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I" + CSRC, src, "-o", exe], check=True)

    def run(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, ln.split())) for ln in out.splitlines()]
    return run


def held(waves, bytes_, per_simd):
    """Blocks a CU holds: LDS in steps, and ceil(waves / 4) wavefronts of a
    block on some SIMD."""
    by_lds = LDS // (-(-bytes_ // STEP) * STEP)
    return min(by_lds, 4 * per_simd // waves if waves < 4 else per_simd // -(-waves // 4))


def test_counted_blocks_are_resident(shapes):
    rows = [(s, w, m, r, 5000, 0) for s in (544, 4976, 20032, 26304, 62000, 131000)
            for w in (720, 4256, 5888, 10160, 11168, 27000) for m in (8, 12)
            for r in (2, 3, 4, 5, 8)]
    for (s, w, m, r, _, _), (waves, per_cu, grid) in zip(rows, shapes(rows)):
        if s + w > LDS:
            assert (waves, per_cu) == (1, 1)
            continue
        assert per_cu <= held(waves, s + waves * w, r)
        assert waves * per_cu == max(k * held(k, s + k * w, r) for k in range(1, m + 1)
                                     if s + k * w <= LDS)
        assert grid == min(-(-5000 // waves), 256 * per_cu)


# shared and per-wavefront bytes of plans whose last block was counted but not
# resident: three blocks of 54528 bytes are 163584 of 163840 but 165120 in
# steps; two blocks of 10 wavefronts, of 5 per SIMD, are 3 + 3 on some
@pytest.mark.parametrize("shared,wave,per_simd,shape",
                         [(13888, 10160, 3, (12, 1)), (20032, 5888, 5, (8, 2)),
                          (26304, 11168, 3, (12, 1)), (9920, 11168, 3, (12, 1))])
def test_shapes_of_known_plans(shapes, shared, wave, per_simd, shape):
    assert shapes([(shared, wave, 12, per_simd, 1, 0)])[0][:2] == shape


def test_grids(shapes):
    """Blocks hold their wavefronts' candidates, or one each where a small
    batch is dealt out; never more than are resident, and at least one."""
    rows = [(26304, 11168, 12, 3, n, spread) for n in (1, 11, 12, 13, 256, 257, 3072, 100000)
            for spread in (0, 1)]
    for (_, _, _, _, n, spread), (waves, per_cu, grid) in zip(rows, shapes(rows)):
        assert (waves, per_cu) == (12, 1)
        assert grid == min(256, n if spread else -(-n // 12))
