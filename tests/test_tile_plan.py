"""The tile plan of the bf16 contractions (host code, compiled here): the shapes of the GPU test of tiles take the tiles,
ring depths and splits that it names, and every plan is one that the kernels are built and correct for."""
import os
import random
import shutil
import subprocess

import pytest

from tests.test_gpu_gemm_tiles import SHAPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = r"""
#include <cstdio>
#include "tile_plan.hpp"
int main() {
  int M, N, K, conv, gelu, ln;
  unsigned long scratch;
  while (std::scanf("%d %d %d %d %d %d %lu", &M, &N, &K, &conv, &gelu, &ln, &scratch) == 7) {
    const tp::k::TilePlan p = tp::k::plan_tiles({M, N, K, conv != 0, gelu != 0, ln != 0}, scratch);
    std::printf("%d %d %d %d\n", p.bn, p.bm, p.ring, p.splits);
  }
}
"""
SCRATCH = 32 << 20
# tiles (features x rows) and ring depths that exist
BUILT = {(32, 32): {4, 6}, (64, 32): {5}, (64, 64): {2, 4}, (128, 128): {2, 3}, (256, 128): {3}, (256, 256): {2}}


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run([cxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2306_03622_amd", "csrc", "kernels"),
                    str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)

    def run(shapes):          # (M, N, K, conv, gelu, ln, scratch)
        text = "\n".join(" ".join(str(int(v)) for v in s) for s in shapes)
        out = subprocess.run([str(d / "driver")], input=text, capture_output=True, text=True, check=True).stdout
        plans = [tuple(int(v) for v in line.split()) for line in out.splitlines()]
        assert len(plans) == len(shapes)
        return plans

    return run


def test_the_gpu_test_covers_the_tiles_it_names(plan):
    got = plan([(batch, width, width, 0, 0, 0, SCRATCH) for width, batch, _ in SHAPES])
    for (width, batch, want), p in zip(SHAPES, got):
        assert p == want, (width, batch, want, p)
    named = {p[:3] for p in got}
    assert named == {(bn, bm, r) for (bn, bm), rings in BUILT.items() for r in rings}
    # row-major (ragged) and blocked weights each
    for packed in (False, True):
        assert {p[:3] for (w, _, _), p in zip(SHAPES, got) if (w % 128 == 0) == packed} == named


def test_deep_contractions_are_split_with_and_without_a_layernorm(plan):
    # FFN2 of an encoder layer: few tiles and a deep k; shallower ones and many tiles stay whole
    want = [((128, 768, 3072), (32, 32, 6, 2)), ((64, 64, 16384), (32, 32, 6, 28)), ((128, 512, 4096), (32, 32, 6, 4)),
            ((128, 512, 2048), (32, 32, 6, 1)), ((512, 256, 6144), (64, 32, 5, 7)), ((512, 256, 3072), (32, 32, 6, 1)),
            ((256, 1024, 16384), (64, 32, 5, 3)), ((1024, 768, 3072), (64, 64, 4, 1))]
    assert plan([(m, n, k, 0, 0, 1, SCRATCH) for (m, n, k), _ in want]) == [p for _, p in want]
    assert all(p[3] == 1 for p in plan([(m, n, k, 0, 0, 1, 0) for (m, n, k), _ in want]))        # no scratch
    assert plan([(64, 64, 16384, 0, 0, 0, SCRATCH)]) == [(32, 32, 6, 28)]


def test_every_plan_is_built_and_in_bounds(plan):
    rng = random.Random(3)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    shapes = []
    for _ in range(20000):
        conv = rng.random() < 0.3
        n = log(1, 65536) if rng.random() < 0.2 else 8 * log(1, 8192)
        k = 64 * log(1, 128) if conv else 8 * log(1, 2048)
        ln = not conv and n % 64 == 0 and n <= 1024
        shapes.append((log(33, 4 << 20), n, k, conv, rng.random() < 0.5, ln, rng.choice([0, 1 << 16, SCRATCH])))
    for (m, n, k, conv, gelu, ln, scratch), (bn, bm, ring, z) in zip(shapes, plan(shapes)):
        s = (m, n, k, conv, gelu, ln, scratch, bn, bm, ring, z)
        assert ring in BUILT[bn, bm], s
        assert 1 <= z <= -(-k // 64) and (z == 1 or z * m * n * 4 <= scratch), s
        if n % 8:
            assert (bn, bm, ring, z) == (32, 32, 4, 1), s
        elif m * n * 2 >= 1 << 31:        # tiles whose epilogue has 64-bit offsets
            assert bn == 256 and z == 1, s
