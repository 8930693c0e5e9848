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
  int M, N, K, conv, gelu, ln, far;
  unsigned long scratch;
  while (std::scanf("%d", &M) == 1 && M > 0) {
    if (std::scanf("%d %d %d %d %d %d %lu", &N, &K, &conv, &gelu, &ln, &far, &scratch) != 7) return 1;
    const tp::k::TilePlan p = tp::k::plan_tiles({M, N, K, conv != 0, gelu != 0, ln != 0, far != 0}, scratch);
    std::printf("%d %d %d %d\n", p.bn, p.bm, p.ring, p.splits);
  }
  int tn, tm, splits;                       // after the shapes: grids, whose tiles are listed in workgroup order
  while (std::scanf("%d %d %d %d", &tn, &tm, &splits, &far) == 4)
    for (int id = 0; id < tn * tm * splits; ++id) {
      const tp::k::TileAt t = far ? tp::k::tile_at<true>(id, tn * tm * splits, tn, tm, splits)
                                  : tp::k::tile_at<false>(id, tn * tm * splits, tn, tm, splits);
      std::printf("%d %d %d\n", t.tx, t.ty, t.z);
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

    def run(shapes, grids=()):          # (M, N, K, conv, gelu, ln, far, scratch); (tn, tm, splits, far)
        text = "\n".join(" ".join(str(int(v)) for v in s) for s in [*shapes, (0,), *grids])
        out = subprocess.run([str(d / "driver")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]

    return run


def test_the_gpu_test_covers_the_tiles_it_names(plan):
    got = plan([(batch, width, width, 0, 0, 0, 0, SCRATCH) for width, batch, _ in SHAPES])
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
    assert plan([(m, n, k, 0, 0, 1, 0, SCRATCH) for (m, n, k), _ in want]) == [p for _, p in want]
    assert all(p[3] == 1 for p in plan([(m, n, k, 0, 0, 1, 0, 0) for (m, n, k), _ in want]))        # no scratch
    assert plan([(64, 64, 16384, 0, 0, 0, 0, SCRATCH)]) == [(32, 32, 6, 28)]


def test_every_plan_is_built_and_in_bounds(plan):
    rng = random.Random(3)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    shapes = []
    for _ in range(20000):
        conv = rng.random() < 0.3
        n = log(1, 65536) if rng.random() < 0.2 else 8 * log(1, 8192)
        k = 64 * log(1, 128) if conv else 8 * log(1, 2048)
        ln = not conv and n % 64 == 0 and n <= 1024
        shapes.append((log(33, 4 << 20), n, k, conv, rng.random() < 0.5, ln, rng.random() < 0.3,
                       rng.choice([0, 1 << 16, SCRATCH])))
    plans, near = plan(shapes), plan([(*s[:6], 0, s[7]) for s in shapes])
    for (m, n, k, conv, gelu, ln, far, scratch), (bn, bm, ring, z), other in zip(shapes, plans, near):
        s = (m, n, k, conv, gelu, ln, far, scratch, bn, bm, ring, z)
        assert z == other[3], s           # the k splits, and so the order of the sums, do not depend on where weights lie
        assert ring in BUILT[bn, bm], s
        assert 1 <= z <= -(-k // 64) and (z == 1 or z * m * n * 4 <= scratch), s
        if n % 8:
            assert (bn, bm, ring, z) == (32, 32, 4, 1), s
        elif m * n * 2 >= 1 << 31:        # tiles whose epilogue has 64-bit offsets
            assert bn == 256 and z == 1, s


@pytest.mark.parametrize("far", [0, 1])
def test_every_tile_is_computed_once(plan, far):
    grids = [(1, 1, 1), (1, 7, 1), (3, 5, 1), (8, 32, 1), (16, 33, 4), (5, 1, 1), (12, 130, 1), (7, 9, 3)]
    got = plan([], [(*g, far) for g in grids])
    for tn, tm, splits in grids:
        n = tn * tm * splits
        tiles, got = got[:n], got[n:]
        assert sorted(tiles) == sorted((x, y, z) for x in range(tn) for y in range(tm) for z in range(splits))
    assert not got


@pytest.mark.parametrize("tn,tm,splits", [(8, 32, 1), (16, 10, 1), (32, 63, 1), (24, 64, 1), (9, 25, 1), (8, 13, 4)])
def test_weights_in_host_memory_are_read_by_few_xcds(plan, tn, tm, splits):
    # workgroup i runs on XCD i % 8: a column of tiles (one k split of one block of weights) lies on one XCD, or on
    # two where an eighth of the tiles ends inside it, instead of on all
    readers = {}
    for i, (x, _, z) in enumerate(plan([], [(tn, tm, splits, 1)])):
        readers.setdefault((x, z), set()).add(i % 8)
    assert sum(len(r) for r in readers.values()) <= tn * splits + 7
