"""The host rules that shape launches, compiled and run on the CPU."""
import heapq
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_01800_amd", "csrc")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")

MAIN = r"""
#include <cstdio>
#include "launch_plan.hpp"
int main() {
  long long cus, n;
  while (std::scanf("%lld %lld", &cus, &n) == 2) {
    if (n == 0) {
      long long nx, ny, nb;
      if (std::scanf("%lld %lld %lld", &nx, &ny, &nb) != 3) return 1;
      std::printf("%d\n", (int)ppe::mg_two_launches(nx, ny, nb, cus));
      continue;
    }
    std::vector<ppe::ConvpPart> parts(n);
    for (auto& p : parts) {
      long long t, c, h;
      if (std::scanf("%lld %lld %lld", &t, &c, &h) != 3) return 1;
      p = {t, c, h};
    }
    const ppe::ConvpRuns r = ppe::convp_runs(parts, cus);
    std::printf("%lld %lld %lld %d\n", (long long)r.run, (long long)r.wgs, (long long)r.span, (int)r.fills);
  }
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(d / "plan"), str(d / "plan.cpp")], check=True)
    return str(d / "plan")


def run_plans(exe, plans):
    text = "".join(f"{cus} {len(parts)} " + " ".join(f"{t} {c} {h}" for t, c, h in parts) + "\n"
                   for cus, parts in plans)
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.split("\n")
    return [tuple(int(v) for v in line.split()) for line in out if line]


def image(nx, ny, copies):
    """Tiles of 16 x 32 pixels, workgroup columns, and tile halves with rows of the image."""
    w = -(-nx // 16)
    return w * -(-ny // 32), copies, w * -(-ny // 16)


def work_off(parts, run, cus):
    """Tiles and workgroups on the unit that ends last, workgroups started in order."""
    free = [0] * cus
    for _ in range(max(c for _, c, _ in parts)):
        for t, c, _ in parts:
            for k in range(0, t, run):
                heapq.heapreplace(free, free[0] + min(run, t - k) + 1)
    return max(free)


MIXED = [(896, 192), (256, 320), (256, 896), (960, 640), (128, 192), (384, 512), (704, 576), (320, 256), (768, 832)]


@pytest.mark.parametrize("parts", [
    [image(256, 256, 24)], [image(256, 160, 48)], [image(256, 256, 6)], [image(128, 128, 24)],
    [image(1024, 1024, 1)], [image(1000, 360, 2)], [image(16, 16, 300)], [image(32, 32, 300)], [image(64, 64, 150)],
    [image(96, 16, 1)], [image(256, 256, 33)], [image(nx, ny, 1) for nx, ny in MIXED],
    [image(nx // 2, ny // 2, 1) for nx, ny in MIXED], [image(nx // 4, ny // 4, 2) for nx, ny in MIXED],
    [image(nx // 8, ny // 8, 4) for nx, ny in MIXED],
])
@pytest.mark.parametrize("cus", [256, 64])
def test_runs_of_tiles_keep_the_units_busy(exe, parts, cus):
    """The chosen run against every other one, worked off workgroup by workgroup: within
    a tile and a tenth of the best."""
    (run, wgs, span, fills), = run_plans(exe, [(cus, parts)])
    assert wgs == sum(c * -(-t // run) for t, c, _ in parts)
    best = min(work_off(parts, r, cus) for r in range(1, max(t for t, _, _ in parts) + 1))
    assert work_off(parts, run, cus) <= 1.1 * best + 1
    if fills:
        assert 4 * sum(t * c for t, c, _ in parts) >= 3 * cus and sum(h * c for _, c, h in parts) >= cus * span / 2


@pytest.mark.parametrize("nx,ny,images", [(256, 256, 24), (256, 160, 48), (256, 256, 6), (512, 512, 3)])
def test_batches_take_one_round_of_workgroups(exe, nx, ny, images):
    """Batches whose tiles over the compute units, taken as the run, start more
    workgroups than there are units, whole runs among the late ones."""
    tiles = image(nx, ny, 1)[0]
    even = -(-tiles * images // 256)
    assert images * -(-tiles // even) > 256
    (run, wgs, span, fills), = run_plans(exe, [(256, [image(nx, ny, images)])])
    assert wgs <= 256 and span == run and fills


@pytest.mark.parametrize("nx,ny,images,want", [
    (16, 16, 600, 0),  # three rounds of half-empty tiles
    (16, 16, 200, 1),  # one round: nothing would run beside them
    (32, 32, 600, 1),  # full tiles
])
def test_half_empty_tiles(exe, nx, ny, images, want):
    (_, _, _, fills), = run_plans(exe, [(256, [image(nx, ny, images)])])
    assert fills == want


@pytest.mark.parametrize("nx,ny,nb,want", [
    (128, 128, 1, 1), (8, 8, 32, 1), (32, 128, 8, 1),      # one round of the first launch
    (8, 8, 64, 0), (16, 16, 128, 0), (32, 32, 64, 0), (128, 32, 8, 0), (64, 64, 8, 0), (96, 32, 8, 0),
    (128, 128, 4, 1), (112, 96, 4, 1), (128, 64, 4, 0),    # two rounds
    (112, 128, 6, 1), (96, 96, 8, 0), (128, 128, 16, 1),   # three and more
])
def test_coarsest_solve_of_many_right_hand_sides(exe, nx, ny, nb, want):
    out = subprocess.run([exe], input=f"256 0 {nx} {ny} {nb}\n", check=True, capture_output=True, text=True).stdout
    assert int(out) == want
