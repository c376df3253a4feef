"""CPU tests of the saliency kernels' strip arithmetic (csrc/css_strips.h, the
code that the plan and the kernels compile), built with the host compiler: over
a batch's grids, the strips of every frame cover each of its cells exactly once
and every strip index that the grid holds beyond them is recognised as surplus."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_00188_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")

# argv: units width extra slots per_simd, then rows cols of each frame.  Prints
# "seg_rows strips"; fails on the first strip out of place.
PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "css_strips.h"
int main(int argc, char** argv) {
  const int64_t units = atoll(argv[1]);
  const int32_t width = atoi(argv[2]), extra = atoi(argv[3]);
  const double slots = atof(argv[4]);
  const int32_t per_simd = atoi(argv[5]);
  std::vector<int32_t> meta;
  for (int i = 6; i + 1 < argc; i += 2) meta.insert(meta.end(), {0, atoi(argv[i]), atoi(argv[i + 1])});
  const int32_t n = int32_t(meta.size() / 3);
  const stlite::CssPlan plan = stlite::css_plan(meta.data(), n, units, width, extra, slots, per_simd);
  for (int32_t f = 0; f < n; ++f) {
    const int32_t R = meta[3 * f + 1], C = meta[3 * f + 2];
    int32_t row = 0, col = 0;  // where the next strip has to start
    for (int32_t s = 0; s < plan.strips; ++s) {
      stlite::CssStrip at{};
      const bool used = stlite::css_strip(s, R, C, width, plan.seg_rows, &at);
      if (used != (row < R)) { printf("frame %d strip %d: used %d at row %d\n", f, s, int(used), at.row_begin); return 1; }
      if (!used) continue;
      const int32_t end = row + plan.seg_rows < R ? row + plan.seg_rows : R;
      if (at.row_begin != row || at.row_end != end || at.col != col) { printf("frame %d strip %d: rows %d .. %d, column %d\n", f, s, at.row_begin, at.row_end, at.col); return 1; }
      col += width;
      if (col >= C) { col = 0; row = end; }
    }
    if (row < R) { printf("frame %d: rows from %d have no strip\n", f, row); return 1; }
  }
  printf("%d %d\n", plan.seg_rows, plan.strips);
  return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("css_strips")
    src, exe = str(d / "strips.cpp"), str(d / "strips")
    with open(src, "w") as f:
        f.write(PROGRAM)
    # the kernels' products wrap in hardware: -fwrapv does the same here
    subprocess.run(["g++", "-std=c++17", "-O2", "-fwrapv", "-Wall", f"-I{CSRC}", src, "-o", exe], check=True)

    def run(units, width, extra, slots, per_simd, frames):
        args = [str(x) for x in (units, width, extra, slots, per_simd)] + [str(x) for rc in frames for x in rc]
        r = subprocess.run([exe, *args], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout
        return tuple(int(x) for x in r.stdout.split())
    return run


WALKS = [(14, 4, 2560.0, 0), (16, 8, 2048.0, 2), (16, 12, 1024.0, 1)]  # 3 x 3, 5 x 5, 9 x 9


@pytest.mark.parametrize("walk", WALKS, ids=["3x3", "5x5", "9x9"])
@pytest.mark.parametrize("frames,units", [
    ([(36, 80)], 112), ([(36, 80)] * 48, 112), ([(16, 16)] * 3, 4),
    ([(1, 1), (1, 40), (33, 1), (3, 17), (9, 14), (40, 15), (5, 29), (4, 4)], 4),
    # very tall frames beside very wide ones, up to 2^22 cells each: strips of
    # the wide frame times rows of the tall one pass 2^31
    ([(4194304, 1), (1, 120000)], 1), ([(200000, 1), (1, 2000000)], 112), ([(4194304, 1), (1, 4194304)], 1),
    ([(7200, 1), (1, 100000)], 1), ([(2048, 2048), (1, 4194304)], 4),
])
def test_strips_cover_every_frame_once(plan, walk, frames, units):
    seg_rows, strips = plan(units, *walk, frames)
    assert 4 <= seg_rows or seg_rows >= max(r for r, _ in frames)
    assert strips >= 1


def test_long_frames_stay_whole_where_they_fill_the_chip(plan):
    """One screen in 112 units is cut into segments, 48 of them are not."""
    assert plan(112, *WALKS[0], [(36, 80)])[0] < 36
    assert plan(112, *WALKS[0], [(36, 80)] * 48)[0] == 36


def _search(units, width, extra, slots, per_simd, frames):
    """The plan by trying every split."""
    top, best = max([r for r, _ in frames]), None
    pair = 1.3 if per_simd == 2 else 1.0
    for parts in range(1, 17):
        seg = max(-(-top // parts), 4)
        steps = sum(-(-c // width) * (r + -(-r // seg) * extra) for r, c in frames)
        strips = sum(-(-c // width) * -(-r // seg) for r, c in frames)
        most = max(-(-r // seg) * -(-c // width) for r, c in frames)
        longest, on_simd = float(min(seg, top) + extra), -(-strips * units // 1024)
        if per_simd and on_simd <= 4 * per_simd:
            cost = longest * (float(on_simd // per_simd) * pair + on_simd % per_simd)
        else:
            cost = max(longest, steps * units / slots) * pair
        if best is None or (cost < best[0] and most * len(frames) <= 1 << 22):
            best = (cost, seg, most)
        if seg == 4:
            break
    return best[1:]


def test_plan_is_the_best_split(plan):
    """The search ends early; its plan is the full search's."""
    rng = random.Random(7)
    for i in range(150):
        n = rng.choice([1, 2, 3, 10, 48, 300])
        top = rng.choice([3, 40, 400, 60000])
        frames = [(rng.randint(1, top), rng.randint(1, rng.choice([4, 90, 900]))) for _ in range(n)]
        units, walk = rng.choice([1, 4, 24, 112]), rng.choice(WALKS)
        assert plan(units, *walk, frames) == _search(units, *walk, frames), (units, walk, n, top)


def test_plans_of_the_edge_grids(plan):
    """What test_gpu_css_gate.py's edge tests run: 4-row strips in 4 units and
    in one layer, whole frames in 400."""
    from tests.test_gpu_css_gate import EDGES
    frames = EDGES + [(6, 31)]
    assert [plan(u, *WALKS[0], frames)[0] for u in (1, 4, 400)] == [4, 4, 22]


def test_wide_walks_fill_whole_rounds(plan):
    """One strip per SIMD at 7 x 7 and 9 x 9: three frames of 36 x 80 in 8 units
    are cut into one round of strips, not one and a half."""
    for frames, units in (([(36, 80)] * 3, 8), ([(36, 80)], 24), ([(16, 16)] * 48, 8)):
        for extra in (10, 12):
            seg, _ = plan(units, 16, extra, 1024.0, 1, frames)
            assert units * sum(-(-c // 16) * -(-r // seg) for r, c in frames) <= 1024
