// How the saliency kernels cut frames into strips: a strip is `width` output
// columns of `seg_rows` frame rows, and one wave walks it.  The host plan and
// the kernels' index arithmetic, with nothing of HIP in it.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace stlite {

// Strips of a saliency call over frames (offset, rows, cols) x n_frames: a
// strip's rows, and the largest number of strips in a frame.
struct CssPlan {
  int32_t seg_rows, strips;
};

// The chip's SIMDs, and what two strips that share one cost against one alone
// (5 x 5).
constexpr int64_t kCssSimds = 1024;
constexpr double kCssPair = 1.3;

// A strip of n rows costs n + `extra` row steps (halo rows and start-up), and
// the split (whole frames, or at least 4 rows) with the least cost is taken.
// Bound by the memory (per_simd 0, the 3 x 3 walk): the longest strip's steps, or
// all steps over the `slots` strips that the chip holds at once.  Bound by
// each SIMD's issue (per_simd strips at once, the k x k walks): while there are
// few rounds of strips, their number times the longest strip; else the same as
// above.  Without the rounds, 7 x 7 and 9 x 9 were cut into one and a half: 8
// units x 3 frames of 36 x 80 took 25.5 and 34.5 us, in one round 15.1 and 19.7;
// over 44 layouts the split's distance from the best one is 1 % (geometric
// mean) at 7 x 7 and 9 x 9, 1.5 % at 5 x 5, and was 8 % and 7 %.
// The grid has room for the largest frame's strips in every frame, so a split
// that would make it large is not taken.
//
// A further split only adds halo steps, so the search ends once all steps over
// the slots are the larger term: many frames are walked once (with 32-bit
// divisions: 2000 frames took 10 us of the host before every call).
inline CssPlan css_plan(const int32_t* frame_meta, int32_t n_frames, int64_t units, int32_t width, int32_t extra,
                        double slots, int32_t per_simd) {
  auto parts_of = [](int32_t a, int32_t b) { return int32_t((uint32_t(a) + uint32_t(b) - 1) / uint32_t(b)); };
  int32_t max_rows = 1;
  for (int32_t f = 0; f < n_frames; ++f) max_rows = std::max(max_rows, frame_meta[3 * f + 1]);
  CssPlan plan{max_rows, 1};
  const double shared_step = per_simd == 2 ? kCssPair : 1.0;  // a step with every slot of a SIMD taken
  double best_cost = 0.0;
  for (int32_t parts = 1; parts <= 16; ++parts) {
    const int32_t seg = std::max(parts_of(max_rows, parts), 4);
    int64_t steps = 0, strips = 0, most = 1;
    for (int32_t f = 0; f < n_frames; ++f) {
      const int32_t rows = frame_meta[3 * f + 1];
      const int64_t n = parts_of(rows, seg), across = parts_of(frame_meta[3 * f + 2], width);
      steps += across * (rows + n * extra);
      strips += across * n;
      most = std::max(most, n * across);
    }
    const double longest = std::min(seg, max_rows) + extra, shared = double(steps * units) / slots;
    const int64_t on_simd = (strips * units + kCssSimds - 1) / kCssSimds;
    const bool rounds = per_simd > 0 && on_simd <= 4 * per_simd;
    const double cost = rounds ? longest * (double(on_simd / per_simd) * shared_step + double(on_simd % per_simd))
                               : std::max(longest, shared) * shared_step;
    if (parts == 1 || (cost < best_cost && most * n_frames <= (int64_t(1) << 22))) {
      plan = CssPlan{seg, int32_t(most)};
      best_cost = cost;
    }
    if (seg == 4 || (!rounds && shared >= longest)) break;
  }
  return plan;
}

// Strip `strip` of a frame of R x C: its output rows row_begin .. row_end - 1
// and first column.  False past the frame's last strip (the grid gives every
// frame the largest one's number of strips, so one frame's surplus times
// another's height can pass 2^31: the product is taken in 64 bits).
struct CssStrip {
  int32_t row_begin, row_end, col;
};
constexpr bool css_strip(int32_t strip, int32_t R, int32_t C, int32_t width, int32_t seg_rows, CssStrip* out) {
  const int32_t across = (C + width - 1) / width;
  const int32_t seg = strip / across;
  const int64_t row = int64_t(seg) * seg_rows;
  if (row >= R) return false;
  out->row_begin = int32_t(row);
  out->row_end = out->row_begin + seg_rows < R ? out->row_begin + seg_rows : R;
  out->col = (strip - seg * across) * width;
  return true;
}

}  // namespace stlite
