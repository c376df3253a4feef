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

// A strip of n rows costs n + `extra` row steps (halo rows and start-up) and
// the chip holds `slots` strips at once: whole frames when they fill it, else
// the split (at least 4 rows) with the least of the longest strip's steps and
// all steps over the slots.  The grid has room for the largest frame's strips
// in every frame, so a split that would make it large is not taken.
//
// A further split only adds halo steps, so the search ends once all steps over
// the slots are the larger term: many frames are walked once (with 32-bit
// divisions: 2000 frames took 10 us of the host before every call).
inline CssPlan css_plan(const int32_t* frame_meta, int32_t n_frames, int64_t units, int32_t width, int32_t extra,
                        double slots) {
  auto parts_of = [](int32_t a, int32_t b) { return int32_t((uint32_t(a) + uint32_t(b) - 1) / uint32_t(b)); };
  int32_t max_rows = 1;
  for (int32_t f = 0; f < n_frames; ++f) max_rows = std::max(max_rows, frame_meta[3 * f + 1]);
  CssPlan plan{max_rows, 1};
  double best_cost = 0.0;
  for (int32_t parts = 1; parts <= 16; ++parts) {
    const int32_t seg = std::max(parts_of(max_rows, parts), 4);
    int64_t steps = 0, most = 1;
    for (int32_t f = 0; f < n_frames; ++f) {
      const int32_t rows = frame_meta[3 * f + 1];
      const int64_t n = parts_of(rows, seg), across = parts_of(frame_meta[3 * f + 2], width);
      steps += across * (rows + n * extra);
      most = std::max(most, n * across);
    }
    const double longest = std::min(seg, max_rows) + extra, shared = double(steps * units) / slots;
    const double cost = std::max(longest, shared);
    if (parts == 1 || (cost < best_cost && most * n_frames <= (int64_t(1) << 22))) {
      plan = CssPlan{seg, int32_t(most)};
      best_cost = cost;
    }
    if (seg == 4 || shared >= longest) break;
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
