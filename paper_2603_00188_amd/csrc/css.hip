// Component-centric Spatial Saliency (Eq. css_calc of the paper):
//   H_{u,v} = mean over the in-grid Moore neighbours n of cos(h_{u,v}, h_n),
//   Phi = 1 - H  (0 when a frame is 1x1; 0 on text tokens).
//
// Text tokens get Phi = 0 from work-groups at the end of the same grid.
//
// One wave sweeps a vertical strip of a frame row by row.  A strip is 16
// loaded columns: 14 output columns plus one halo column on each side.  Four
// lanes share a cell, each holding 32 of the 128 dimensions, so a dot product
// is 16 v_dot2 per lane and a two-step quad reduction.
//
// Each unordered neighbour pair is evaluated once, when its lower (or eastern)
// row arrives: a cell's E (r, c+1) with its own row, its S (r+1, c), SE (r+1,
// c+1) and SW (r+1, c-1) with the next one.  Row r's mean combines its own
// forward cosines, its west neighbour's E, and the previous row's S / SE / SW
// carried in registers.  Only the row that arrives is read from LDS (a cell's
// own, east and west key); the row above stays in registers.
//
// Rows stream into an LDS ring by direct memory->LDS DMA, three rows ahead of
// the row being combined, so every key is read from HBM once per strip.  The
// strips of one frame are given to work-groups that land on the same XCD,
// where the halo columns hit the shared L2.  Frames are cut into row segments
// where whole ones would leave the chip idle.
//
// With the TSG gate given (GATED), a token whose gate is 0 gets Phi = 0 (its
// saliency is multiplied away by M = 0 in Eq. modal_scoring).  Each lane's
// gate byte is loaded with its row's DMA, so the loads complete in the same
// order as the ring rows.
//
// Over the concatenated key space (H > 1 heads, one Phi per layer) a row is H
// ring items, one per head; the five dot products are summed over the heads
// before the norms are applied.
//
// Bound by HBM where the grid fills the chip (112 units x 48 frames of 36 x 80:
// 774 us, 5.2 TB/s of keys, 785 with a gate), by the length of a strip where it does not: one
// such frame took 33.7 us as whole strips and takes 22.8 in segments, three
// 16 x 16 frames in 4 units 15.2 and 6.8.  Concatenated over 4 heads, 48 frames
// took 2667 us on the matrix cores with each wave loading its own neighbour
// rows, and take 762 here.
//
// The neighbourhood-size ablation widens the window to k x k, k = 2 KR + 1 in
// {5, 7, 9} (css_wide_kernel): H = mean over the in-grid cells of the square
// other than the centre.  There the cosines form a small dense contraction,
// which runs on the matrix cores: a wave walks a strip of 16 output columns
// downwards with the keys of the 2 KR + 1 output rows around it in registers
// (A operands).  Each neighbour row's 16 + 2 KR columns (two 16-key B blocks)
// are multiplied with every output row within KR of it; a per-lane mask keeps
// the products with |dc| <= KR, scales them by the neighbour's inverse norm
// and adds them in the accumulator lanes, and one 16-lane reduction per output
// finishes the sum.  Halo columns shared by neighbouring strips are re-read
// through L2 (the strips of one frame go to one XCD).
#include "css_strips.h"
#include "stlite_internal.h"
#include "tile_lds.h"

namespace stlite {
namespace {

constexpr int kStripCells = 16;  // loaded columns per strip (one per lane quad)
constexpr int kStripOut = kCssStripOut;  // output columns per strip
constexpr int kRowElems = kStripCells * kHeadDim;
constexpr int kRowLoads = kStripCells * kHeadDim * 2 / (64 * 16);  // wave-loads of 16 B per lane: 4
constexpr int kRing = 4;                                           // ring slots, one (row, head) each

// The 16-byte chunk ch (dims 8ch .. 8ch+7) of loaded cell g sits at slot
// ch ^ 4 (g & 1): lanes 0..7 of a b128 read then cover all 32 banks.
__device__ inline int chunk_slot(int g, int ch) { return ch ^ ((g & 1) << 2); }

// DMA of one strip row (16 cells, column-clamped) into `dst`.
__device__ inline void row_dma(const uint16_t* krow, int32_t c0, int32_t C, uint16_t* dst) {
  const int lane = threadIdx.x & 63;
  // The slot being refilled was last read one item ago; make sure those LDS
  // reads have completed before the DMA can land.
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  // A buffer load into LDS over the frame row: tracked by the vector-memory
  // counter only, so the ring reads keep exact lgkmcnt waits.
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(krow), 0, C * (kHeadDim * 2), kBufferFlags);
#pragma unroll
  for (int m = 0; m < kRowLoads; ++m) {
    const int g = 4 * m + (lane >> 4);
    const int slot = lane & 15;
    const int ch = chunk_slot(g, slot);  // the mapping is its own inverse
    const int32_t col = min(max(c0 - 1 + g, 0), C - 1);
    // The LDS address goes through an opaque copy, so the compiler does not
    // tie the DMA to the ring array and add its own (full) vmcnt waits before
    // the ring is read; the kernel waits for exactly the rows it needs.
    uint32_t lds = uint32_t(reinterpret_cast<uintptr_t>(dst + 4 * m * kHeadDim));
    asm volatile("" : "+s"(lds));
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_t)(uintptr_t)lds, 16,
                                             uint32_t(col) * (kHeadDim * 2) + uint32_t(ch) * 16u, 0, 0, 0);
  }
}

// Lane (g, s) holds chunks s, s+4, s+8, s+12 of cell g.
struct Slice {
  bf16x8_t c[4];
};

__device__ inline Slice read_slice(const uint16_t* row, int g, int s) {
  Slice x;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    x.c[j] = *reinterpret_cast<const bf16x8_t*>(row + g * kHeadDim + chunk_slot(g, 4 * j + s) * 8);
  return x;
}

// sum + a . b over the lane's 32 dimensions.
__device__ inline float dot_slice(const Slice& a, const Slice& b, float sum) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint4 va = __builtin_bit_cast(uint4, a.c[j]), vb = __builtin_bit_cast(uint4, b.c[j]);
    const uint32_t wa[4] = {va.x, va.y, va.z, va.w};
    const uint32_t wb[4] = {vb.x, vb.y, vb.z, vb.w};
#pragma unroll
    for (int i = 0; i < 4; ++i)
      sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, wa[i]), __builtin_bit_cast(bf16x2_t, wb[i]),
                                            sum, false);
  }
  return sum;
}

// Sum over the four lanes of a quad (lanes 4g .. 4g+3), in the vector unit
// (__shfl_xor goes through LDS, ten times a row here).
__device__ inline float quad_sum(float x) {
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0xB1, 0xf, 0xf, false));  // lane ^ 1
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x4E, 0xf, 0xf, false));  // lane ^ 2
  return x;
}

// 1/||k|| from ||k||^2 (0 for a zero key) without a branch: tiny square norms
// are scaled by 2^120 first, so that v_rsq_f32 (1 ulp) sees a normal number.
__device__ inline float inv_norm_select(float ss) {
  const bool tiny = ss < 0x1p-100f;
  const float r = __builtin_amdgcn_rsqf(tiny ? ss * 0x1p120f : ss) * (tiny ? 0x1p60f : 1.0f);
  return ss == 0.0f ? 0.0f : r;
}

// Phi = 0 on work-group x's piece of a text run (text_run) of a unit: run
// x % runs, every text_pieces-th kRunPiece tokens of it.  16-byte stores and
// long runs cut up: one wave with 4-byte stores took 414 us for a run of 2^20
// tokens in 4 units, this 6.6.  Short runs are bound by the latency of finding
// them.  (There are n_frames + 1 runs; the work-groups past them, one per
// further sequence, exit.  Zeroing short runs from the strips beside them was no
// faster over small frames, and these light work-groups between one unit's
// strips and the next one's spread the strips over the shader engines: without
// them 9 x 9 over 5 frames of 36 x 80 in 112 units took 211 us instead of 168.)
__device__ inline void zero_text(const CssArgs& a, int32_t unit, int32_t x) {
  float* out = a.phi + size_t(unit) * a.lay.total_tokens;
  const int32_t runs = a.lay.n_frames + a.lay.n_seqs;
  const int32_t piece = __builtin_amdgcn_readfirstlane(a.text_pieces > 1 ? x / runs : 0);
  const int32_t g = x - piece * runs;
  if (g > a.lay.n_frames) return;
  int32_t b, e;
  text_run(a.lay, g, &b, &e);
  if (e - b <= 256) {  // a few stores: not worth the alignment's arithmetic
    for (int32_t j = b + int32_t(threadIdx.x); piece == 0 && j < e; j += 64) out[j] = 0.0f;
    return;
  }
  for (int64_t j = b + int64_t(piece) * kRunPiece; j < e; j += int64_t(a.text_pieces) * kRunPiece)
    fill_run(out, int32_t(j), int32_t(min(j + kRunPiece, int64_t(e))), 0.0f, threadIdx.x, 64);
}

// Grid: x = strips (14 output columns of `a.seg_rows` frame rows) of every
// frame in XCD-aware order, then the text runs (a launch of their own took
// ~4.5 us of a pass over a small batch); y = unit, or layer with H > 1.
template <int H, bool GATED>
__global__ __launch_bounds__(64) void css_kernel(CssArgs a) {
  static_assert(H == 1 || !GATED, "the gate is per unit");
  __shared__ __attribute__((aligned(16))) uint16_t ring[kRing][kRowElems];
  const Layout& lay = a.lay;
  const int unit = blockIdx.y;
  if (int32_t(blockIdx.x) >= a.grid_x) {
    zero_text(a, unit, int32_t(blockIdx.x) - a.grid_x);
    return;
  }
  // XCD-aware order: work-groups i, i + 8, i + 16, ... share an XCD, so they
  // take consecutive strips (the grid width is a multiple of 8).
  const int32_t per_xcd = a.grid_x >> 3;
  const int32_t logical = int32_t(blockIdx.x & 7) * per_xcd + int32_t(blockIdx.x >> 3);
  const int32_t f = logical / a.strips, strip = logical - f * a.strips;
  if (f >= lay.n_frames) return;
  const int32_t off = lay.frame_meta[3 * f], R = lay.frame_meta[3 * f + 1], C = lay.frame_meta[3 * f + 2];
  CssStrip at;
  if (!css_strip(strip, R, C, kStripOut, a.seg_rows, &at)) return;
  const int32_t ra = at.row_begin, rb = at.row_end, c0 = at.col;  // output rows ra .. rb - 1
  const int32_t first = max(ra - 1, 0), last = min(rb, R - 1);  // key rows

  const int lane = threadIdx.x & 63, g = lane >> 2, s = lane & 3;
  const int32_t col = c0 - 1 + g;
  const bool out_lane = g >= 1 && g <= kStripOut && col < C;
  const bool has_w = col >= 1, has_e = col + 1 < C;
  const int32_t ncols = 1 + (col > 0 ? 1 : 0) + (col < C - 1 ? 1 : 0);
  const size_t head_stride = size_t(lay.total_tokens) * kHeadDim;
  const uint16_t* kframe = a.k + (size_t(unit) * H * lay.total_tokens + off) * kHeadDim;
  // Phi of the frame through a buffer resource: lanes without an output store
  // to an offset past the end, which the hardware drops, so the store needs no
  // branch (and the number of memory operations per step stays fixed).
  const uint32_t frame_bytes = uint32_t(R) * uint32_t(C) * 4u;
  const __amdgpu_buffer_rsrc_t phi_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(a.phi + size_t(unit) * lay.total_tokens + off, 0, frame_bytes, kBufferFlags);
  const int ge = min(g + 1, kStripCells - 1), gw = max(g - 1, 0);
  // The gate bytes of the frame (GATED): lanes without an output read an
  // offset past the end, which returns 0.
  const __amdgpu_buffer_rsrc_t gate_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(GATED ? a.gate + size_t(unit) * lay.total_tokens + off : nullptr), 0,
      GATED ? uint32_t(R) * uint32_t(C) : 0u, kBufferFlags);
  const uint32_t gate_none = uint32_t(R) * uint32_t(C);
  uint32_t gates[kRing];  // GATED: gate byte of row x + u - 1 in gates[u] (x: first row of the unrolled loop)
  gates[0] = 1u;

  // Item (row, head) into ring slot j; rows past `last` repeat it and hit L2,
  // so that the number of operations in flight is the same on every path.
  auto issue = [&](int32_t row, int h, int j, int gate) {
    row_dma(kframe + h * head_stride + size_t(min(row, last)) * C * kHeadDim, c0, C, ring[j]);
    if (GATED && h == 0)
      gates[gate] = __builtin_amdgcn_raw_buffer_load_b8(
          gate_rsrc, out_lane ? uint32_t(min(row, last) * C + col) : gate_none, 0, 0);
  };
  // Stores of Phi among the steps of the kRing - 1 items before an item of
  // head h: those of the last head (the store follows a row's last item).
  auto stores_before = [](int h) {
    int n = 0;
    for (int i = 1; i < kRing; ++i) n += (h - i + kRing * H) % H == H - 1 ? 1 : 0;
    return n;
  };
  // Items 0 .. kRing - 2 in flight, with stores the hardware drops where the
  // steps that issue them in the loop would store: every wait counts the same.
#pragma unroll
  for (int j = 0; j < kRing - 1; ++j) {
    issue(first + j / H, j % H, j, j + 1);
    asm volatile("" ::: "memory");
    if ((j - (kRing - 1) + kRing * H) % H == H - 1) __builtin_amdgcn_raw_buffer_store_b32(0u, phi_rsrc, frame_bytes, 0, 0);
    asm volatile("" ::: "memory");
  }

  Slice own[H];  // row x - 1, every head
#pragma unroll
  for (int h = 0; h < H; ++h)
#pragma unroll
    for (int j = 0; j < 4; ++j) own[h].c[j] = __builtin_bit_cast(bf16x8_t, make_uint4(0, 0, 0, 0));
  float rn_own = 0.0f;           // its inverse norm
  float cE_own = 0.0f, cE_w = 0.0f;  // its cosine with the east cell, and the west cell's
  float carry = 0.0f;            // sum of row x-2's cosines with (x - 1, col)

  // Row x arrives (u: its place in the unrolled loop): Phi of row x - 1.
  auto step = [&](int32_t x, int u) {
    const int32_t r = x - 1;
    // Norm and cosine products (own, E, S, SE, SW), in two sums over the heads:
    // one sum through all of them rounds more.  Phi against 64 bits at 4 heads,
    // independent neighbours 2.44e-8 -> 2.20e-8, neighbours alike 9.7e-7 ->
    // 7.0e-7; at 2 heads, alike, 6.4e-7 -> 5.6e-7.
    constexpr int kSums = H < 2 ? H : 2;
    float sums[kSums][5] = {};
    // A copy taken here: the byte's register takes the one loaded below.
    uint32_t open = GATED ? gates[u] : 1u;
    if (GATED) asm volatile("" : "+v"(open));
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int j = (u * H + h) % kRing;
      issue(x + (h + kRing - 1) / H, (h + kRing - 1) % H, (j + kRing - 1) % kRing, u);
      wait_outstanding((kRowLoads + (GATED ? 1 : 0)) * (kRing - 1) + stores_before(h));  // item (x, h) has landed
      const Slice dn = read_slice(ring[j], g, s);
      const Slice e = read_slice(ring[j], ge, s);
      const Slice w = read_slice(ring[j], gw, s);
      float* const sum = sums[h * kSums / H];
      sum[0] = dot_slice(dn, dn, sum[0]);
      sum[1] = dot_slice(dn, e, sum[1]);
      sum[2] = dot_slice(own[h], dn, sum[2]);
      sum[3] = dot_slice(own[h], e, sum[3]);
      sum[4] = dot_slice(own[h], w, sum[4]);
      own[h] = dn;
      // The sums are formed here: left to later, every item's slices stay live.
      if (H > 1) __builtin_amdgcn_sched_barrier(0);
    }
    const bool has_s = x < R;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
#pragma unroll
      for (int j = 1; j < kSums; ++j) sums[0][i] += sums[j][i];
      sums[0][i] = quad_sum(sums[0][i]);
    }
    const float nrm = sums[0][0], dE = sums[0][1], dS = sums[0][2], dSE = sums[0][3], dSW = sums[0][4];
    const float rn = H == 1 ? inv_norm_select(nrm) : (nrm > 0.0f ? 1.0f / sqrtf(nrm) : 0.0f);
    const float rnE = __shfl(rn, (ge << 2) | s);
    const float rnW = __shfl(rn, (gw << 2) | s);
    const float cE = has_e ? dE * rn * rnE : 0.0f;
    const float cS = has_s ? dS * rn_own * rn : 0.0f;
    const float cSE = has_s && has_e ? dSE * rn_own * rnE : 0.0f;
    const float cSW = has_s && has_w ? dSW * rn_own * rnW : 0.0f;
    // Cosines owned by the west / east neighbours of this cell.
    const float cE_from_w = __shfl(cE, (gw << 2) | s);
    const float cSE_w = __shfl(cSE, (gw << 2) | s);
    const float cSW_e = __shfl(cSW, (ge << 2) | s);
    const float sum = carry + cE_own + cS + cSE + cSW + cE_w;
    carry = cS + (has_w ? cSE_w : 0.0f) + (has_e ? cSW_e : 0.0f);
    const int32_t nrows = 1 + (r > 0 ? 1 : 0) + (has_s ? 1 : 0);
    const int32_t nn = nrows * ncols - 1;
    const bool store = r >= ra && r < rb && out_lane && s == 0;
    const uint32_t byte_off = store ? uint32_t(r * C + col) * 4u : frame_bytes;
    const float mean = H == 1 ? sum * __builtin_amdgcn_rcpf(float(nn)) : sum / float(nn);
    const bool zero = nn <= 0 || (GATED && open == 0u);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(zero ? 0.0f : 1.0f - mean), phi_rsrc, byte_off, 0, 0);
    rn_own = rn;
    cE_own = cE;
    cE_w = has_w ? cE_from_w : 0.0f;
  };

  // Item (x, h) lives in slot (x H + h) % kRing; unrolled so that each slot
  // is fixed.  Steps past row rb only keep the counts uniform.
  constexpr int kUnroll = H >= kRing ? 1 : kRing / H;
  for (int32_t x = first; x <= rb; x += kUnroll)
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) step(x + u, u);
  wait_vmcnt<0>();  // no DMA into LDS may outlive the work-group
}

constexpr int kWideCols = 16;  // output columns of a wave's strip

__device__ inline float sumsq8(uint4 v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  float s = 0.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w[j]), __builtin_bit_cast(bf16x2_t, w[j]), s, false);
  return s;
}

// Sum over the four 16-lane rows of a wave (lanes n, n + 16, n + 32, n + 48):
// each swap leaves one operand with the even (low) halves twice and the other
// with the odd (high) ones.
__device__ inline float sum_rows16(float x) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum over the 16 lanes of a row, by rotations inside the row.
__device__ inline float sum_lanes16(float x) {
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x128, 0xf, 0xf, false));
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x124, 0xf, 0xf, false));
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x122, 0xf, 0xf, false));
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x121, 0xf, 0xf, false));
  return x;
}

// LDS ring of the k x k walk: slots of 16 + 2 KR strip keys (rounded up to
// whole 4-key wave-loads) for the KR rows below the one being multiplied
// (already read as output rows) and kWideAhead rows in flight.
constexpr int kWideAhead = 2;
template <int KR>
struct WideRing {
  static constexpr int kKeys = (kWideCols + 2 * KR + 3) / 4 * 4;
  static constexpr int kLoads = kKeys / 4;  // wave-loads of 16 B per lane
  static constexpr int kSlots = KR + kWideAhead;
  static constexpr int kElems = kKeys * kHeadDim;
};

// Grid: x = strips (16 output columns of `a.seg_rows` frame rows, one wave
// each) in XCD-aware order, a.strips = the largest number of them in a frame,
// then the text runs; y = unit.
//
// A wave walks its strip downwards.  Every key row reaches LDS once, by DMA
// kWideAhead rows ahead, and is read from there twice: when it arrives, as the A
// operand of an output row (kept in registers for the 2 KR + 1 rows around
// it), and KR rows later as the 16 + 2 KR neighbour keys (two B blocks) that
// meet the 2 KR + 1 output rows within KR of it.  The walk is unrolled by
// 2 KR + 1, so that an output row's registers are fixed.
//
// 5 x 5: bound by the HBM stream (4.65 TB/s counted) and by issue; 7 x 7 and
// 9 x 9, one wave per SIMD, by issue (0.62 of the waves' time).  A wave tile of
// 4 x 16 outputs that loads its own neighbour rows moves 1 + 2 (4 + 2 KR) / 4
// keys per output through L2 (5 at KR = 2); the walk moves 1 + KR / 8.  112
// units x 20 frames of 36 x 80: 5 x 5 932 -> 375 us (4.4 TB/s of keys), 7 x 7
// 1102 -> 530, 9 x 9 1258 -> 605; 3 frames of 16 x 16 in 4 units: 16.2 -> 8.7,
// 18.2 -> 13.2, 20.1 -> 17.3.  Frames of four rows are the walk's weak side
// (300 of 4 x 5 in 112 units: 5 x 5 189 -> 144, 7 x 7 195 -> 234, 9 x 9 194 ->
// 264): a strip's start is as long as its rows.
//
// Fragments are read as bf16 vectors throughout: a read through another type
// makes the compiler wait for every DMA in flight before it.
template <int KR>
__global__ __launch_bounds__(64, KR == 2 ? 2 : 1) void css_wide_kernel(CssArgs a) {
  using Ring = WideRing<KR>;
  constexpr int NA = 2 * KR + 1;
  constexpr int kPerRow = Ring::kLoads + 1;  // vector-memory operations per step: the DMA and the store of Phi
  __shared__ __attribute__((aligned(16))) uint16_t ring[Ring::kSlots * Ring::kElems];
  const Layout& lay = a.lay;
  const int unit = blockIdx.y;
  if (int32_t(blockIdx.x) >= a.grid_x) {
    zero_text(a, unit, int32_t(blockIdx.x) - a.grid_x);
    return;
  }
  const int32_t per_xcd = a.grid_x >> 3;
  const int32_t logical = int32_t(blockIdx.x & 7) * per_xcd + int32_t(blockIdx.x >> 3);
  const int32_t f = logical / a.strips, t = logical - f * a.strips;
  if (f >= lay.n_frames) return;
  const int32_t off = lay.frame_meta[3 * f], R = lay.frame_meta[3 * f + 1], C = lay.frame_meta[3 * f + 2];
  CssStrip at;
  if (!css_strip(t, R, C, kWideCols, a.seg_rows, &at)) return;
  const int32_t ra = at.row_begin, rb = at.row_end, c0 = at.col;          // output rows ra .. rb - 1
  const int32_t first = max(ra - KR, 0), last = min(rb - 1 + KR, R - 1);  // key rows
  const uint16_t* kframe = a.k + (size_t(unit) * lay.total_tokens + off) * kHeadDim;
  const int lane = threadIdx.x, n = lane & 15, q = lane >> 4;

  const uint32_t frame_bytes = uint32_t(R) * uint32_t(C) * 4u;
  const __amdgpu_buffer_rsrc_t phi_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(a.phi + size_t(unit) * lay.total_tokens + off, 0, frame_bytes, kBufferFlags);

  // DMA of key row x (rows past `last` repeat it): strip key g is column
  // c0 - KR + g clamped into the frame; its chunk ch sits at ch ^ (g & 15).
  uint32_t dma_off[Ring::kLoads];
#pragma unroll
  for (int m = 0; m < Ring::kLoads; ++m) {
    const int g = 4 * m + (lane >> 4);
    const int32_t col = min(max(c0 - KR + g, 0), C - 1);
    dma_off[m] = uint32_t(col) * (kHeadDim * 2) + uint32_t((lane & 15) ^ (g & 15)) * 16u;
  }
  const uint32_t ring_base = uint32_t(reinterpret_cast<uintptr_t>(ring));
  auto issue = [&](int32_t x, int32_t slot) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(kframe + size_t(min(x, last)) * C * kHeadDim), 0, C * (kHeadDim * 2), kBufferFlags);
#pragma unroll
    for (int m = 0; m < Ring::kLoads; ++m) {
      uint32_t lds = ring_base + uint32_t(slot * Ring::kElems + 4 * m * kHeadDim) * 2u;
      asm volatile("" : "+s"(lds));
      const uint32_t from = dma_off[m];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_t)(uintptr_t)lds, 16, from, 0, 0, 0);
    }
  };
  auto next_slot = [](int32_t s) { return s + 1 == Ring::kSlots ? 0 : s + 1; };

  // Operand addresses inside a slot: A = strip keys KR + n, B block nb = strip
  // keys 16 nb + n (past the strip: its last key, masked below).
  int a_off[4], b_off[2][4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int ka = KR + n;
    a_off[kk] = ka * kHeadDim + (((4 * kk + q) ^ (ka & 15)) << 3);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int kb = min(16 * nb + n, Ring::kKeys - 1);
      b_off[nb][kk] = kb * kHeadDim + (((4 * kk + q) ^ (kb & 15)) << 3);
    }
  }

  // Accumulator element (i, n) of block nb pairs output column c0 + 4 q + i
  // with neighbour column c0 - KR + 16 nb + n: dc = 16 nb + n - KR - 4 q - i.
  bool near[2][4], off_self[2][4];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int32_t d = 16 * nb + n - 4 * q - i;  // dc + KR
      const int32_t cc = c0 - KR + 16 * nb + n;
      near[nb][i] = d >= 0 && d <= 2 * KR && cc >= 0 && cc < C;
      off_self[nb][i] = near[nb][i] && d != KR;
    }
  // The lane's output column (lanes n < 4 store) and where its inverse norm
  // lies among the strip keys.
  const int32_t col = c0 + 4 * q + (n & 3);
  const int strip_key = KR + 4 * q + (n & 3);
  const int32_t cols_in = min(col + KR, C - 1) - max(col - KR, 0) + 1;

  bf16x8_t ha[NA][4];
  float psum[NA][4], rn_out[NA];
#pragma unroll
  for (int o = 0; o < NA; ++o) {
    rn_out[o] = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) psum[o][i] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) ha[o][kk] = __builtin_bit_cast(bf16x8_t, make_uint4(0, 0, 0, 0));
  }
  auto load_a = [&](int32_t slot, bf16x8_t (&h)[4]) {
    const uint16_t* base = ring + slot * Ring::kElems;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) h[kk] = *reinterpret_cast<const bf16x8_t*>(base + a_off[kk]);
  };
  // Phi of output row o, or (row outside the strip) a store the hardware drops.
  auto store = [&](int32_t o, const float (&h)[4], float rn) {
    const float h0 = sum_lanes16(h[0]), h1 = sum_lanes16(h[1]), h2 = sum_lanes16(h[2]), h3 = sum_lanes16(h[3]);
    const float x = (n & 2) ? ((n & 1) ? h3 : h2) : ((n & 1) ? h1 : h0);
    const int32_t rows_in = min(o + KR, R - 1) - max(o - KR, 0) + 1;
    const int32_t nn = rows_in * cols_in - 1;
    const float phi = nn > 0 ? 1.0f - x * rn / float(nn) : 0.0f;
    const bool keep = o >= ra && o < rb && n < 4 && col < C;
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(phi), phi_rsrc,
                                          keep ? uint32_t(o * C + col) * 4u : frame_bytes, 0, 0);
  };

  // Rows first .. first + KR + kWideAhead - 1 in flight; the first KR become
  // output rows before the walk starts.  Stores past the frame's end stand in
  // for the steps that did not run, so that every wait counts the same.
#pragma unroll
  for (int x = 0; x < KR; ++x) issue(first + x, x);
#pragma unroll
  for (int x = 0; x < kWideAhead; ++x) {
    issue(first + KR + x, KR + x);
    asm volatile("" ::: "memory");  // the waits count on this order
    __builtin_amdgcn_raw_buffer_store_b32(0u, phi_rsrc, frame_bytes, 0, 0);
    asm volatile("" ::: "memory");
  }
  wait_vmcnt<kWideAhead * kPerRow>();
#pragma unroll
  for (int x = 0; x < KR; ++x) load_a(x, ha[x]);  // (rows past `last` hold its copy and are never stored)

  bf16x8_t v[2][4];  // neighbour row b's B fragments
  auto load_b = [&](int32_t slot) {
    const uint16_t* base = ring + slot * Ring::kElems;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) v[nb][kk] = *reinterpret_cast<const bf16x8_t*>(base + b_off[nb][kk]);
  };
  load_b(0);

  int32_t slot_b = 0, slot_a = KR;  // slots of rows b and b + KR
  // Step of neighbour row b, J = register set of output row b + KR.  The row's
  // norms are formed under the matrix work, the next row's fragments are read
  // under the vector work that follows it.
  auto step = [&](int32_t b, int J) {
    // A row past the frame's last one is no neighbour: it only completes output
    // row b - KR (9 x 9 over 300 frames of 4 x 5 in 112 units 412 -> 264 us, over
    // 48 of 36 x 80 1587 -> 1454; not at 5 x 5, where the branch cost short
    // strips 0.4 us of 8.6).
    if (KR > 2 && b > last) return store(b - KR, psum[(J + 1) % NA], rn_out[(J + 1) % NA]);
    const int JB = (J + KR + 1) % NA;  // register set of output row b
    // Row b is in registers: its slot takes row b + KR + kWideAhead.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issue(b + KR + kWideAhead, slot_b);
    slot_b = next_slot(slot_b);
    wait_vmcnt<kWideAhead * kPerRow>();  // row b + KR has landed
    load_a(slot_a, ha[J]);
    slot_a = next_slot(slot_a);
#pragma unroll
    for (int i = 0; i < 4; ++i) psum[J][i] = 0.0f;
    f32x4_t acc[NA][2];
#pragma unroll
    for (int x = 1; x <= NA; ++x) {
      const int o = (J + x) % NA;  // the row just read comes last
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        acc[o][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          acc[o][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ha[o][kk], v[nb][kk], acc[o][nb], 0, 0, 0);
      }
    }
    float rn[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      float ss = 0.0f;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) ss += sumsq8(__builtin_bit_cast(uint4, v[nb][kk]));
      rn[nb] = inv_norm_select(sum_rows16(ss));
    }
    const float r0 = __shfl(rn[0], strip_key & 15), r1 = __shfl(rn[1], strip_key & 15);
    rn_out[JB] = strip_key < 16 ? r0 : r1;
    // Rows past the strip's last one are its copy and weigh nothing.
    if (KR == 2 && b > last) rn[0] = rn[1] = 0.0f;
    __builtin_amdgcn_sched_barrier(0);
    load_b(slot_b);
#pragma unroll
    for (int o = 0; o < NA; ++o)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool keep = o == JB ? off_self[nb][i] : near[nb][i];
          psum[o][i] = fmaf(acc[o][nb][i], keep ? rn[nb] : 0.0f, psum[o][i]);
        }
    store(b - KR, psum[(J + 1) % NA], rn_out[(J + 1) % NA]);
  };
  const int32_t end = rb - 1 + KR;  // the last output row is complete after neighbour row end
  for (int32_t b = first; b <= end; b += NA) {
#pragma unroll
    for (int j = 0; j < NA; ++j)
      if (b + j <= end) step(b + j, (KR + j) % NA);
  }
  wait_vmcnt<0>();  // no DMA into LDS may outlive the work-group
}

}  // namespace

hipError_t launch_css_wide(const CssArgs& a_in, int32_t nbhd, hipStream_t stream) {
  CssArgs a = a_in;
  const int64_t logical = int64_t(a.lay.n_frames) * a.strips;  // a.strips: max over frames of 16-column strips
  a.grid_x = int32_t((logical + 7) / 8 * 8);
  const dim3 grid(unsigned(a.grid_x) + unsigned(a.lay.n_frames + a.lay.n_seqs) * a.text_pieces, a.lay.n_units);
  switch (nbhd) {
    case 5: hipLaunchKernelGGL(css_wide_kernel<2>, grid, dim3(64), 0, stream, a); break;
    case 7: hipLaunchKernelGGL(css_wide_kernel<3>, grid, dim3(64), 0, stream, a); break;
    case 9: hipLaunchKernelGGL(css_wide_kernel<4>, grid, dim3(64), 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_css(const CssArgs& a_in, hipStream_t stream) {
  CssArgs a = a_in;
  const int64_t logical = int64_t(a.lay.n_frames) * a.strips;  // a.strips: max over frames of 14-column strips
  a.grid_x = int32_t((logical + 7) / 8 * 8);
  const dim3 grid(unsigned(a.grid_x) + unsigned(a.lay.n_frames + a.lay.n_seqs) * a.text_pieces, a.lay.n_units);
  if (a.gate)
    hipLaunchKernelGGL((css_kernel<1, true>), grid, dim3(64), 0, stream, a);
  else
    hipLaunchKernelGGL((css_kernel<1, false>), grid, dim3(64), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_css_concat(const CssArgs& a_in, hipStream_t stream) {
  CssArgs a = a_in;
  const int32_t H = a.lay.n_kv_heads, n_layers = a.lay.n_units / H;
  const int64_t logical = int64_t(a.lay.n_frames) * a.strips;
  a.grid_x = int32_t((logical + 7) / 8 * 8);
  const dim3 grid(unsigned(a.grid_x) + unsigned(a.lay.n_frames + a.lay.n_seqs) * a.text_pieces, n_layers);
  if (H == 2)
    hipLaunchKernelGGL((css_kernel<2, false>), grid, dim3(64), 0, stream, a);
  else if (H == 4)
    hipLaunchKernelGGL((css_kernel<4, false>), grid, dim3(64), 0, stream, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace stlite
