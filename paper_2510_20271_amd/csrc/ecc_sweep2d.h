// 2D sweep for gfx950 (device templates shared by the hard and the soft kernels): coefficient c(p) (Eq. 3 of the paper) + LDS histogram,
// one wavefront per column strip, marching down the rows.
//
// Layout.  A wave owns a strip of 248 output columns; its 64 lanes hold four
// consecutive columns each, 256 columns starting four before the first output
// column, so lanes 0 and 63 are halo lanes and a row of the strip is a single
// 16-byte-aligned 1 KiB load (buffer_load_dwordx4).  The rows of the strip
// stream through registers; nothing is staged in LDS, and a vertex is read
// from HBM once per strip plus the 8/248 halo.
//
// Stencil, bit-sliced down the rows.  "q comes before p" is a strict "<"
// towards the four later neighbours (+x and the three in the next row): the
// sign bit of the float difference q - p (zeros are made +0 on load so that
// equal values give +0).  Each lane shifts those sign bits into four 32-bit
// words per column, one bit per row, so after 32 rows a word holds one
// later-neighbour relation of 32 vertices of a column.  The four earlier
// neighbours need no compare: [q before p] = not [p before q], which is the
// bit the row above (word shifted by one bit) or the column to the left /
// right (the neighbouring word, one lane over at a lane boundary) produced for
// ITS later neighbour.  Vertices outside the grid read as +inf, which makes
// every bit that involves them come out right ("never before p") with no
// boundary cases.  All Boolean work then runs on whole words: 32 vertices per
// lane per instruction.
//
// Coefficient from arc starts.  The vertices before p cut the 8-ring around p
// into arcs; a diagonal joins its two edge neighbours only if all three come
// before p.  c(p) = 1 - (#arcs), and an arc starts at edge neighbour k when k
// comes before p but not both its clockwise predecessors:
//     start_k = r_k & ~(r_{k-1} & r_{k-2}),   c = 1 - sum_k start_k.
// Vertices with exactly one start have c = 0 (regular vertices: almost all of
// a smooth field).  Only the others are walked bit by bit and binned into the
// block's LDS histogram; their values come from a small LDS ring into which the
// wave copies each row as it becomes current (re-reading them from memory
// would miss the L2 once per critical vertex, a 128-byte line for 4 bytes).
#pragma once
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "ecc_device.h"
#include "ecc_internal.h"

namespace ecc {

constexpr int kNC = 4;                       // columns per lane
constexpr int kStripOut = (kWave - 2) * kNC;  // 248 output columns per wave
constexpr int kPF = 4;                        // rows in flight ahead of the row being compared
constexpr int kChunkRows = 8;                 // rows per chunk = rows of the LDS value ring

__device__ __forceinline__ unsigned word_from_right(unsigned v) {  // lane i <- lane i+1
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, true);
}
__device__ __forceinline__ unsigned word_from_left(unsigned v) {  // lane i <- lane i-1
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);
}
__device__ __forceinline__ unsigned long long ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// w <- (w << 1) | signbit(d)
__device__ __forceinline__ unsigned push_sign(unsigned w, float d) {
  return __builtin_amdgcn_alignbit(w, __float_as_uint(d), 31);
}

// The three differences of a row step whose left operand lives in a
// neighbouring lane, as DPP-modified subtractions (no separate lane move):
//   dE  = cur_first[i+1] - cur_last[i]     (+x neighbour of a lane's last column)
//   dNE = nxt_first[i+1] - cur_last[i]
//   dNW = nxt_last[i-1]  - cur_first[i]
// Lanes without a source lane read 0; their bits belong to halo lanes and are
// never used.  The s_nop covers the two wait states a DPP read needs after a
// VALU write of its source register.
__device__ __forceinline__ void lane_edge_differences(float cur_first, float cur_last, float nxt_first,
                                                      float nxt_last, float& dE, float& dNE, float& dNW) {
  asm("s_nop 1\n\t"
      "v_sub_f32_dpp %0, %3, %4 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_sub_f32_dpp %1, %5, %4 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_sub_f32_dpp %2, %6, %3 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
      : "=&v"(dE), "=&v"(dNE), "=&v"(dNW)
      : "v"(cur_first), "v"(cur_last), "v"(nxt_first), "v"(nxt_last));
}

// Four consecutive elements of a row, by one raw buffer load: wave-uniform resource + scalar row offset + constant
// lane offset, so addressing costs no vector instruction, and dwords past the end of the item read as 0 instead of
// faulting.  Loads are dword-aligned whatever the row's own alignment is.  ANY = false: every row starts at a
// multiple of four bytes.  ANY = true (one- and two-byte elements): the load takes one dword more, and the row's
// bytes are picked out by a funnel shift whose amount is the same for all lanes of a row (a lane's columns are a
// multiple of four bytes from its neighbour's).  Rows of an odd width went element by element before, four loads a
// lane and row: a 4677 x 3307 uint8 page took 42 us, now 25 (sweep 30 -> 13); a
// training step on 16 x 217 x 181 float32 images with 512 thresholds 146 -> 118 us.
template <typename T, bool ANY> struct Row4;
template <> struct Row4<float, false> {
  typedef __attribute__((ext_vector_type(4))) unsigned vec;
  vec v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
  }
  __device__ __forceinline__ float get(int e) const { return __uint_as_float(v[e]); }
};
// two-byte elements, widened to float32 element by element
template <typename T> struct Row4<T, false> {
  typedef __attribute__((ext_vector_type(2))) unsigned vec;
  vec v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
  }
  __device__ __forceinline__ float get(int e) const { return widen16<T>(v[e >> 1] >> (16 * (e & 1))); }
};
template <typename T> struct Row4<T, true> {
  typedef __attribute__((ext_vector_type(3))) unsigned vec;
  vec v;
  unsigned shift;  // bits (wave-uniform)
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    v = __builtin_amdgcn_raw_buffer_load_b96(r, voff, soff & ~3u, 0);
    shift = (soff & 3u) * 8u;
  }
  __device__ __forceinline__ float get(int e) const {
    const unsigned w = __builtin_amdgcn_alignbit(v[(e >> 1) + 1], v[e >> 1], shift);
    return widen16<T>(w >> (16 * (e & 1)));
  }
};
template <> struct Row4<uint8_t, false> {
  unsigned v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    v = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
  }
  __device__ __forceinline__ float get(int e) const { return (float)((v >> (8 * e)) & 0xffu); }
};
template <> struct Row4<uint8_t, true> {
  typedef __attribute__((ext_vector_type(2))) unsigned vec;
  vec v;
  unsigned shift;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff & ~3u, 0);
    shift = (soff & 3u) * 8u;
  }
  __device__ __forceinline__ float get(int e) const {
    const unsigned w = __builtin_amdgcn_alignbit(v[1], v[0], shift);
    return (float)((w >> (8 * e)) & 0xffu);
  }
};

// One strip: lanes hold columns c0 + 4*lane + e; output rows y0 .. y1-1
// (y0 < y1 <= H).
//
// Rows are "current" one after the other; a step pushes the four later-
// neighbour bits of every column of the current row into the words and copies
// the row into the wave's LDS ring.  A chunk is up to kChunkRows steps; the bits of the row above a chunk's first row are bit 0
// of the previous chunk's words (one warm-up step on row y0-1 provides them
// for the first chunk; above the grid they are all ones, i.e. "never before
// p" once complemented).
//
// Tilt: the field swept is Y(p) = X(p) + t(p) with t = fl(fl(a_x x) + fl(a_y y)),
// every operation a float32 one in this order (directional curves; NoTilt: Y = X).
//
// Lanes lane_lo .. lane_hi put out their vertices; the others are halo lanes.  A strip inside the
// grid has one halo lane on each side (1 .. 62).  A strip that starts at the grid's first column
// (open_left) or ends at its last one (open_right) has no neighbour lane there: the vertices beyond
// the grid are "never before p" (always, for the top-cell order), and the words that would come
// from the missing lane are set to say so once per chunk.
// OPEN: the strip may be such a first / last strip (compiled apart, so that the strips inside the
// grid carry none of this).
// EDGE: some column of the wave lies outside the grid (a grid narrower than a wave, or the last strip of a width
// that is no multiple of four); such columns load whatever is there and are replaced.
// ANY: see Row4.
template <typename T, typename Sink, bool EDGE, bool ANY, typename Tilt, bool OPEN = false>
__device__ __forceinline__ void sweep_strip(const T* __restrict__ g, int64_t item_elems, int H, int W,
                                            int c0, int y0, int y1, WaveQueue<Sink>& queue,
                                            float* ring /* [kChunkRows][64][kNC] */, WaveRange& range,
                                            const Tilt& tilt, int lane_lo_ = 1, int lane_hi_ = kWave - 2,
                                            bool open_left_ = false, bool open_right_ = false) {
  const int lane_lo = OPEN ? lane_lo_ : 1, lane_hi = OPEN ? lane_hi_ : kWave - 2;
  const bool open_left = OPEN && open_left_, open_right = OPEN && open_right_;
  const int lane = threadIdx.x & (kWave - 1);
  bool ok[kNC];  // column inside the grid
#pragma unroll
  for (int e = 0; e < kNC; ++e) {
    const int x = c0 + kNC * lane + e;
    ok[e] = x >= 0 && x < W;
  }
  const bool out_lane = lane >= lane_lo && lane <= lane_hi;
  // what a relation towards a vertex beyond the grid reads: never before p, or always (top-cell order)
  constexpr unsigned kBeyond = Tilt::kTop ? 0xffffffffu : 0u;
  const bool first_lane = open_left && lane == 0, last_lane = open_right && lane == kWave - 1;

  // The resource starts at the first streamed row (and at column c0 unless the strip is an EDGE one), rounded down
  // to a dword; `soff` is the byte offset of a row from there.
  const int ya = max(y0 - 1, 0);
  const int64_t first = (int64_t)ya * W + (EDGE ? 0 : c0);
  const unsigned skew = ANY ? (unsigned)(reinterpret_cast<uintptr_t>(g + first) & 3) : 0u;
  int64_t left = (item_elems - first) * (int64_t)sizeof(T) + skew;
  if (ANY) left = (left + 3) & ~(int64_t)3;  // (the dword that holds the item's last bytes counts whole)
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(g + first) - skew), 0,
      (int)(left > 0x7fffffff ? 0x7ffffffc : left), 0x00020000);
  // EDGE: lanes wholly outside the grid load what the first / last lane inside loads (c0 is a multiple of four, -4
  // at the least)
  const unsigned voff = (unsigned)(EDGE ? min(max(c0 + kNC * lane, 0), (W - 1) / kNC * kNC) : kNC * lane) *
                        (unsigned)sizeof(T);
  const unsigned row_bytes = (unsigned)W * (unsigned)sizeof(T);
  unsigned soff = skew;  // offset of the next row to load
  // The last row this segment needs is y1 (the row below its last output row), or
  // the grid's last row; the rows the pipeline would fetch beyond it are not read
  // from memory again: the offset stays on that row (a cache hit).
  const unsigned soff_last = skew + (unsigned)(min(y1, H - 1) - ya) * row_bytes;
  auto next_row = [&]() { soff = min(soff + row_bytes, soff_last); };

  typedef Row4<T, ANY> Row;
  // value of column e of a loaded row, which is row y of the grid
  float lx[kNC];  // the column's share of the tilt (zero made +0: equal values must differ by +0)
#pragma unroll
  for (int e = 0; e < kNC; ++e)
    lx[e] = Tilt::kOn ? add_rn(mul_rn(tilt.ax, (float)(c0 + kNC * lane + e)), 0.0f) : 0.0f;
  // (zeros come out as +0 in every mode, so that equal values differ by +0; a column
  // outside the grid reads as "never before p": +inf, or -inf where the order is reversed)
  auto value_at = [&](const Row& r, int e, int y) -> float {
    float f = r.get(e);
    if (Tilt::kNeg) {
      // 0 - f, zeros coming out as +0.  Kept opaque: left to itself the compiler replaces later
      // uses of it by a negated source operand, which turns +0 into -0 in a difference.
      f = 0.0f - f;
      asm volatile("" : "+v"(f));
    }
    else if (Tilt::kOn) f = add_rn(f, add_rn(lx[e], mul_rn(tilt.ay, (float)y)));
    else if (HasNegZero<T>::value) f += 0.0f;
    if (EDGE) f = ok[e] ? f : (Tilt::kTop ? -INFINITY : INFINITY);
    return f;
  };
  auto original = [](float f) -> float { return Tilt::kNeg ? -f : f; };  // the value that is binned
  Row pf[kPF];
  float cur[kNC], nxt[kNC];
  int yn = ya + 2;  // row of the grid that becomes nxt at the next step
  {
    Row a, b;
    a.load(rsrc, voff, soff);
    next_row();
    b.load(rsrc, voff, soff);
    next_row();
#pragma unroll
    for (int k = 0; k < kPF; ++k) {
      pf[k].load(rsrc, voff, soff);
      next_row();
    }
#pragma unroll
    for (int e = 0; e < kNC; ++e) {
      cur[e] = value_at(a, e, ya);
      nxt[e] = value_at(b, e, ya + 1);
    }
  }

  // Range (single-pass mode).  The smallest vertex of the grid is critical
  // (c = 1) and so is the largest one unless it lies on the grid's boundary (an
  // interior vertex with all eight neighbours before it has c = 1 as well), so
  // the range is taken over the critical vertices and the boundary vertices:
  // EDGE strips look at all their values, interior strips at the grid's first
  // and last row here and at the critical vertices where they are pushed.
  if (Sink::kTrackRange && !EDGE) {
    if (y0 == 0) {
      Row t;
      t.load(rsrc, voff, skew);
#pragma unroll
      for (int e = 0; e < kNC; ++e) range.add(original(value_at(t, e, 0)));
    }
    if (y1 >= H) {
      Row t;
      t.load(rsrc, voff, skew + (unsigned)(H - 1 - ya) * row_bytes);
#pragma unroll
      for (int e = 0; e < kNC; ++e) range.add(original(value_at(t, e, H - 1)));
    }
  }

  unsigned wE[kNC], wN[kNC], wNE[kNC], wNW[kNC];
#pragma unroll
  for (int e = 0; e < kNC; ++e) wE[e] = wN[e] = wNE[e] = wNW[e] = 0;

  int slot = 0;  // ring row of the current row
  auto step = [&]() {
    *reinterpret_cast<float4*>(ring + (slot * kWave + lane) * kNC) =
        make_float4(cur[0], cur[1], cur[2], cur[3]);
    ++slot;
    if (Sink::kTrackRange && EDGE) {
#pragma unroll
      for (int e = 0; e < kNC; ++e) range.add_if(original(cur[e]), ok[e]);
    }
    if (Sink::kTrackRange && !EDGE) {  // the grid's first / last column (wave-uniform conditions)
      if (open_left) range.add_if(original(cur[0]), first_lane);
      if (open_right) range.add_if(original(cur[kNC - 1]), last_lane);
    }
    float dE, dNE, dNW;
    lane_edge_differences(cur[0], cur[kNC - 1], nxt[0], nxt[kNC - 1], dE, dNE, dNW);
#pragma unroll
    for (int e = 0; e < kNC; ++e) {
      wE[e] = push_sign(wE[e], e + 1 < kNC ? cur[e + 1] - cur[e] : dE);
      wN[e] = push_sign(wN[e], nxt[e] - cur[e]);
      wNE[e] = push_sign(wNE[e], e + 1 < kNC ? nxt[e + 1] - cur[e] : dNE);
      wNW[e] = push_sign(wNW[e], e > 0 ? nxt[e - 1] - cur[e] : dNW);
    }
#pragma unroll
    for (int e = 0; e < kNC; ++e) {
      cur[e] = nxt[e];
      nxt[e] = value_at(pf[0], e, yn);
    }
    ++yn;
#pragma unroll
    for (int q = 0; q + 1 < kPF; ++q) pf[q] = pf[q + 1];
    pf[kPF - 1].load(rsrc, voff, soff);
    next_row();
  };

  // relations of the strip's outermost columns towards vertices beyond the grid (the lane that would
  // supply the other operand does not exist: the differences pushed there mean nothing)
  auto beyond_the_grid = [&]() {
    if (open_left) wNW[0] = first_lane ? kBeyond : wNW[0];
    if (open_right) {
      wE[kNC - 1] = last_lane ? kBeyond : wE[kNC - 1];
      wNE[kNC - 1] = last_lane ? kBeyond : wNE[kNC - 1];
    }
  };
  unsigned oN[kNC], oNE[kNC], oNW[kNC];  // bit 0: the row above the first output row
#pragma unroll
  for (int e = 0; e < kNC; ++e) oN[e] = oNE[e] = oNW[e] = Tilt::kTop ? 0 : 1;  // (reversed order: always before p)
  if (y0 > 0) {
    step();  // warm-up on row y0-1
    beyond_the_grid();
#pragma unroll
    for (int e = 0; e < kNC; ++e) {
      oN[e] = wN[e];
      oNE[e] = wNE[e];
      oNW[e] = wNW[e];
    }
  }

  for (int r = y0; r < y1; r += kChunkRows) {
    const int n = min(kChunkRows, y1 - r);
#pragma unroll
    for (int e = 0; e < kNC; ++e) wE[e] = wN[e] = wNE[e] = wNW[e] = 0;
    slot = 0;
    int k = 0;
    for (; k + kPF <= n; k += kPF) {
#pragma unroll
      for (int q = 0; q < kPF; ++q) step();
    }
    for (; k < n; ++k) step();
    beyond_the_grid();
    if constexpr (Sink::kZeroFill) {  // the sink's per-vertex output is 0 except at critical vertices
      for (int j = 0; j < n; ++j) queue.sink.template zero_row<EDGE>(r + j, c0 + kNC * lane, ok, out_lane);
    }
    const bool bottom = r + n >= H;  // the grid's last row has nothing below it
    const int pad = 32 - n;          // row r+j sits at bit 31-j
    const unsigned rows = 0xffffffffu << pad;

    unsigned E[kNC], N[kNC], NE[kNC], NW[kNC], pN[kNC], pNE[kNC], pNW[kNC];
#pragma unroll
    for (int e = 0; e < kNC; ++e) {
      if (bottom) {
        if (Tilt::kTop) {  // reversed order: what lies outside the grid comes before p
          wN[e] |= 1u;
          wNE[e] |= 1u;
          wNW[e] |= 1u;
        } else {
          wN[e] &= ~1u;
          wNE[e] &= ~1u;
          wNW[e] &= ~1u;
        }
      }
      E[e] = wE[e] << pad;
      N[e] = wN[e] << pad;
      NE[e] = wNE[e] << pad;
      NW[e] = wNW[e] << pad;
      // the row above is one bit up (bit 31 from the previous chunk)
      pN[e] = __builtin_amdgcn_alignbit(oN[e], N[e], 1);
      pNE[e] = __builtin_amdgcn_alignbit(oNE[e], NE[e], 1);
      pNW[e] = __builtin_amdgcn_alignbit(oNW[e], NW[e], 1);
      oN[e] = wN[e];
      oNE[e] = wNE[e];
      oNW[e] = wNW[e];
    }
    // words of the columns just left / right of this lane's four
    const unsigned E_left = word_from_left(E[kNC - 1]);
    const unsigned pNEE_left = word_from_left(pNE[kNC - 1] | E[kNC - 1]);
    unsigned pNW_right = word_from_right(pNW[0]);
    // [p before its neighbour] towards a neighbour beyond the grid, where no lane supplies the word
    unsigned E_left_ = E_left, pNEE_left_ = pNEE_left;
    if (open_left) {
      E_left_ = first_lane ? ~kBeyond : E_left;
      pNEE_left_ = first_lane ? ~kBeyond : pNEE_left;
    }
    if (open_right) pNW_right = last_lane ? ~kBeyond : pNW_right;
    // A chunk uses the top kChunkRows (8) bits of a word, so the four columns of a
    // lane are packed into one word (column e in byte 3-e) and walked in one loop.
    static_assert(kChunkRows * kNC <= 32, "four columns of a chunk must fit one word");
    unsigned pE = 0, pNn = 0, pW = 0, pS = 0, nz = 0;
#pragma unroll
    for (int e = 0; e < kNC; ++e) {
      const unsigned El = e > 0 ? E[e - 1] : E_left_;                             // [p before its -x neighbour]
      const unsigned pNEEl = e > 0 ? (pNE[e - 1] | E[e - 1]) : pNEE_left_;        // SW or W relation, complemented
      const unsigned pNWr = e + 1 < kNC ? pNW[e + 1] : pNW_right;                 // SE relation, complemented
      const unsigned sE = E[e] & (pNWr | pN[e]);
      const unsigned sN = N[e] & ~(NE[e] & E[e]);
      const unsigned sW = ~(El | (NW[e] & N[e]));
      const unsigned sS = pNEEl & ~pN[e];
      const unsigned x1 = sE ^ sN, c1 = sE & sN, x2 = sW ^ sS, c2 = sW & sS;
      const unsigned one = (x1 ^ x2) & ~(c1 | c2);
      const unsigned crit = ok[e] ? (~one & rows) : 0u;
      const unsigned top = 0xff000000u;
      pE |= (sE & top) >> (8 * e);
      pNn |= (sN & top) >> (8 * e);
      pW |= (sW & top) >> (8 * e);
      pS |= (sS & top) >> (8 * e);
      nz |= (crit & top) >> (8 * e);
    }
    if (!out_lane) nz = 0u;
    while (ballot(nz != 0)) {
      const bool active = nz != 0;
      const int b = active ? 31 - __clz(nz) : 0;
      nz &= ~(1u << b);
      const int c = 1 - (int)((pE >> b) & 1u) - (int)((pNn >> b) & 1u) - (int)((pW >> b) & 1u) -
                    (int)((pS >> b) & 1u);
      const int pos = 31 - b;  // column pos / 8, row pos % 8 of the chunk
      const float v = original(ring[((pos & 7) * kWave + lane) * kNC + (pos >> 3)]);
      if (Sink::kTrackRange && !EDGE) range.add_if(v, active);
      queue.push(active, v, c, c0 + kNC * lane + (pos >> 3), r + (pos & 7));
    }
  }
  queue.flush();
}

// Work unit of a wave: (segment of rows) x (strip of columns) of one item;
// blockIdx.y is the item, the four waves of a block take adjacent strips.
template <typename T, typename Sink, typename Tilt>
__device__ __forceinline__ void sweep2d_wave(const T* __restrict__ g, int H, int W, int64_t N, int nstrip,
                                             int nseg, int rows_per_seg, WaveQueue<Sink>& queue, float* ring,
                                             WaveRange& range, const Tilt& tilt) {
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  if (unit < nstrip * nseg) {
    const int seg = unit / nstrip, strip = unit - seg * nstrip;
    const int y0 = seg * rows_per_seg;
    const int y1 = min(y0 + rows_per_seg, H);
    // Strip s puts out the columns [248 s, 248 s + 248).  With 256 columns or more the strips inside the grid start
    // four columns early (a halo lane on each side), the first strip starts at column 0 (its first lane puts out,
    // two halo lanes at the end) and the last strip ends at column W - 1 (its last lane puts out, the lanes before
    // its first column are halo).  That last one needs a width that is a multiple of four; otherwise it, like every
    // strip of a narrower grid, is an EDGE strip, and so is the strip before it when its halo lane reaches beyond
    // the grid (the range must not see what is read there).
    const bool left = strip == 0, right = strip == nstrip - 1;  // (W >= 256: at least two strips)
    constexpr bool kNarrow = sizeof(T) < 4;
    if (W < kNC * kWave || ((W % kNC) != 0 && (strip + 1) * kStripOut + kNC > W)) {
      sweep_strip<T, Sink, true, kNarrow>(g, N, H, W, strip * kStripOut - kNC, y0, y1, queue, ring, range, tilt);
      return;
    }
    int c0 = strip * kStripOut - kNC, lo = 1, hi = kWave - 2;
    if (left) {
      c0 = 0;
      lo = 0;
      hi = kWave - 3;
    }
    if (right) {
      c0 = W - kNC * kWave;
      lo = (strip * kStripOut - c0) / kNC;
      hi = kWave - 1;
    }
    auto strip_of = [&](auto any) {
      constexpr bool ANY = decltype(any)::value;
      if (left || right)
        sweep_strip<T, Sink, false, ANY, Tilt, true>(g, N, H, W, c0, y0, y1, queue, ring, range, tilt, lo, hi, left, right);
      else
        sweep_strip<T, Sink, false, ANY>(g, N, H, W, c0, y0, y1, queue, ring, range, tilt);
    };
    if constexpr (kNarrow) {
      if (((reinterpret_cast<uintptr_t>(g) | (uintptr_t)W * sizeof(T)) & 3) != 0) {
        strip_of(std::true_type());
        return;
      }
    }
    strip_of(std::false_type());
  }
}

struct Plan2d {
  int nstrip, nseg, rows_per_seg;
  dim3 grid;
};
// What the sweep feeds: it decides how many rows a wave takes.  A wave's march is a chain of dependent steps (about
// 0.4 us a row when it has a SIMD for itself), so a launch that does not fill the chip wants short segments; every
// segment reads five rows more than it puts out, and a block has costs of its own at its end.
enum class Feed2d { kHist, kBlockLists, kSharedLists, kSigmoid };

// LDS of a block besides the sink's own needs: value rings + queues of the four waves
template <typename Entry>
constexpr size_t ring_bytes2d() {
  return (size_t)4 * kChunkRows * kWave * kNC * sizeof(float) + (size_t)4 * kQueueCap * sizeof(Entry);
}
static inline bool table_in_lds2d(int bins) { return (size_t)bins * 8 + ring_bytes2d<float2>() <= 64 * 1024; }  // the thresholds

// rows a wave takes; tubes: strips of all items; bytes: of an element; bins, levels (one bin per level): of a kHist sweep
static inline int64_t rows2d(const Shape& s, int64_t nstrip, int64_t tubes, Feed2d feed, int bytes, int bins, bool levels) {
  const int64_t H = s.H, total = s.N * s.batch;
  auto waves = [&](int64_t rows) { return tubes * ((H + rows - 1) / rows); };
  if (feed == Feed2d::kSigmoid) {
    // 8 rows while that gives up to three waves for each of the 1024 SIMDs (ecc_soft_fwd + ecc_soft_bwd on
    // 4 x 1024^2, T = 64: 46 -> 36 us; one 2048^2, T = 256: 69 -> 50 us); else 24 when that still leaves two rounds
    // of waves, else 16
    if (waves(8) <= 3072) return 8;
    return waves(24) >= 8192 ? 24 : 16;
  }
  if (feed == Feed2d::kBlockLists) {
    // A list per block: nothing is merged at a block's end.  Measured with 8 / 16 / 24 / 32 rows (us a call, float32): 1024 x
    // 28^2 13.4 / 13.8 / 13.7 / 15.6, 1024^2 13.5 / 15.7 / 17.9 / 20.3, 2048^2 16.9 / 18.1 / 19.8 / 22.0 (white noise 42.5 / 62.7 / 83.6 /
    // 106), 16 x 512^2 16.5 / 18.0 / 20.2 / 21.4, 64 x 256^2 15.1 / 15.4 / 17.9 / 19.3, 64 directions of 256^2 15.3 / 15.3 / 17.8 / 18.1;
    // 32 x 512^2 23.6 / 21.6 / 24.6 / 25.3, 4096^2 30.7 / 32.7 / 28.8 / 30.3, 8 x 4096^2 149 / 137 / 135 / 138: eight rows up to four
    // waves a SIMD (or few vertices), then by the height (24 rows leave a low image's last segment and block half empty).  32
    // rows take 5 to 9 % less on smooth images up to 1024 rows high (512 x 256^2 57.3 / 52.6 with 16 / 32, 128 x 512^2 52.9 / 48.7)
    // and more on white noise (128 x 512^2 137 / 154): not taken.
    int64_t rows = H <= 1024 ? 16 : 24;
    // But a block an image where its four waves have all but equal shares and every SIMD four waves: 1024 x 128^2 40.4 -> 35.7
    // (noise 72.1 -> 69.9), 2000 x 96^2 63.3 -> 52.5, 1502 x 89 x 194 noise 112 -> 96, 4000 x 142 x 57 float16 noise 340 -> 231; with two
    // waves a SIMD it costs (512 x 128^2 21.6 -> 23.3).
    const int64_t quarter = ((H + 3) / 4 + kChunkRows - 1) / kChunkRows * kChunkRows;
    if (nstrip == 1 && s.batch >= 1024 && quarter >= 24 && quarter <= 40) return quarter;
    // (below 32 rows the lists' room, rounded up to segments, would grow)
    if ((H >= 32 && waves(8) <= 4608) || (total < ((int64_t)1 << 22) && nstrip * ((H + 7) / 8) <= 2048)) rows = 8;
    // Many waves cost more in the blocks' heads than short segments gain (500000 x 8 101 / 81 / 76 / 78 / 78,
    // 2000000 x 8 361 / 284 / 260 / 248 / 236)
    while (rows < 64 && waves(rows) > 24576) rows *= 2;
    return rows;
  }
  if (feed == Feed2d::kHist) {
    // A histogram per block, merged at its end (hist_out).  The least of what a launch was found to take, in us, over the rows
    // that a wave may take (5400 calls of 2^17 to 2^27 vertices, element types of one, two and four bytes, 60 to 4096 bins,
    // smooth fields and noise, each with 8 to 128 rows; the rows chosen are within 1.2 % of the best in the mean): a row
    // costs a tenth, more for every block on the CU, by what is read, and more for every round of blocks that the LDS
    // holds; two rows are read beside a segment's own; a block clears and merges its histogram; and blocks of one item meet
    // at its counters, or at the rows that they share.  (One byte a vertex: bound by the march, less by memory.)  Of a batch of small images whose rows leave waves of a block without
    // work the blocks say so themselves: 1867 x 124 x 270 float32 80 us with 32 rows, 137 with 128.
    struct Cost {
      double halo, read, round, block, bins, meet;
    };
    const Cost k = bytes == 1 ? Cost{3.0, 0.05, 0.01, 0.0, 0.1, 0.006} : Cost{2.0, bytes == 2 ? 0.07 : 0.15, 0.085, 0.05, 0.4, 0.0014};
    const size_t ring = ring_bytes2d<float2>();
    const size_t lds = ring + (size_t)bins * (!levels && table_in_lds2d(bins) ? 8 : 4);
    const double resident = (double)std::min<size_t>(5, (size_t)160 * 1024 / lds);
    int64_t best = kChunkRows;
    double least = 0.0;
    unsigned last = 0;
    for (unsigned aim : {8u, 16u, 24u, 32u, 40u, 48u, 56u, 64u, 80u, 96u, 128u}) {  // (32-bit divisions: small calls wait for the host)
      const unsigned segs = ((unsigned)H + aim - 1u) / aim;
      if (segs == last) continue;  // (the same segments)
      const unsigned rows = (((unsigned)H + segs - 1u) / segs + kChunkRows - 1u) / kChunkRows * kChunkRows;
      const int64_t blocks = (nstrip * segs + 3) / 4;
      const double cu = (double)blocks * (double)s.batch / 256.0;
      const double cost = ((double)rows + k.halo) * (0.1 + k.read * std::max(1.0, cu) + k.round * std::ceil(cu / resident)) +
                          cu * (k.block + k.bins * bins / 1024.0) + k.meet * (double)blocks / shared_rows(blocks, bins);
      if (last == 0 || cost < least) {
        least = cost;
        best = aim;
      }
      last = segs;
    }
    return best;
  }
  if (waves(16) <= 1024) return 16;  // at most one wave per SIMD even with short segments
  // Many small images with lists that blocks share (batches beyond the lists per block): four units each as well, rather
  // than one wave of a block's four (8192 x 64^2 215 -> 149 us; 1024 of them, one wave a SIMD, 54 -> 61).
  if (feed == Feed2d::kSharedLists && nstrip == 1 && H <= 64 && tubes > 4096)
    return ((H + 3) / 4 + kChunkRows - 1) / kChunkRows * kChunkRows;
  // One large image gains 30 % from 24 -> 64 rows at 4096^2, 20 % from 16 -> 32 at 2048^2: about 1536 waves, within
  // 32 .. 64 rows per segment.  Shared lists beyond 2^27 vertices: 48 rows where images are up to 34 strips (8432 columns)
  // wide, 4 to 6 % less (16 x 4096^2: 241 / 251 / 237 / 246 / 259 us with 24 / 32 / 48 / 64 / 96 rows, 3 x 8192^2 202 -> 188,
  // 40 x 2048^2 179 -> 169, 5 x 5000 x 7000 180 -> 172); wider ones gain on some fields and lose on others (3 x 7000 x 9000 165 ->
  // 176, 12000^2 170 -> 158).  Up to 2^27 vertices shorter segments gain on smooth fields (16 x 1024^2 float64 79 -> 66 with
  // 24 rows) and lose on white noise, where the blocks contend for the lists (256 x 256^2 float64 1692 -> 2017): not taken.
  const int64_t want = std::max<int64_t>(1, 1536 / tubes);
  int64_t rows = ((H + want - 1) / want + kChunkRows - 1) / kChunkRows * kChunkRows;
  // plenty of tubes (a large batch of small images): up to 128 rows, but two segments per image at least
  // (2048 x 128^2 loses 17 % with one segment of 128)
  int64_t longest = feed == Feed2d::kSharedLists && total > kMidTotal2d && nstrip <= 34 ? 48 : 64;
  if (tubes >= 1024)
    longest = std::max<int64_t>(64, std::min<int64_t>(128, ((H + 1) / 2 + kChunkRows - 1) / kChunkRows * kChunkRows));
  return rows < 32 ? 32 : (rows > longest ? longest : rows);
}

template <typename T>
static Plan2d plan2d(const Shape& s, Feed2d feed, int bins = 1, bool levels = false) {
  Plan2d p;
  const int H = (int)s.H, W = (int)s.W;
  p.nstrip = (W + kStripOut - 1) / kStripOut;
  const int64_t tubes = (int64_t)p.nstrip * s.batch;
  const int64_t aim = rows2d(s, p.nstrip, tubes, feed, (int)sizeof(T), bins, levels);
  int64_t nseg = (H + aim - 1) / aim;
  if (feed == Feed2d::kSigmoid) nseg = std::min(nseg, (32768 + tubes - 1) / tubes);
  if (nseg < 1) nseg = 1;
  // whole chunks per segment; segment + prefetch must stay below 2^31 bytes
  int64_t rows = (H + nseg - 1) / nseg;
  const int64_t gran = kChunkRows;
  rows = (rows + gran - 1) / gran * gran;
  const int64_t row_bytes = (int64_t)W * (int64_t)sizeof(T);
  const int64_t cap = ((((int64_t)1 << 31) / row_bytes - 16) / kChunkRows) * kChunkRows;
  if (rows > cap) rows = cap;
  if (rows > (1 << 20)) rows = 1 << 20;  // (what the sigmoid sinks' queue entries hold)
  p.rows_per_seg = (int)rows;
  p.nseg = (int)((H + p.rows_per_seg - 1) / p.rows_per_seg);
  const int units = p.nstrip * p.nseg;
  p.grid = dim3((unsigned)((units + 3) / 4), (unsigned)s.batch);
  return p;
}
}  // namespace ecc
