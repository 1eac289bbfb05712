// 3D sweep for gfx950 over one- and two-byte element types: the stencil of ecc_sweep3d.h (read that first) with two
// vertices to a register and four rows to a word.
//
// What bounds the tube sweep is the number of vector instructions it issues: 13 relations towards later neighbours, a
// subtraction and a shift each.  Elements of at most 16 bits map, order and all, to signed 16-bit keys, so that
//   - one v_pk_sub_i16 (saturating: the sign is right for any two keys) gives a relation of two rows,
//   - one v_perm_b32, whose selectors 8 .. 11 spread the sign bits of its operands over a byte each, collects the
//     relation of the tube's four rows, and one v_bfi_b32 files it under the plane's bit:
// four instructions for four relations where float32 takes eight.  A word holds a relation of 4 rows (bytes) x 8 planes
// (bits), so a tube's state is 13 words and not 61.  The words of the halo rows above
// and below the tube are formed by the wave itself (16 instructions of 86 a plane); the waves of a block need no barrier.
// Lane-shifted operands cost a move each, as packed subtractions take no DPP modifier: 12 a plane.
//
// A plane of a wave (four rows of 62 columns) takes 86 vector instructions (uint16; three fewer where keys need no flip) and
// about 20 of the Boolean phase, against 117 and 15 of the float32 sweep, through which these types went before.  Dense chunks
// of levels are taken vertex by vertex from the keys still in registers, the coefficients turned into nibbles (about 5
// instructions a vertex where the queue takes 40).  Whole calls, through the float32 sweep and now: 256^3 uint16 noise over 4096
// levels 66.0 -> 37 us (81 -> 39 vector instructions for a row of 62 columns, by the counters), 128^3 uint8 noise 26.3 -> 14.3,
// 193 x 229 x 193 int16 over a known range 35.0 -> 24.8, 256^3 float16 60 -> 37 (three launches instead of five), 512^3 uint16
// smooth 143 -> 134, noise 326 -> 151.  Five waves on a SIMD instead of four change nothing.  By the counters the vector units of
// these launches are at 0.56 (256^3 noise) and 0.42 (193 x 229 x 193) of their peak: segments of eight planes, which fill the chip,
// have about five planes' worth of work besides their own, and a wave's march has few others to overlap with.
#pragma once
#include "ecc_sweep3d.h"

namespace ecc {

namespace s3p {

constexpr int kR = 4;      // rows of a tube = bytes of a word
constexpr int kChunk = 8;  // planes of a chunk = bits of a byte
constexpr int kDenseBits = 6;  // critical vertices of a lane's 32 from which a chunk is taken vertex by vertex

typedef short short2v __attribute__((ext_vector_type(2)));

// q - p of two pairs of keys, saturated
__device__ __forceinline__ unsigned sub(unsigned q, unsigned p) {
  return __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(__builtin_bit_cast(short2v, q),
                                                                    __builtin_bit_cast(short2v, p)));
}
// the same with the low key of p on both sides
__device__ __forceinline__ unsigned sub_low(unsigned q, unsigned p) {
  const short2v v = __builtin_bit_cast(short2v, p);
  return __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(__builtin_bit_cast(short2v, q), (short2v)(v.x)));
}
// signs of (lo.lo, lo.hi, hi.lo, hi.hi) in the four bytes: 0x00 or 0xff
__device__ __forceinline__ unsigned signs(unsigned lo, unsigned hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x0b0a0908u);
}
__device__ __forceinline__ unsigned bfi(unsigned mask, unsigned a, unsigned b) { return (a & mask) | (b & ~mask); }
template <int K> __device__ __forceinline__ unsigned put(unsigned w, unsigned s) { return bfi(0x01010101u << K, s, w); }

// Two elements as signed 16-bit keys in the order of their values; REV: in the reversed order.  (-0.0 and +0.0 get the
// same key.)  level(): the element back from its key, for the integer types.
template <typename T, bool REV> struct Keys;
template <bool REV> struct Keys<uint8_t, REV> {
  static constexpr unsigned kFlip = REV ? 0xffffu : 0u;
  static __device__ __forceinline__ unsigned of(unsigned v) { return v ^ (kFlip << 16 | kFlip); }
};
template <bool REV> struct Keys<int16_t, REV> : Keys<uint8_t, REV> {};
template <bool REV> struct Keys<uint16_t, REV> {
  static constexpr unsigned kFlip = REV ? 0x7fffu : 0x8000u;
  static __device__ __forceinline__ unsigned of(unsigned v) { return v ^ (kFlip << 16 | kFlip); }
};
template <bool REV> struct FloatKeys {
  static constexpr unsigned kFlip = 0u;  // (no levels)
  static __device__ __forceinline__ unsigned of(unsigned v) {  // sign and magnitude to two's complement
    const short2v m = __builtin_bit_cast(short2v, v) >> 15;
    const unsigned mu = __builtin_bit_cast(unsigned, m);
    const short2v k = __builtin_bit_cast(short2v, (v & 0x7fff7fffu) ^ mu) - m;
    return __builtin_bit_cast(unsigned, k) ^ (REV ? 0xffffffffu : 0u);
  }
};
template <bool REV> struct Keys<F16, REV> : FloatKeys<REV> {};
template <bool REV> struct Keys<Bf16, REV> : FloatKeys<REV> {};
// the value of a key of one of the floating types
template <typename T, bool REV> __device__ __forceinline__ float key_value(int k) {
  if (REV) k = ~k;
  const unsigned bits = k < 0 ? (unsigned)(-k) | 0x8000u : (unsigned)k;
  return widen16<T>(bits);
}

// c's four slices to one signed nibble per vertex: nibble q of x[r] is the coefficient of bit 4q + r (two rounds of
// exchanging odd and even fields, 16 instructions for 32 vertices); 0 where valid has no bit
__device__ __forceinline__ void nibbles(const s3::Slices& s, unsigned valid, unsigned (&x)[4]) {
  const unsigned d0 = s.d0 & valid, d1 = s.d1 & valid, d2 = s.d2 & valid, d3 = s.d3 & valid;
  const unsigned m1 = 0x55555555u, m2 = 0x33333333u;
  const unsigned a0 = bfi(m1, d0, d1 << 1), a1 = bfi(m1, d0 >> 1, d1);
  const unsigned b0 = bfi(m1, d2, d3 << 1), b1 = bfi(m1, d2 >> 1, d3);
  x[0] = bfi(m2, a0, b0 << 2);
  x[1] = bfi(m2, a1, b1 << 2);
  x[2] = bfi(m2, a0 >> 2, b0);
  x[3] = bfi(m2, a1 >> 2, b1);
}

// The elements of a lane's six rows of a plane, as loaded
template <typename T> struct Raw {
  unsigned v[kR + 2];
};
template <typename T> __device__ __forceinline__ unsigned load_raw(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s) {
  if constexpr (sizeof(T) == 1) return __builtin_amdgcn_raw_buffer_load_b8(r, v, s, 0);
  else return __builtin_amdgcn_raw_buffer_load_b16(r, v, s, 0);
}

// One tube: columns xs .. xs+63 (outputs xs+1 .. xs+62), output rows yb0 .. yb0+3, output planes z0 .. z1-1.
// SAFE, S, F: as in s3::sweep_tube.  Lanes and rows outside the grid load an element inside it, and the relations that
// involve them are set as the order of the mode has them (so no key has to stand for "beyond the grid").
template <typename T, typename Sink, bool SAFE, typename TiltT>
__device__ __forceinline__ void sweep_tube(const T* __restrict__ g, int D, int H, int W, int xs,
                                           int yb0, int z0, int z1, s3::TubeQueue<Sink>& queue, WaveRange& range,
                                           int S = kWave, int F = 1) {
  using s3::ballot;
  using s3::from_left;
  using s3::from_right;
  constexpr bool REV = TiltT::kNeg;
  typedef Keys<T, REV> Key;
  const int lane = threadIdx.x & (kWave - 1);
  const int fold = SAFE ? lane / S : 0;
  const int xl = SAFE ? lane - fold * S : lane;
  const int x = xs + xl;
  const int yb = yb0 + fold * kR;
  const bool inb = !SAFE || (fold < F && x >= 0 && x < W);
  const bool out_lane = xl >= 1 && xl <= S - 2 && inb;

  const int64_t plane = (int64_t)H * W;
  const unsigned plane_bytes = (unsigned)plane * (unsigned)sizeof(T);
  const unsigned pitch = (unsigned)W * (unsigned)sizeof(T);
  // byte offsets of the six rows from the resource's base: SAFE: a lane's own, from the plane's first element;
  // otherwise the lane's (vb) and the rows' (wave-uniform) from the tube's column 0
  unsigned roff[kR + 2];
#pragma unroll
  for (int j = 0; j <= kR + 1; ++j) {
    if (SAFE)
      roff[j] = ((unsigned)min(max(yb - 1 + j, 0), H - 1) * (unsigned)W + (unsigned)min(max(x, 0), W - 1)) * (unsigned)sizeof(T);
    else
      roff[j] = (unsigned)(yb0 - 1 + j) * pitch;
  }
  const unsigned vb = (unsigned)lane * (unsigned)sizeof(T);
  // The resource is one plane (from the tube's first column); what the pipeline would fetch beyond the last plane that
  // the segment needs is that plane again.  (Counted in 32 bits: 64-bit comparisons take vector instructions.)
  const T* pnext = g + (int64_t)max(z0 - 1, 0) * plane + (SAFE ? 0 : xs);
  int more = min(z1, D - 1) - max(z0 - 1, 0);  // planes after the next one
  auto load_plane = [&](Raw<T>& raw) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(pnext), 0, (int)(plane_bytes - (SAFE ? 0u : (unsigned)xs * (unsigned)sizeof(T))), 0x00020000);
#pragma unroll
    for (int j = 0; j <= kR + 1; ++j)
      raw.v[j] = SAFE ? load_raw<T>(rsrc, roff[j], 0u) : load_raw<T>(rsrc, vb, roff[j]);
    pnext += more > 0 ? plane : 0;
    --more;
  };

  // SAFE: bytes of the rows 1+b .. 4+b inside the grid, and of the halo words' centres and neighbours
  unsigned row_in[3], col_in[3], halo_c12 = 0, halo_q12 = 0, halo_c3 = 0, halo_q3 = 0;
  if (SAFE) {
    unsigned rows = 0;  // bit j: row yb - 1 + j is inside the grid
#pragma unroll
    for (int j = 0; j <= kR + 1; ++j) rows |= (yb - 1 + j >= 0 && yb - 1 + j < H && fold < F) ? 1u << j : 0u;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      row_in[b] = 0;
#pragma unroll
      for (int j = 0; j < kR; ++j) row_in[b] |= (rows >> (j + b) & 1u) ? 0xffu << (8 * j) : 0u;
    }
    const unsigned col = inb ? 0xffffffffu : 0u;
    // (the columns next to this one, from the grid and not from the next lane: a fold's last lane is a halo lane)
#pragma unroll
    for (int a = 0; a < 3; ++a) col_in[a] = (fold < F && x + a - 1 >= 0 && x + a - 1 < W) ? 0xffffffffu : 0u;
    const unsigned r0 = rows & 1u, r1 = rows >> 1 & 1u, r4 = rows >> kR & 1u, r5 = rows >> (kR + 1) & 1u;
    halo_c12 = col & ((r0 ? 0x00ff00ffu : 0u) | (r5 ? 0xff00ff00u : 0u));
    halo_q12 = (r1 ? 0x00ff00ffu : 0u) | (r4 ? 0xff00ff00u : 0u);  // (rows; the columns are applied where it is used)
    halo_c3 = col & (r0 ? 0xffffffffu : 0u);
    halo_q3 = r1 ? 0xffffffffu : 0u;
  }
  // a word of relations with centres inside `c` and neighbours inside `q`: towards a vertex beyond the grid "never
  // before p", from beyond the grid always (top-cell order: the other way round)
  auto inside = [&](unsigned w, unsigned c, unsigned q) { return TiltT::kTop ? c & (w | ~q) : q & (w | ~c); };

  const T* const seg0 = g + (int64_t)z0 * plane;
  auto fetch = [&](unsigned inpl, unsigned zrel, int) { return (float)seg0[zrel * (unsigned)plane + inpl]; };

  // Words.  U[(b+1)*3 + a+1]: towards (x+a, row+b) of the plane above.  Halo words: h1, h2 hold relations of the rows
  // above (0) and below (5) the tube with the plane above -- bytes U(0,+1) of row 0, U(0,-1) of row 5, U(1,+1), U(1,-1);
  // U(-1,+1), U(-1,-1), -, - -- and h3 those of row 0 with row 1 of its own plane: N, NE, NW, -.
  unsigned E = 0, N = 0, NE = 0, NW = 0, U[9], h1 = 0, h2 = 0, h3 = 0;
#pragma unroll
  for (int q = 0; q < 9; ++q) U[q] = 0;
  unsigned cM = 0, cN = 0, cX = 0;  // the current plane: rows (1,2), (3,4), (0,5)
  unsigned En = 0, Nn = 0, NEn = 0, NWn = 0, h3n = 0;
  short2v klo = (short2v)(32767), khi = (short2v)(-32768);

  // Plane u arrives; K: bit of the plane below it (the current one), KI: bit of its own in-plane relations.
  auto arrive = [&](const Raw<T>& raw, auto upward, auto kc) {
    constexpr int K = decltype(kc)::value;
    const unsigned A = Key::of(raw.v[0] | raw.v[1] << 16), B = Key::of(raw.v[2] | raw.v[3] << 16),
                   C = Key::of(raw.v[4] | raw.v[5] << 16);
    const unsigned M = __builtin_amdgcn_alignbit(B, A, 16), Q = __builtin_amdgcn_alignbit(C, B, 16);
    const unsigned X = __builtin_amdgcn_perm(C, A, 0x07060100u), Y = __builtin_amdgcn_perm(Q, M, 0x07060100u);
    const unsigned rA = from_right(A), rB = from_right(B), rC = from_right(C), rM = from_right(M), rQ = from_right(Q),
                   rY = from_right(Y);
    const unsigned lA = from_left(A), lB = from_left(B), lC = from_left(C), lM = from_left(M), lQ = from_left(Q),
                   lY = from_left(Y);
    if constexpr (decltype(upward)::value) {
      U[0] = put<K>(U[0], signs(sub(lA, cM), sub(lB, cN)));
      U[1] = put<K>(U[1], signs(sub(A, cM), sub(B, cN)));
      U[2] = put<K>(U[2], signs(sub(rA, cM), sub(rB, cN)));
      U[3] = put<K>(U[3], signs(sub(lM, cM), sub(lQ, cN)));
      U[4] = put<K>(U[4], signs(sub(M, cM), sub(Q, cN)));
      U[5] = put<K>(U[5], signs(sub(rM, cM), sub(rQ, cN)));
      U[6] = put<K>(U[6], signs(sub(lB, cM), sub(lC, cN)));
      U[7] = put<K>(U[7], signs(sub(B, cM), sub(C, cN)));
      U[8] = put<K>(U[8], signs(sub(rB, cM), sub(rC, cN)));
      h1 = put<K>(h1, signs(sub(Y, cX), sub(rY, cX)));
      const unsigned dl = sub(lY, cX);
      h2 = put<K>(h2, signs(dl, dl));
    }
    const unsigned sE = signs(sub(rM, M), sub(rQ, Q)), sN = signs(sub(B, M), sub(C, Q)),
                   sNE = signs(sub(rB, M), sub(rC, Q)), sNW = signs(sub(lB, M), sub(lC, Q));
    const unsigned side = __builtin_amdgcn_perm(lY, rY, 0x05040100u);  // row 1 of the columns to the right and left
    const unsigned s3w = signs(sub_low(Y, X), sub_low(side, X)) ;      // N, -, NE, NW
    if constexpr (K + 1 < kChunk) {
      E = put<(K + 1) & 7>(E, sE);
      N = put<(K + 1) & 7>(N, sN);
      NE = put<(K + 1) & 7>(NE, sNE);
      NW = put<(K + 1) & 7>(NW, sNW);
      h3 = put<(K + 1) & 7>(h3, s3w);
    } else {  // the first plane of the next chunk
      En = sE;
      Nn = sN;
      NEn = sNE;
      NWn = sNW;
      h3n = s3w;
    }
    cM = M;
    cN = Q;
    cX = X;
  };
  // the nine words of the plane above, as seen by the neighbour they point to (rows, then lanes, shifted)
  auto seen_from_above = [&](unsigned (&d)[9]) {
    d[0] = from_right(U[3]);                                           // E
    d[1] = from_right(__builtin_amdgcn_perm(U[0], h2, 0x01070605u));   // NE: row + 1 towards (-1, -1)
    d[2] = __builtin_amdgcn_perm(U[1], h1, 0x01070605u);               // N
    d[3] = from_left(__builtin_amdgcn_perm(U[2], h1, 0x03070605u));    // NW
    d[4] = from_left(U[5]);                                            // W
    d[5] = from_left(__builtin_amdgcn_perm(U[8], h1, 0x06050402u));    // SW: row - 1 towards (1, 1)
    d[6] = __builtin_amdgcn_perm(U[7], h1, 0x06050400u);               // S
    d[7] = from_right(__builtin_amdgcn_perm(U[6], h2, 0x06050400u));   // SE
    d[8] = U[4];
  };
  auto keep_inside_up = [&]() {
    const unsigned c = row_in[1] & col_in[1];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int a = 0; a < 3; ++a) U[b * 3 + a] = inside(U[b * 3 + a], c, row_in[b] & col_in[a]);
    h1 = inside(h1, halo_c12, halo_q12 & bfi(0x0000ffffu, col_in[1], col_in[2]));
    h2 = inside(h2, halo_c12, halo_q12 & col_in[0]);
  };

  typedef std::integral_constant<int, kChunk - 1> Last;
  unsigned carry[9];  // bit 0 of every byte: the plane below the chunk, as seen by its upper neighbours
#pragma unroll
  for (int q = 0; q < 9; ++q) carry[q] = TiltT::kTop ? 0u : 0xffffffffu;  // below the grid: "never before p" once complemented
  Raw<T> rawx, rawy;
  {
    Raw<T> r0;
    load_plane(r0);
    load_plane(rawx);
    load_plane(rawy);
    arrive(r0, std::false_type(), Last());
    if (z0 > 0) {  // r0 was plane z0 - 1; plane z0 follows
      arrive(rawx, std::true_type(), Last());
      if (SAFE) keep_inside_up();
      unsigned d[9];
      seen_from_above(d);
#pragma unroll
      for (int q = 0; q < 9; ++q) carry[q] = d[q] >> 7;
      rawx = rawy;
      load_plane(rawy);
    }
  }
  // now the current plane is z0; rawx = plane z0+1, rawy = plane z0+2 (in flight)
  E = En;
  N = Nn;
  NE = NEn;
  NW = NWn;
  h3 = h3n;
  for (int z = z0; z < z1; z += kChunk) {
    const int n = min(kChunk, z1 - z);
    unsigned kept[kChunk][2];  // keys of the chunk's vertices (dense chunks of levels)
    auto step = [&](auto kc) {
      constexpr int K = decltype(kc)::value;
      if constexpr (Sink::kDense) {
        kept[K][0] = cM;
        kept[K][1] = cN;
      }
      if (Sink::kTrackRange) {  // (halo lanes and rows beyond the grid hold vertices of the grid too)
        klo = __builtin_elementwise_min(klo, __builtin_elementwise_min(__builtin_bit_cast(short2v, cM), __builtin_bit_cast(short2v, cN)));
        khi = __builtin_elementwise_max(khi, __builtin_elementwise_max(__builtin_bit_cast(short2v, cM), __builtin_bit_cast(short2v, cN)));
      }
      Raw<T>& raw = (K & 1) ? rawy : rawx;
      const Raw<T> now = raw;
      load_plane(raw);
      arrive(now, std::true_type(), kc);
    };
    // (a chunk of fewer planes is the segment's last: the bits of the others mean nothing and are masked)
    do {
      step(std::integral_constant<int, 0>());
      if (n <= 1) break;
      step(std::integral_constant<int, 1>());
      if (n <= 2) break;
      step(std::integral_constant<int, 2>());
      if (n <= 3) break;
      step(std::integral_constant<int, 3>());
      if (n <= 4) break;
      step(std::integral_constant<int, 4>());
      if (n <= 5) break;
      step(std::integral_constant<int, 5>());
      if (n <= 6) break;
      step(std::integral_constant<int, 6>());
      if (n <= 7) break;
      step(std::integral_constant<int, 7>());
    } while (false);
    if (SAFE) {
      const unsigned c = row_in[1] & col_in[1];
      keep_inside_up();
      E = inside(E, c, row_in[1] & col_in[2]);
      N = inside(N, c, row_in[2] & col_in[1]);
      NE = inside(NE, c, row_in[2] & col_in[2]);
      NW = inside(NW, c, row_in[2] & col_in[0]);
      h3 = inside(h3, halo_c3, halo_q3 & bfi(0x0000ffffu, col_in[1], bfi(0x00ff0000u, col_in[2], col_in[0])));
    }
    if (z + n >= D) {  // the grid's last plane has nothing above it
      const unsigned bit = 0x01010101u << (n - 1);
#pragma unroll
      for (int q = 0; q < 9; ++q) U[q] = TiltT::kTop ? (U[q] | bit) : (U[q] & ~bit);
    }
    const unsigned planes = (0xffu >> (kChunk - n)) * 0x01010101u;

    unsigned a[8], mu[8], md[8], d[9];
    a[0] = E;
    a[1] = NE;
    a[2] = N;
    a[3] = NW;
    a[4] = ~from_left(E);
    a[5] = ~from_left(__builtin_amdgcn_perm(NE, h3, 0x06050402u));
    a[6] = ~__builtin_amdgcn_perm(N, h3, 0x06050400u);
    a[7] = ~from_right(__builtin_amdgcn_perm(NW, h3, 0x06050403u));
    mu[0] = a[0] & U[5];
    mu[1] = a[1] & U[8];
    mu[2] = a[2] & U[7];
    mu[3] = a[3] & U[6];
    mu[4] = a[4] & U[3];
    mu[5] = a[5] & U[0];
    mu[6] = a[6] & U[1];
    mu[7] = a[7] & U[2];
    const unsigned up0 = U[4];
    seen_from_above(d);
    unsigned below[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      below[q] = bfi(0xfefefefeu, d[q] << 1, carry[q]);
      carry[q] = d[q] >> 7;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) md[q] = a[q] & ~below[q];
    const unsigned dn0 = ~below[8];

    unsigned s[8], t[6];
    s3::arc_starts(mu, up0, &s[0]);
    s3::arc_starts(md, dn0, &s[4]);
    s3::arc_starts(a, 0xffffffffu, &t[0]);
    t[4] = up0;
    t[5] = dn0;
    s3::Slices sl;
    const unsigned valid = out_lane ? (SAFE ? planes & row_in[1] : planes) : 0u;
    unsigned nz = s3::count_pq(s, t, sl) & valid;
    E = En;
    N = Nn;
    NE = NEn;
    NW = NWn;
    h3 = h3n;
    if constexpr (Sink::kDense) {
      if (ballot(__builtin_popcount(nz) >= kDenseBits)) {  // (wave-uniform)
        unsigned cn[4];
        nibbles(sl, valid, cn);
#pragma unroll
        for (int k = 0; k < kChunk; ++k) {
#pragma unroll
          for (int j = 0; j < kR; ++j) {
            const int c = __builtin_amdgcn_sbfe((int)cn[k & 3], 4 * (2 * j + (k >> 2)), 4);
            const unsigned v = (j & 1 ? kept[k][j >> 1] >> 16 : kept[k][j >> 1] & 0xffffu) ^ Key::kFlip;
            queue.sink.add_level(v, TiltT::kTop ? -c : c);
          }
        }
        continue;
      }
    }
    const unsigned inpl0 = (unsigned)(yb * W + x);
    while (ballot(nz != 0)) {
      const bool active = nz != 0;
      const int b = active ? 31 - __clz(nz) : 0;
      nz &= ~(1u << b);
      const unsigned cu = ((sl.d0 >> b) & 1u) | (((sl.d1 >> b) & 1u) << 1) | (((sl.d2 >> b) & 1u) << 2) |
                          (((sl.d3 >> b) & 1u) << 3);
      const int c = (int)(cu ^ 8u) - 8;
      // top cells: (-1)^3 times the vertex coefficient
      queue.template push<false>(active, inpl0 + (unsigned)(b >> 3) * (unsigned)W, (unsigned)(z - z0 + (b & 7)),
                                 TiltT::kTop ? -c : c, 0.f, fetch);
    }
  }
  if constexpr (Sink::kTrackRange) {
    const int lo = min((int)klo.x, (int)klo.y), hi = max((int)khi.x, (int)khi.y);
    range.add(key_value<T, REV>(lo));
    range.add(key_value<T, REV>(hi));
  }
  queue.flush(fetch);
}

}  // namespace s3p

// Work unit of a wave: as in sweep3d_wave (row groups of four, strips of 62 columns, a narrow last strip folded).
template <typename T, typename Sink, typename TiltT>
__device__ __forceinline__ void sweep3dp_wave(const T* __restrict__ g, int D, int H, int W,
                                              const Tiling3& tl, int nseg, int planes_per_seg, s3::TubeQueue<Sink>& queue, WaveRange& range) {
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  int seg, strip, group;
  bool tail, active;
  decode_unit3(tl, unit, seg, strip, group, tail, active);
  if (!active || seg >= nseg) return;
  const int z0 = seg * planes_per_seg, z1 = min(z0 + planes_per_seg, D);
  const int xs = strip * s3::kOut - 1, yb = group * s3p::kR;
  const bool safe = tail || (xs < 0) || (xs + kWave > W) || (yb == 0) || (yb + s3p::kR + 1 > H);
  if (safe)
    s3p::sweep_tube<T, Sink, true, TiltT>(g, D, H, W, xs, yb, z0, z1, queue, range, tail ? tl.S : kWave,
                                          tail ? tl.F : 1);
  else
    s3p::sweep_tube<T, Sink, false, TiltT>(g, D, H, W, xs, yb, z0, z1, queue, range);
}

}  // namespace ecc
