// Soft ECC: evaluation of a drained batch of critical vertices against the thresholds, shared by the sinks of
// the strip (2D) and the tube (3D) sweep.
//
// A wave calls it with up to 64 entries, threshold-major: lane l takes the thresholds l, l + 64, ..., some slots of 64 at
// a time, and runs over the entries, so that the sums over p of Eq. 6 / Eq. 9 / Eq. 10 of the paper need no
// cross-lane reduction; the contraction of Eq. 8 with the upstream gradient is a fixed-order sum over the lanes.
//
// The running sums live in the unit's own row of partial sums in the workspace and not in registers: a batch's sums
// (formed from zero: shorter chains of float32 additions) are added to them (the first batch of a unit starts the row;
// most units have one or two).  Registers held across the sweep were what limited it: sums, thresholds and upstream
// gradient of four thresholds a lane took the 3D kernels from 124 to 162 .. 204 vector registers (three or two waves on a
// SIMD instead of four) and tied the path to 256 thresholds.  256^3 with 64 thresholds: forward 42.6 -> 38.6 us, backward
// 73.8 -> 50.3 us.
//
// Eq. 8's sum over the lanes takes four entries together: two exchange steps interleave them over the lanes of a quad, so
// that the other four steps serve all four at once (12 additions instead of 24; backward pass of 32 x 512^2, T = 64:
// 35.9 -> 31.0 us).
#pragma once
#include "ecc_device.h"

namespace ecc {

struct StagedValue {
  double y;  // packed, see SoftArg
  float c;
};

// NC: coordinates; CHI / DERIV: which sums a row holds, {chi} {A0, A_1 .. A_NC} in this order, STRIDE floats a
// threshold; GRADX: the contraction with the upstream gradient; WIDE: see SoftArg
template <int NC, bool CHI, bool DERIV, bool GRADX, int STRIDE, bool WIDE>
struct SoftEval {
  typedef SoftArg<WIDE> Arg;
  static constexpr int kA = CHI ? 1 : 0, kSums = kA + (DERIV ? 1 + NC : 0);
  const float* tau;
  const float* gup;  // this item's upstream gradient, or null for all ones
  float* row;        // this unit's sums, or null
  int T;
  float kneg;
  bool started;      // the row holds sums

  __device__ __forceinline__ void init(const float* tau_, int T_, float kneg_, const float* gup_, float* row_) {
    tau = tau_;
    T = T_;
    kneg = kneg_;
    gup = gup_;
    row = row_;
    started = false;
  }
  __device__ __forceinline__ void store(int j, const float (&a)[kSums > 0 ? kSums : 1]) const {
    float* p = row + (int64_t)j * STRIDE;
    if constexpr (STRIDE == 4) {
      *reinterpret_cast<float4*>(p) = make_float4(a[0], kSums > 1 ? a[kSums > 1 ? 1 : 0] : 0.f,
                                                  kSums > 2 ? a[kSums > 2 ? 2 : 0] : 0.f,
                                                  kSums > 3 ? a[kSums > 3 ? 3 : 0] : 0.f);
    } else {
#pragma unroll
      for (int k = 0; k < kSums; ++k) p[k] = a[k];
      if constexpr (kSums < STRIDE) {
#pragma unroll
        for (int k = kSums; k < STRIDE; ++k) p[k] = 0.f;
      }
    }
  }
  // S slots of 64 thresholds from slot t0 on; get(e, v, r): value and coordinates (relative to the unit's origin)
  // of entry e; returns the lanes' share: lane e < n holds its entry's contraction over these slots
  template <int S, typename Get>
  __device__ __forceinline__ float slots(int t0, int n, float csat, const Get& get) const {
    const int lane = threadIdx.x & (kWave - 1);
    typename Arg::Tau tj[S];
    float gj[S], acc[S][kSums > 0 ? kSums : 1];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int j = lane + kWave * (t0 + s);
      const bool ok = j < T;
      tj[s] = ok ? tau[j] : 0.0f;
      if (GRADX) gj[s] = ok ? (gup ? gup[j] : 1.0f) : 0.0f;
#pragma unroll
      for (int k = 0; k < kSums; ++k) {
        acc[s][k] = 0.0f;
      }
    }
    float mine = 0.0f;
    auto entry = [&](int e, bool valid) -> float {
      StagedValue v;
      float r[NC];
      get(e, v, r);
      if (GRADX && !valid) v.c = 0.0f;
      float gd = 0.0f;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float ex = soft_exp_neg(Arg::z(tj[s], v.y), kneg);
        const float sg = __builtin_amdgcn_rcpf(1.0f + ex);
        if constexpr (CHI) acc[s][0] += v.c * sg;
        if constexpr (DERIV || GRADX) {
          const float d = ex * sg * sg;  // sigma (1 - sigma)
          if constexpr (DERIV) {
            const float cd = v.c * d;
            acc[s][kA] += cd;
#pragma unroll
            for (int k = 0; k < NC; ++k) acc[s][kA + 1 + k] += cd * r[k];
          }
          if constexpr (GRADX) gd += gj[s] * d;
        }
      }
      return gd;
    };
    if constexpr (GRADX) {
      for (int e = 0; e < n; e += 4) {
        float g[4];  // (beyond the last entry: that one again with c = 0, its sum not used)
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = entry(min(e + q, n - 1), e + q < n);
        // lane l ends with entry e + (l & 3) summed over all lanes
        const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0;
        const float r01 = (b0 ? g[1] : g[0]) + dpp_move<0xB1, 0xf>(b0 ? g[0] : g[1]);
        const float r23 = (b0 ? g[3] : g[2]) + dpp_move<0xB1, 0xf>(b0 ? g[2] : g[3]);
        float r = (b1 ? r23 : r01) + dpp_move<0x4E, 0xf>(b1 ? r01 : r23);
        r += dpp_move<0x124, 0xf>(r);  // row_ror:4
        r += dpp_move<0x128, 0xf>(r);  // row_ror:8
        r = swap_add16(r);
        r = swap_add32(r);
        if ((lane & ~3) == e) mine += r;
      }
    } else {
      for (int e = 0; e < n; ++e) entry(e, true);
    }
    if (row) {  // wave-uniform
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int j = lane + kWave * (t0 + s);
#pragma unroll
        for (int k = 0; k < kSums; ++k) {
          float old = (started && j < T) ? row[(int64_t)j * STRIDE + k] : 0.0f;
          if (CHI && k == 0) old += csat;
          acc[s][k] += old;
        }
        if (j < T) store(j, acc[s]);
      }
    }
    return mine;
  }
  // SLOTS: slots taken together at most (they share the reads of an entry; one where registers are short)
  template <int SLOTS, typename Get>
  __device__ __forceinline__ float run(int n, float csat, const Get& get) {
    const int nt = (T + kWave - 1) / kWave;
    float mine = 0.0f;
    int t = 0;
    if constexpr (SLOTS >= 4)
      for (; t + 4 <= nt; t += 4) mine += slots<4>(t, n, csat, get);
    if constexpr (SLOTS >= 2)
      for (; t + 2 <= nt; t += 2) mine += slots<2>(t, n, csat, get);
    for (; t < nt; ++t) mine += slots<1>(t, n, csat, get);
    started = true;
    return mine;
  }
  // a unit without entries leaves zeros
  __device__ __forceinline__ void finish() const {
    if (!row || started) return;  // wave-uniform
    const float zero[kSums > 0 ? kSums : 1] = {};
    for (int j = threadIdx.x & (kWave - 1); j < T; j += kWave) store(j, zero);
  }
};

// A launch with few wave units (small batches, small grids) and many thresholds is as long as one wave's walk over
// its thresholds while most of the chip idles.  Such a launch runs in layers of blocks (gridDim.z): every
// layer sweeps the grid again, which is cheap then, and evaluates its own share of the thresholds, a multiple of 64.
// Up to about three waves for each of the 1024 SIMDs (most_waves); for volumes, whose sweep is the larger part of the
// call, half of that up to 256 thresholds (256 x 12^3, T = 192: 22.5 us in three layers, 16.2 in one).  No layers where a
// contraction over all thresholds is formed.
// Forward pass with derivatives on 16 x 217 x 181 with 512 thresholds: 91 us in one layer of 224 waves, 21 us in four
// layers of 448 (8 rows a wave instead of 16).
static inline unsigned soft_layers(int64_t waves, int T, int64_t most_waves = 3072) {
  const int64_t slots = (T + kWave - 1) / kWave;
  int64_t n = most_waves / (waves < 1 ? 1 : waves);
  n = n < 1 ? 1 : (n > slots ? slots : n);
  const int64_t per = (slots + n - 1) / n;
  return (unsigned)((slots + per - 1) / per);
}
// first threshold and number of thresholds of a layer
__device__ __forceinline__ void soft_layer(int T, int& j0, int& n) {
  const int slots = (T + kWave - 1) / kWave, per = (slots + (int)gridDim.z - 1) / (int)gridDim.z * kWave;
  j0 = min((int)blockIdx.z * per, T);
  n = min(per, T - j0);
}

// least and greatest threshold, by the whole wave
__device__ __forceinline__ void threshold_span(const float* tau, int T, float& lo, float& hi) {
  lo = INFINITY;
  hi = -INFINITY;
  for (int j = threadIdx.x & (kWave - 1); j < T; j += kWave) {
    const float t = tau[j];
    lo = fminf(lo, t);
    hi = fmaxf(hi, t);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fminf(lo, __shfl_xor(lo, o));
    hi = fmaxf(hi, __shfl_xor(hi, o));
  }
}

// Lanes with `keep` get consecutive positions; *csat receives the sum of c over the lanes with `ones` (dropped
// entries whose sigmoids are all 1).  Returns the number of kept entries, `pos` the lane's position.
__device__ __forceinline__ int pack_entries(bool keep, bool ones, float c, int n, float& csat, int& pos) {
  const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
  const int kept = __builtin_popcountll(m);
  csat = 0.0f;
  if (kept != n) {  // wave-uniform
    const float sum = wave_sum_lane63(ones ? c : 0.0f);
    csat = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sum), kWave - 1));
  }
  pos = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
  return kept;
}

}  // namespace ecc
