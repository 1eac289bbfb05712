// Soft single-direction ECC for 2D grids, fused into the strip sweep of
// ecc_sweep2d.h: forward (Eq. 6 of the paper) and derivatives (Eq. 8-10).
//
// Every term of Eq. 6 / Eq. 8-10 carries the integer factor c(p), so only the
// critical vertices (c != 0) contribute.  The sweep finds them with the
// bit-sliced stencil and hands them to this file's sinks 64 at a time, straight
// from the wave's LDS queue.  A sink evaluates the sigmoid on entries x
// thresholds pairs only:
//   - threshold-major: lane l owns thresholds tau_l, tau_{l+64}, ... and runs over
//     the entries (LDS broadcast reads): the sums over p of Eq. 6 / Eq. 9 / Eq. 10
//     need no cross-lane reduction;
//   - backward: the same pass also forms, per entry, the contraction of Eq. 8 with
//     the upstream gradient as a fixed-order sum over the lanes (grad_X);
// see ecc_soft_eval.h.
// grad_X is zero away from critical vertices; the sweep writes those zeros row
// by row for the vertices it owns, before any entry of those rows is drained
// (measured a little quicker than a fill kernel in front of the sweep).
// Each wave keeps its partial sums in a row of the workspace; a second kernel adds the
// rows in a fixed order in float64, so results are run-to-run identical.
//
// y = X(p) + alpha <u,p> and z = tau_j - y are formed in float64 and z is rounded once (two float32 subtractions of y
// carried as two floats round twice; a float64 one and its conversion cost 1 to 2 % of these kernels); exp2 and the
// reciprocal run on the float32 transcendental unit.  An entry whose y lies so far outside
// [min tau, max tau] that every sigmoid is 0 or 1 (see soft_sat_bounds) is not evaluated at all: it adds
// c to every threshold (sigma = 1) or nothing, and nothing to the derivatives.
#include "ecc_sweep2d.h"
#include "ecc_soft_eval.h"
#include "ecc_soft_saved.h"
#include "ecc_soft_reduce.h"

namespace ecc {

// What the queue holds per critical vertex: the value and its place, eight bytes, so that rings, queues and the
// stages below take 40 KB a block and four blocks fit a CU (44 KB and three with y formed as a vertex is queued).
struct SoftEntry {
  float v;       // value the sweep ran on
  unsigned rel;  // row - row0 << 12 | column - col0 << 4 | c & 15
};
struct SoftStaged {
  double y;  // X(p) + alpha <u,p>, packed (see SoftArg)
  float c;
  unsigned rel;
};

// CHI / DERIV / GRADX: what is formed (see ecc_soft_eval.h); SAVE: every entry is also appended to the unit's list
// in the state buffer.  ZERO: the sweep clears grad_X row by row.
template <bool CHI, bool DERIV, bool GRADX, bool SAVE, int STRIDE, bool WIDE>
struct SoftSink {
  typedef SoftEntry Entry;
  static constexpr bool kTrackRange = false;
  static constexpr bool kZeroFill = GRADX;
  double ux, uy, alpha;
  float sat_lo, sat_hi;  // y <= sat_lo: every sigma is 1;  y >= sat_hi: every sigma is 0 (soft_sat_bounds)
  // The sweep ran on the tilted field (c of the tilted field): the value it hands over
  // is the tilted one in float32; X is read again so that y is formed as always.
  const float* xsrc;  // this item's grid, or null when the sweep ran on X itself
  int W;
  int col0, row0;     // origin of the wave's unit: coordinates are summed relative to it
  SoftStaged* stage;  // wave-private LDS, 64 entries
  SoftEval<2, CHI, DERIV, GRADX, STRIDE, WIDE> eval;
  float* gx;          // GRADX: grad_X of this item or null
  float lambda;
  SavedEntry* list;     // SAVE: this unit's list
  unsigned cap, saved;  // saved: entries seen so far (wave-uniform; may pass cap)

  __device__ __forceinline__ Entry make(float v, int c, int col, int row) const {
    Entry e;
    e.v = v;
    e.rel = ((unsigned)(row - row0) << 12) | ((unsigned)(col - col0) << 4) | ((unsigned)c & 15u);
    return e;
  }
  template <bool EDGE>
  __device__ __forceinline__ void zero_row(int row, int col, const bool (&ok)[kNC], bool out_lane) const {
    if (!gx || !out_lane) return;
    float* p = gx + (int64_t)row * W + col;
    if (!EDGE) {
      typedef float Four __attribute__((ext_vector_type(4), aligned(4)));  // (one store at any row alignment)
      *reinterpret_cast<Four*>(p) = Four{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
      for (int e = 0; e < kNC; ++e)
        if (ok[e]) p[e] = 0.f;
    }
  }
  __device__ __forceinline__ void consume(const Entry* buf, int n) {
    const int lane = threadIdx.x & (kWave - 1);
    const bool in = lane < n;
    const Entry q = buf[in ? lane : 0];
    const int col = col0 + (int)((q.rel >> 4) & 255u), row = row0 + (int)(q.rel >> 12);
    const int ci = (int)(q.rel << 28) >> 28;
    float v = q.v;
    if (xsrc) v = xsrc[(int64_t)row * W + col];  // wave-uniform condition
    const double y = (double)v + alpha * (ux * (double)col + uy * (double)row);
    SoftStaged e;
    e.y = SoftArg<WIDE>::pack(y);
    e.c = (float)ci;
    e.rel = q.rel;
    if constexpr (SAVE) {
      if (in && saved + (unsigned)lane < cap) {
        SavedEntry o;
        o.y = y;
        o.idx = row * W + col;
        o.c = ci;
        list[saved + lane] = o;
      }
      saved += (unsigned)n;
    }
    float csat;
    int pos;
    const float yf = (float)y;
    const bool keep = in && yf > sat_lo && yf < sat_hi;
    n = pack_entries(keep, in && yf <= sat_lo, e.c, n, csat, pos);
    if (keep) stage[pos] = e;
    if (!CHI) csat = 0.0f;  // (grad_X stays 0 at a saturated vertex)
    if (n == 0 && csat == 0.0f) return;
    const SoftStaged* st = stage;
    const float g = eval.template run<2>(n, csat, [st](int i, StagedValue& o, float (&r)[2]) {
      const SoftStaged s = st[i];
      o.y = s.y;
      o.c = s.c;
      r[0] = (float)((s.rel >> 4) & 255u);
      r[1] = (float)(s.rel >> 12);
    });
    if constexpr (GRADX) {
      if (gx && lane < n) {
        const SoftStaged s = stage[lane];
        gx[(int64_t)(row0 + (int)(s.rel >> 12)) * W + col0 + (int)((s.rel >> 4) & 255u)] = -lambda * s.c * g;
      }
    }
  }
};

static unsigned state_cap(const Plan2d& pl) {
  // room for one vertex in eight of a unit's rows x 248 columns; 64 more for the units of 8 rows that small launches
  // take (a small unit's share varies; there are 3072 of them at most)
  const unsigned v = (unsigned)pl.rows_per_seg * (unsigned)kStripOut / 8u;
  return pl.rows_per_seg == 8 && pl.nseg > 1 ? v + 64u : v;
}
size_t soft2d_state_bytes(const Shape& s) {
  if (!soft2d_supported(s, 1)) return 256;
  const Plan2d pl = plan2d<float>(s, Feed2d::kSigmoid);
  return state_bytes(s.batch, (size_t)pl.nstrip * pl.nseg, state_cap(pl));
}

// LDS: [4 waves] value rings, then [4 waves] queues of SoftEntry, then [4 waves] stages
constexpr size_t kSoftLds = ring_bytes2d<SoftEntry>() + (size_t)4 * kWave * sizeof(SoftStaged);

// The sweep of a wave with sink `queue.sink`, whose own fields the kernels below have set; partial (may be null):
// rows of STRIDE floats a threshold, one row a unit.  TILTC: the sweep runs on the tilted field, so c(p) is that
// field's coefficient.
template <bool TILTC, int STRIDE, typename Sink>
__device__ __forceinline__ void soft2d_sweep(WaveQueue<Sink>& queue, const float* __restrict__ grid, int H, int W,
                                             int64_t N, int nstrip, int nseg, int rows_per_seg, const float* u,
                                             float alpha, const float* tau, int T, float kneg, const float* gup,
                                             float* partial) {
  extern __shared__ int smem[];
  const int wv = threadIdx.x >> 6;
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(wv), units = nstrip * nseg;
  float* ring = reinterpret_cast<float*>(smem) + wv * (kChunkRows * kWave * kNC);
  SoftEntry* qbuf = reinterpret_cast<SoftEntry*>(smem + 4 * kChunkRows * kWave * kNC);
  queue.buf = qbuf + wv * kQueueCap;
  queue.count = 0;
  Sink& s = queue.sink;
  s.stage = reinterpret_cast<SoftStaged*>(qbuf + 4 * kQueueCap) + wv * kWave;
  s.ux = (double)u[0];
  s.uy = (double)u[1];
  s.alpha = (double)alpha;
  float lo, hi;
  threshold_span(tau, T, lo, hi);
  soft_sat_bounds(lo, hi, kneg, T, s.sat_lo, s.sat_hi);
  s.W = W;
  s.col0 = (unit % nstrip) * kStripOut - kNC;
  s.row0 = (unit / nstrip) * rows_per_seg;
  const bool on = unit < units;
  int j0, nj;
  soft_layer(T, j0, nj);
  s.eval.init(tau + j0, nj, kneg, gup ? gup + (int64_t)blockIdx.y * T + j0 : nullptr,
              on && partial ? partial + (((int64_t)blockIdx.y * units + unit) * (int64_t)T + j0) * STRIDE : nullptr);
  const float* g = grid + (int64_t)blockIdx.y * N;
  s.xsrc = TILTC ? g : nullptr;
  WaveRange range;
  if constexpr (TILTC) {
    const DirArgs da = {u, alpha, 1, 2};
    sweep2d_wave<float>(g, H, W, N, nstrip, nseg, rows_per_seg, queue, ring, range, load_tilt(da, 0));
  } else {
    sweep2d_wave<float>(g, H, W, N, nstrip, nseg, rows_per_seg, queue, ring, range, NoTilt());
  }
  s.eval.finish();
}

// partial[(item * units + unit) * T + j]
template <bool TILTC, bool WIDE>
__global__ __launch_bounds__(256, 4) void soft2d_fwd_kernel(const float* __restrict__ grid, int H, int W,
                                                         int64_t N, int nstrip, int nseg, int rows_per_seg,
                                                         const float* __restrict__ u, float alpha,
                                                         const float* __restrict__ tau, int T, float kneg,
                                                         float* __restrict__ partial) {
  WaveQueue<SoftSink<true, false, false, false, 1, WIDE>> queue;
  soft2d_sweep<TILTC, 1>(queue, grid, H, W, N, nstrip, nseg, rows_per_seg, u, alpha, tau, T, kneg, nullptr, partial);
}

// partial[((item * units + unit) * T + j) * 4 + {0: A0, 1: Ax, 2: Ay}]
template <bool TILTC, bool WIDE>
__global__ __launch_bounds__(256, 4) void soft2d_bwd_kernel(const float* __restrict__ grid, int H, int W,
                                                         int64_t N, int nstrip, int nseg, int rows_per_seg,
                                                         const float* __restrict__ u, float alpha,
                                                         const float* __restrict__ tau, int T, float kneg,
                                                         float lambda, const float* __restrict__ gup,
                                                         float* __restrict__ grad_X,
                                                         float* __restrict__ partial) {
  WaveQueue<SoftSink<false, true, true, false, 4, WIDE>> queue;
  queue.sink.gx = grad_X ? grad_X + (int64_t)blockIdx.y * N : nullptr;
  queue.sink.lambda = lambda;
  soft2d_sweep<TILTC, 4>(queue, grid, H, W, N, nstrip, nseg, rows_per_seg, u, alpha, tau, T, kneg, gup, partial);
}

// Forward pass that saves its critical vertices: chi as soft2d_fwd_kernel, with DERIV the sums of Eq. 9 / Eq. 10 in
// the same pass (they share the sigmoid), and every entry appended to the unit's own list in the state buffer.
// partial[((item * units + unit) * T + j) * 4 + {0: chi, 1: A0, 2: Ax, 3: Ay}]
template <bool TILTC, bool DERIV, bool WIDE>
__global__ __launch_bounds__(256, 4) void soft2d_fwd_save_kernel(const float* __restrict__ grid, int H, int W, int64_t N,
                                                              int nstrip, int nseg, int rows_per_seg,
                                                              const float* __restrict__ u, float alpha,
                                                              const float* __restrict__ tau, int T, float kneg,
                                                              float* __restrict__ partial, StateView sv, unsigned cap) {
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), units = nstrip * nseg;
  WaveQueue<SoftSink<true, DERIV, false, true, 4, WIDE>> queue;
  queue.sink.cap = blockIdx.z == 0 ? cap : 0u;  // (the first layer keeps the list)
  queue.sink.saved = 0u;
  queue.sink.list = sv.lists + ((size_t)blockIdx.y * units + (unit < units ? unit : 0)) * cap;
  const unsigned next_gen = *sv.gen + 1u;  // (the reduction kernel that follows stores it)
  soft2d_sweep<TILTC, 4>(queue, grid, H, W, N, nstrip, nseg, rows_per_seg, u, alpha, tau, T, kneg, nullptr, partial);
  if (unit < units && blockIdx.z == 0 && (threadIdx.x & (kWave - 1)) == 0) {
    sv.counts[(size_t)blockIdx.y * units + unit] = queue.sink.saved;
    if (queue.sink.saved > cap) sv.overflow[blockIdx.y] = next_gen;
  }
}

// origin of a unit's coordinates, for the reduction of ecc_soft_reduce.h
struct Origin2 {
  int nstrip, rows_per_seg;
  __device__ __forceinline__ void operator()(int unit, int (&o)[3]) const {
    o[0] = (unit % nstrip) * kStripOut - kNC;
    o[1] = (unit / nstrip) * rows_per_seg;
    o[2] = 0;
  }
};

// grad_X from the saved lists (Eq. 8 contracted with the upstream gradient).  A block takes one
// unit of the forward sweep.  It clears the part of grad_X the unit owns (its rows x its 248
// output columns), then goes through the unit's list 256 entries at a time: entries whose
// sigmoids are all saturated are dropped (grad_X stays 0 there, see soft_sat_bounds), the others
// are packed into an LDS stage and get eight lanes each -- every lane sums an eighth of the
// thresholds, three lane swaps add the eight partial sums.  A unit's work is spread over four
// waves because the lists are uneven: with a tilt, whole regions of the image are saturated and
// the call lasts as long as its busiest unit.
// An item whose lists cannot be used (header of another shape, a unit ran out of room) is
// computed from the grid instead, vertex by vertex with the plain stencil: slow, but rare.
template <bool TILTC, bool WIDE>
__global__ __launch_bounds__(256) void soft2d_bwd_saved_kernel(const float* __restrict__ grid, int H, int W, int64_t N,
                                                               int nstrip, int nseg, int rows_per_seg,
                                                               const float* __restrict__ u, float alpha,
                                                               const float* __restrict__ tau, int T, float kneg,
                                                               float lambda, const float* __restrict__ gup,
                                                               float* __restrict__ grad_X, StateView sv,
                                                               SoftStateHeader expect) {
  const int item = blockIdx.y, unit = blockIdx.x, units = nstrip * nseg;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  typedef typename SoftArg<WIDE>::Tau Tau;
  extern __shared__ double lds[];  // [T] thresholds, [T] upstream gradient
  Tau* const stau = reinterpret_cast<Tau*>(lds);
  float* const sg = reinterpret_cast<float*>(stau + T);
  __shared__ StagedEntry stage[256];
  __shared__ float sred[2][4];
  __shared__ int skept[4];
  // Everything the block needs from memory is requested up front, so that the call costs one
  // round trip to memory and not four in a row: the state's header words, the unit's count and
  // the first 256 entries of its list (or as many as the unit has room for, whatever the count says).
  const bool usable = state_usable(sv, expect, item);
  const unsigned cnt_raw = sv.counts[(size_t)item * units + unit];
  const SavedEntry* list = sv.lists + ((size_t)item * units + unit) * expect.cap;
  SavedEntry first = list[min((unsigned)threadIdx.x, expect.cap - 1u)];
  float lo = INFINITY, hi = -INFINITY;
  for (int j = threadIdx.x; j < T; j += 256) {
    const float t = tau[j];
    stau[j] = t;
    sg[j] = gup ? gup[(int64_t)item * T + j] : 1.0f;
    lo = fminf(lo, t);
    hi = fmaxf(hi, t);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fminf(lo, __shfl_xor(lo, o));
    hi = fmaxf(hi, __shfl_xor(hi, o));
  }
  if (lane == 0) {
    sred[0][wv] = lo;
    sred[1][wv] = hi;
  }
  float* gx = grad_X + (int64_t)item * N;
  const int seg = unit / nstrip, strip = unit - seg * nstrip;
  const int x0 = strip * kStripOut, x1 = min(x0 + kStripOut, W);
  const int y0 = seg * rows_per_seg, y1 = min(y0 + rows_per_seg, H);
  if (usable) {  // block-uniform
    if (((reinterpret_cast<uintptr_t>(gx) | (uintptr_t)(W * 4) | (uintptr_t)(x0 * 4) | (uintptr_t)((x1 - x0) * 4)) & 15) == 0) {
      const int w4 = (x1 - x0) / 4;  // 16-byte stores: rows, first column and width all fit
      for (int y = y0 + wv; y < y1; y += 4)
        if (lane < w4) reinterpret_cast<float4*>(gx + (int64_t)y * W + x0)[lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
      for (int y = y0 + wv; y < y1; y += 4)
        for (int x = x0 + lane; x < x1; x += kWave) gx[(int64_t)y * W + x] = 0.0f;
    }
  }
  __syncthreads();  // thresholds in LDS; the fill has reached memory before any entry is written
  lo = fminf(fminf(sred[0][0], sred[0][1]), fminf(sred[0][2], sred[0][3]));
  hi = fmaxf(fmaxf(sred[1][0], sred[1][1]), fmaxf(sred[1][2], sred[1][3]));
  float sat_lo, sat_hi;
  soft_sat_bounds(lo, hi, kneg, T, sat_lo, sat_hi);

  if (!usable) {
    const float* g = grid + (int64_t)item * N;
    Tilt tilt;
    if (TILTC) {
      const DirArgs da = {u, alpha, 1, 2};
      tilt = load_tilt(da, 0);
    }
    const double ux = (double)u[0], uy = (double)u[1];
    for (int y = y0 + wv; y < y1; y += 4) {
      for (int x = x0 + lane; x < x1; x += kWave) {
        int c;
        if (TILTC) c = coeff_tilted_at<2>(g, tilt, 1, H, W, 0, y, x);
        else c = coeff_at<float, 2>(g, 1, H, W, 0, y, x);
        float out = 0.0f;
        if (c != 0) {
          const double yv = (double)g[(int64_t)y * W + x] + (double)alpha * (ux * (double)x + uy * (double)y);
          if ((float)yv > sat_lo && (float)yv < sat_hi) {
            const double packed = SoftArg<WIDE>::pack(yv);
            float gd = 0.0f;
            for (int j = 0; j < T; ++j) gd += sg[j] * soft_dsig<WIDE>(stau[j], packed, kneg);
            out = -lambda * (float)c * gd;
          }
        }
        gx[(int64_t)y * W + x] = out;
      }
    }
    return;
  }

  saved_lists_to_grad<WIDE>(list, cnt_raw, expect.cap, first, stau, sg, T, kneg, lambda, sat_lo, sat_hi, gx, N, stage, skept);
}

static float kneg2d(float lambda) { return (float)(-(double)lambda * 1.4426950408889634); }

bool soft2d_supported(const Shape& s, int T) {
  return s.D == 1 && s.ndim == 2 && T >= 1 && s.W >= 8 && s.W <= (1 << 22) &&
         s.H <= (1 << 30) && s.N < ((int64_t)1 << 31);
}

// per-unit partial sums (up to four floats per unit and threshold), a multiple of 256 bytes
static size_t soft2d_partial_bytes(const Shape& s, const Plan2d& pl, int T) {
  const size_t n = (size_t)s.batch * pl.nstrip * pl.nseg * (size_t)T * 4 * sizeof(float);
  return (n + 255) / 256 * 256;
}
static double* soft2d_mid(void* ws, const Shape& s, const Plan2d& pl, int T) {
  return reinterpret_cast<double*>(static_cast<char*>(ws) + soft2d_partial_bytes(s, pl, T));
}

size_t soft2d_workspace_bytes(const Shape& s, int T) {
  if (!soft2d_supported(s, T)) return 0;
  const Plan2d pl = plan2d<float>(s, Feed2d::kSigmoid);
  return (size_t)256 + soft2d_partial_bytes(s, pl, T) + soft_reduce_mid_bytes(pl.nstrip * pl.nseg, s.batch, T);
}

static dim3 layered(const Plan2d& pl, const Shape& s, int T) {
  return dim3(pl.grid.x, pl.grid.y, soft_layers((int64_t)pl.nstrip * pl.nseg * s.batch, T));
}

void launch_soft2d_fwd(const float* grid, const Shape& s, const float* u, float alpha, const float* tau,
                       int T, float lambda, float* chi, void* ws, hipStream_t st, bool tiltc) {
  const Plan2d pl = plan2d<float>(s, Feed2d::kSigmoid);
  const bool alone = pl.nstrip * pl.nseg == 1;  // an item is one unit: its row is the result
  float* partial = alone ? chi : static_cast<float*>(ws);
  profile_mark(st, false);
#define ECC_GO(TC, WD)                                                                                                 \
  hipLaunchKernelGGL((soft2d_fwd_kernel<TC, WD>), layered(pl, s, T), dim3(256), kSoftLds, st, grid, (int)s.H, (int)s.W, \
                     s.N, pl.nstrip, pl.nseg, pl.rows_per_seg, u, alpha, tau, T, kneg2d(lambda), partial)
  ECC_SOFT_VARIANT(tiltc, soft_wide(T));
#undef ECC_GO
  profile_mark(st, true);
  if (alone) return;
  const RedOut out = {chi, nullptr, nullptr, nullptr, nullptr, {}};
  launch_soft_reduce<1, true, -1>(partial, soft2d_mid(ws, s, pl, T), pl.nstrip * pl.nseg, s.batch, T, alpha, lambda,
                                  Origin2{pl.nstrip, pl.rows_per_seg}, out, st);
}

void launch_soft2d_bwd(const float* grid, const Shape& s, const float* u, float alpha, const float* tau,
                       int T, float lambda, const float* gup, float* grad_X, float* dtau, float* du,
                       void* ws, hipStream_t st, bool tiltc) {
  const Plan2d pl = plan2d<float>(s, Feed2d::kSigmoid);
  float* partial = (dtau || du) ? static_cast<float*>(ws) : nullptr;
  profile_mark(st, false);
#define ECC_GO(TC, WD)                                                                                          \
  hipLaunchKernelGGL((soft2d_bwd_kernel<TC, WD>), pl.grid, dim3(256), kSoftLds, st, grid, (int)s.H, (int)s.W, s.N, \
                     pl.nstrip, pl.nseg, pl.rows_per_seg, u, alpha, tau, T, kneg2d(lambda), lambda, gup, grad_X,  \
                     partial)
  ECC_SOFT_VARIANT(tiltc, soft_wide(T));
#undef ECC_GO
  profile_mark(st, true);
  if (partial) {
    const RedOut out = {nullptr, dtau, du, nullptr, nullptr, {}};
    launch_soft_reduce<4, false, 2>(partial, soft2d_mid(ws, s, pl, T), pl.nstrip * pl.nseg, s.batch, T, alpha, lambda,
                                    Origin2{pl.nstrip, pl.rows_per_seg}, out, st);
  }
}

static SoftStateHeader state_header(const Shape& s, const Plan2d& pl, bool tiltc) {
  SoftStateHeader h;
  h.magic = kSoftStateMagic;
  h.D = 1;
  h.units = pl.nstrip * pl.nseg;
  h.H = (int)s.H;
  h.W = (int)s.W;
  h.batch = (int)s.batch;
  h.nstrip = pl.nstrip;
  h.nseg = pl.nseg;
  h.rows_per_seg = pl.rows_per_seg;
  h.tiltc = tiltc ? 1 : 0;
  h.cap = state_cap(pl);
  return h;
}

void launch_soft2d_fwd_save(const float* grid, const Shape& s, const float* u, float alpha, const float* tau, int T,
                            float lambda, float* chi, float* dtau, float* du, void* state, void* ws, hipStream_t st,
                            bool tiltc) {
  const Plan2d pl = plan2d<float>(s, Feed2d::kSigmoid);
  const StateView sv = state_view(state, s.batch, (size_t)pl.nstrip * pl.nseg);
  const SoftStateHeader hdr = state_header(s, pl, tiltc);
  float* partial = static_cast<float*>(ws);
  const bool deriv = dtau || du;
  profile_mark(st, false);
#define ECC_GO3(TC, DV, WD)                                                                                   \
  hipLaunchKernelGGL((soft2d_fwd_save_kernel<TC, DV, WD>), layered(pl, s, T), dim3(256), kSoftLds, st, grid, (int)s.H, \
                     (int)s.W, s.N, pl.nstrip, pl.nseg, pl.rows_per_seg, u, alpha, tau, T, kneg2d(lambda), partial, sv, \
                     hdr.cap)
#define ECC_GO(TC, WD) do { if (deriv) ECC_GO3(TC, true, WD); else ECC_GO3(TC, false, WD); } while (0)
  ECC_SOFT_VARIANT(tiltc, soft_wide(T));
#undef ECC_GO3
#undef ECC_GO
  profile_mark(st, true);
  const RedOut out = {chi, dtau, du, sv.hdr, sv.gen, hdr};
  launch_soft_reduce<4, true, 2>(partial, soft2d_mid(ws, s, pl, T), pl.nstrip * pl.nseg, s.batch, T, alpha, lambda,
                                 Origin2{pl.nstrip, pl.rows_per_seg}, out, st);
}

void launch_soft2d_bwd_saved(const float* grid, const Shape& s, const float* u, float alpha, const float* tau, int T,
                             float lambda, const float* gup, float* grad_X, const void* state, hipStream_t st,
                             bool tiltc) {
  const Plan2d pl = plan2d<float>(s, Feed2d::kSigmoid);
  const StateView sv = state_view(const_cast<void*>(state), s.batch, (size_t)pl.nstrip * pl.nseg);
  const SoftStateHeader expect = state_header(s, pl, tiltc);
  const dim3 g((unsigned)(pl.nstrip * pl.nseg), (unsigned)s.batch);
  const size_t lds = (size_t)T * (soft_wide(T) ? sizeof(double) + sizeof(float) : 2 * sizeof(float));
  profile_mark(st, false);
#define ECC_GO(TC, WD)                                                                                              \
  hipLaunchKernelGGL((soft2d_bwd_saved_kernel<TC, WD>), g, dim3(256), lds, st, grid, (int)s.H, (int)s.W, s.N, pl.nstrip, \
                     pl.nseg, pl.rows_per_seg, u, alpha, tau, T, kneg2d(lambda), lambda, gup, grad_X, sv, expect)
  ECC_SOFT_VARIANT(tiltc, soft_wide(T));
#undef ECC_GO
  profile_mark(st, true);
}

}  // namespace ecc
