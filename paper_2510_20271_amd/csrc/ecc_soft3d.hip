// Soft single-direction ECC for 3D grids, fused into the tube sweep of
// ecc_sweep3d.h: forward (Eq. 6 of the paper) and derivatives (Eq. 8-10).
//
// As in 2D, only the critical vertices (c != 0) carry a term.  The tube sweep
// finds them and queues (position, c); when 64 are drained together each lane
// fetches one value, forms y = X(p) + alpha <u,p> in float64 and
// parks the entry in a small LDS stage -- unless y lies so far outside [min tau, max tau]
// that every sigmoid is 0 or 1 (see soft_sat_bounds): such an entry adds c or nothing to every
// threshold and is not evaluated.  Then every lane runs over the staged entries for the
// thresholds it owns (tau_l, tau_{l+64}, ...; see ecc_soft_eval.h), z = tau_j - y formed in
// float64 and rounded once.  The sweep
// clears grad_X plane by plane; it is written at the critical vertices only.
// Each wave keeps its partial sums in a row of the workspace; a second kernel adds them
// in a fixed order in float64, so results are run-to-run identical.
#include "ecc_sweep3d.h"
#include "ecc_soft_eval.h"
#include "ecc_soft_saved.h"
#include "ecc_soft_reduce.h"

#include <algorithm>
#include <cstdlib>

namespace ecc {

// MANY: see many_thresholds below.  Slots of 64 thresholds taken together, and waves on a SIMD that the registers are kept
// within.  Four waves leave 128 registers: the kernels spill 5 to 22 of them around a drain (32 to 76 bytes of scratch a
// lane) and are the faster all the same where the sweep is what takes the time; the tilted forward kernel is not (8 x 96^3,
// T = 64: 27.6 us with four waves, 23.1 with three) and takes three.
constexpr int soft3_slots(bool many) { return many ? 4 : 1; }
constexpr int soft3_waves(bool many) { return many ? 3 : 4; }

struct Soft3Staged {
  double y;         // X(p) + alpha <u,p>, packed (see SoftArg)
  float c;
  unsigned inpl;    // element offset inside the plane
  float rx, ry, rz; // coordinates relative to the unit's origin
  unsigned zrel;    // plane of the segment
};

// CHI / DERIV / GRADX: what is formed (see ecc_soft_eval.h); SAVE: every entry is also appended to the unit's list
// in the state buffer (sweep order, no atomics: the same on every run).
template <bool CHI, bool DERIV, bool GRADX, bool SAVE, int STRIDE, bool MANY>
struct Soft3Sink {
  static constexpr bool kTrackRange = false;
  static constexpr bool kZeroFill = GRADX;
  double ux, uy, uz, alpha;
  float sat_lo, sat_hi;  // y <= sat_lo: every sigma is 1;  y >= sat_hi: every sigma is 0 (soft_sat_bounds)
  int W;
  int64_t plane;       // H * W
  int ox, oy, oz;      // origin of the wave's unit: coordinates are summed relative to it
  Soft3Staged* stage;  // wave-private LDS, 64 entries
  SoftEval<3, CHI, DERIV, GRADX, STRIDE, MANY> eval;
  float* gx;           // GRADX: grad_X of this item or null
  float lambda;
  SavedEntry* list;     // SAVE: this unit's list
  unsigned cap, saved;  // saved: entries seen so far (wave-uniform; may pass cap)

  // lane i < n forms its entry; the entries that have to be evaluated are packed into the stage
  __device__ __forceinline__ void take(int n, float v, int ci, unsigned inpl, unsigned zrel) {
    const int lane = threadIdx.x & (kWave - 1);
    const bool in = lane < n;
    const int yy = (int)(inpl / (unsigned)W), x = (int)(inpl - (unsigned)yy * (unsigned)W), z = oz + (int)zrel;
    const double y = (double)v + alpha * ((ux * (double)x + uy * (double)yy) + uz * (double)z);
    Soft3Staged e;
    e.y = SoftArg<MANY>::pack(y);
    e.c = (float)ci;
    e.inpl = inpl;
    e.rx = (float)(x - ox);
    e.ry = (float)(yy - oy);
    e.rz = (float)(z - oz);
    e.zrel = zrel;
    if constexpr (SAVE) {
      if (in && saved + (unsigned)n <= cap) {  // (a batch that does not fit is left out whole)
        SavedEntry o;
        o.y = y;
        o.idx = (int)((int64_t)z * plane + inpl);
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
    const Soft3Staged* st = stage;
    const float g = eval.template run<soft3_slots(MANY)>(n, csat, [st](int i, StagedValue& o, float (&r)[3]) {
      const Soft3Staged s = st[i];
      o.y = s.y;
      o.c = s.c;
      r[0] = s.rx;
      r[1] = s.ry;
      r[2] = s.rz;
    });
    if constexpr (GRADX) {
      if (gx && lane < n) {
        const Soft3Staged s = stage[lane];
        gx[(int64_t)(oz + (int)s.zrel) * plane + s.inpl] = -lambda * s.c * g;
      }
    }
  }
};

// LDS of a block: exchange words, [4 waves] queue entries and tilts, [4 waves] stages
constexpr size_t kSoft3Lds = kFixedLds3d + (size_t)4 * kWave * sizeof(Soft3Staged);

// The sweep of a wave with sink `queue.sink`, whose own fields the kernels below have set; partial (may be null):
// rows of STRIDE floats a threshold, one row a unit.  TILTC: the sweep runs on the tilted field, so c(p) is that
// field's coefficient.
template <bool TILTC, int STRIDE, typename Sink>
__device__ __forceinline__ void soft3d_sweep(s3::TubeQueue<Sink>& queue, const float* __restrict__ grid, int D, int H,
                                             int W, int64_t N, const Tiling3& tl, int nseg, int planes_per_seg,
                                             const float* u, float alpha, const float* tau, int T, float kneg,
                                             const float* gup, float* partial) {
  extern __shared__ int smem[];
  const int wv = threadIdx.x >> 6;
  unsigned* xch = reinterpret_cast<unsigned*>(smem);
  queue.buf = reinterpret_cast<uint2*>(smem + kXchInts) + wv * kQueueCap;
  queue.tbuf = reinterpret_cast<float*>(smem + kXchInts + 4 * kQueueCap * 2) + wv * kQueueCap;
  queue.count = 0;
  Sink& s = queue.sink;
  s.stage = reinterpret_cast<Soft3Staged*>(smem + kXchInts + 4 * kQueueCap * 3) + wv * kWave;
  s.ux = (double)u[0];
  s.uy = (double)u[1];
  s.uz = (double)u[2];
  s.alpha = (double)alpha;
  float lo, hi;
  threshold_span(tau, T, lo, hi);
  soft_sat_bounds(lo, hi, kneg, T, s.sat_lo, s.sat_hi);
  s.W = W;
  s.plane = (int64_t)H * W;
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(wv), units = gridDim.x * 4;
  unit_origin3(unit, tl, planes_per_seg, kRows3d, s.ox, s.oy, s.oz);
  int j0, nj;
  soft_layer(T, j0, nj);
  s.eval.init(tau + j0, nj, kneg, gup ? gup + (int64_t)blockIdx.y * T + j0 : nullptr,
              partial ? partial + (((int64_t)blockIdx.y * units + unit) * (int64_t)T + j0) * STRIDE : nullptr);
  WaveRange range;
  const float* g = grid + (int64_t)blockIdx.y * N;
  if constexpr (TILTC) {
    const DirArgs da = {u, alpha, 1, 3};
    const Tilt t = load_tilt(da, 0);
    TiltRaw tr;
    tr.ax = t.ax, tr.ay = t.ay, tr.az = t.az;
    sweep3d_wave<float, kRows3d>(g, D, H, W, N, tl, nseg, planes_per_seg, queue, xch, range, tr);
  } else {
    sweep3d_wave<float, kRows3d>(g, D, H, W, N, tl, nseg, planes_per_seg, queue, xch, range, NoTilt());
  }
  s.eval.finish();
}

// partial[(item * units + unit) * T + j]
template <bool TILTC, bool MANY>
__global__ __launch_bounds__(256, soft3_waves(MANY || TILTC)) void soft3d_fwd_kernel(const float* __restrict__ grid, int D, int H, int W,
                                                            int64_t N, Tiling3 tl, int nseg,
                                                            int planes_per_seg, const float* __restrict__ u,
                                                            float alpha, const float* __restrict__ tau, int T,
                                                            float kneg, float* __restrict__ partial) {
  s3::TubeQueue<Soft3Sink<true, false, false, false, 1, MANY>> queue;
  soft3d_sweep<TILTC, 1>(queue, grid, D, H, W, N, tl, nseg, planes_per_seg, u, alpha, tau, T, kneg, nullptr,
                         partial);
}

// partial[((item * units + unit) * T + j) * 4 + {0: A0, 1: Ax, 2: Ay, 3: Az}]
template <bool TILTC, bool MANY>
__global__ __launch_bounds__(256, soft3_waves(MANY)) void soft3d_bwd_kernel(const float* __restrict__ grid, int D, int H, int W,
                                                            int64_t N, Tiling3 tl, int nseg,
                                                            int planes_per_seg, const float* __restrict__ u,
                                                            float alpha, const float* __restrict__ tau, int T,
                                                            float kneg, float lambda, const float* __restrict__ gup,
                                                            float* __restrict__ grad_X, float* __restrict__ partial) {
  s3::TubeQueue<Soft3Sink<false, true, true, false, 4, MANY>> queue;
  queue.sink.gx = grad_X ? grad_X + (int64_t)blockIdx.y * N : nullptr;
  queue.sink.lambda = lambda;
  soft3d_sweep<TILTC, 4>(queue, grid, D, H, W, N, tl, nseg, planes_per_seg, u, alpha, tau, T, kneg, gup,
                         partial);
}

// Forward pass that saves its critical vertices: chi as soft3d_fwd_kernel, with DERIV the sums of Eq. 9 / Eq. 10 in
// the same pass (they share the sigmoid), and the unit's list.
// partial[((item * units + unit) * T + j) * 5 + {0: chi, 1: A0, 2: Ax, 3: Ay, 4: Az}]
template <bool TILTC, bool DERIV, bool MANY>
__global__ __launch_bounds__(256, soft3_waves(MANY)) void soft3d_fwd_save_kernel(
    const float* __restrict__ grid, int D, int H, int W, int64_t N, Tiling3 tl, int nseg, int planes_per_seg,
    const float* __restrict__ u, float alpha, const float* __restrict__ tau, int T, float kneg,
    float* __restrict__ partial, StateView sv, unsigned cap) {
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), units = gridDim.x * 4;
  s3::TubeQueue<Soft3Sink<true, DERIV, false, true, 5, MANY>> queue;
  queue.sink.cap = blockIdx.z == 0 ? cap : 0u;  // (the first layer keeps the list)
  queue.sink.saved = 0u;
  queue.sink.list = sv.lists + ((size_t)blockIdx.y * units + unit) * cap;
  const unsigned next_gen = *sv.gen + 1u;  // (the reduction kernel that follows stores it)
  soft3d_sweep<TILTC, 5>(queue, grid, D, H, W, N, tl, nseg, planes_per_seg, u, alpha, tau, T, kneg, nullptr,
                         partial);
  if (blockIdx.z == 0 && (threadIdx.x & (kWave - 1)) == 0) {
    sv.counts[(size_t)blockIdx.y * units + unit] = queue.sink.saved;
    if (queue.sink.saved > cap) sv.overflow[blockIdx.y] = next_gen;
  }
}

// grad_X from the saved lists (Eq. 8 contracted with the upstream gradient): a block per unit of
// the forward sweep walks that unit's list; grad_X has been cleared by a fill kernel.  An item
// whose lists cannot be used (header of another shape, a unit ran out of room) is computed from
// the grid instead, vertex by vertex with the plain stencil: slow, but rare.
template <bool TILTC, bool WIDE>
__global__ __launch_bounds__(256) void soft3d_bwd_saved_kernel(const float* __restrict__ grid, int D, int H, int W,
                                                               int64_t N, const float* __restrict__ u, float alpha,
                                                               const float* __restrict__ tau, int T, float kneg,
                                                               float lambda, const float* __restrict__ gup,
                                                               float* __restrict__ grad_X, StateView sv,
                                                               SoftStateHeader expect) {
  const int item = blockIdx.y, unit = blockIdx.x, units = gridDim.x;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  typedef typename SoftArg<WIDE>::Tau Tau;
  extern __shared__ double lds[];  // [T] thresholds, [T] upstream gradient
  Tau* const stau = reinterpret_cast<Tau*>(lds);
  float* const sg = reinterpret_cast<float*>(stau + T);
  __shared__ StagedEntry stage[256];
  __shared__ float sred[2][4];
  __shared__ int skept[4];
  // requested up front, in one round trip to memory: the state's header words, the unit's count
  // and the first 256 slots of its list (whatever the count says)
  const bool usable = state_usable(sv, expect, item);
  const unsigned cnt_raw = sv.counts[(size_t)item * units + unit];
  const SavedEntry* list = sv.lists + ((size_t)item * units + unit) * expect.cap;
  const SavedEntry first = list[min((unsigned)threadIdx.x, expect.cap - 1u)];
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
  __syncthreads();
  lo = fminf(fminf(sred[0][0], sred[0][1]), fminf(sred[0][2], sred[0][3]));
  hi = fmaxf(fmaxf(sred[1][0], sred[1][1]), fmaxf(sred[1][2], sred[1][3]));
  float sat_lo, sat_hi;
  soft_sat_bounds(lo, hi, kneg, T, sat_lo, sat_hi);
  float* gx = grad_X + (int64_t)item * N;
  if (!usable) {
    const float* g = grid + (int64_t)item * N;
    Tilt tilt;
    if (TILTC) {
      const DirArgs da = {u, alpha, 1, 3};
      tilt = load_tilt(da, 0);
    }
    const double ux = (double)u[0], uy = (double)u[1], uz = (double)u[2];
    for (int64_t i = (int64_t)unit * 256 + threadIdx.x; i < N; i += (int64_t)units * 256) {
      const int64_t x = i % W, r = i / W, y = r % H, z = r / H;
      int c;
      if (TILTC) c = coeff_tilted_at<3>(g, tilt, D, H, W, z, y, x);
      else c = coeff_at<float, 3>(g, D, H, W, z, y, x);
      if (c != 0) {
        const double yv = (double)g[i] + (double)alpha * ((ux * (double)x + uy * (double)y) + uz * (double)z);
        if ((float)yv > sat_lo && (float)yv < sat_hi) {
          const double packed = SoftArg<WIDE>::pack(yv);
          float gd = 0.0f;
          for (int j = 0; j < T; ++j) gd += sg[j] * soft_dsig<WIDE>(stau[j], packed, kneg);
          gx[i] = -lambda * (float)c * gd;
        }
      }
    }
    return;
  }
  saved_lists_to_grad<WIDE>(list, cnt_raw, expect.cap, first, stau, sg, T, kneg, lambda, sat_lo, sat_hi, gx, N, stage, skept);
}

// origin of a unit's coordinates, for the reduction of ecc_soft_reduce.h
struct Origin3 {
  Tiling3 tl;
  int planes_per_seg;
  __device__ __forceinline__ void operator()(int unit, int (&o)[3]) const {
    unit_origin3(unit, tl, planes_per_seg, kRows3d, o[0], o[1], o[2]);
  }
};

static float kneg3d(float lambda) { return (float)(-(double)lambda * 1.4426950408889634); }

bool soft3d_supported(const Shape& s, int T) {
  return s.ndim == 3 && T >= 1 && sweep3d_supported(s, 1);
}

// per-unit partial sums (up to five floats per unit and threshold), a multiple of 256 bytes
static size_t soft3d_partial_bytes(const Shape& s, const Plan3d& pl, int T) {
  const size_t n = (size_t)s.batch * pl.grid.x * 4 * (size_t)T * 5 * sizeof(float);
  return (n + 255) / 256 * 256;
}

size_t soft3d_workspace_bytes(const Shape& s, int T) {
  if (!soft3d_supported(s, T)) return 0;
  const Plan3d pl = plan3d<float>(s, Fold3::kSoft);
  return (size_t)256 + soft3d_partial_bytes(s, pl, T) + soft_reduce_mid_bytes((int)pl.grid.x * 4, s.batch, T);
}

// Above 128 thresholds the evaluation weighs more than the sweep: four slots share the reads of an entry, three waves a
// SIMD hold their registers (us with one slot and four waves / four slots and three, fields of width 2: backward pass of
// 128^3 with 256 thresholds 66.7 / 47.6, saving forward pass of 8 x 96^3 with 192 57.8 / 51.7, backward pass of 4 x 128^3
// with 192 72.1 / 77.3; forward passes up to 128 thresholds are 2 to 4 % slower with three waves).
static bool many_thresholds(int T) { return T > 128; }

static dim3 layered(const Plan3d& pl, const Shape& s, int T) {
  return dim3(pl.grid.x, pl.grid.y, soft_layers((int64_t)pl.grid.x * 4 * s.batch, T, T <= 256 ? 1536 : 3072));
}

void launch_soft3d_fwd(const float* grid, const Shape& s, const float* u, float alpha, const float* tau, int T,
                       float lambda, float* chi, void* ws, hipStream_t st, bool tiltc) {
  const Plan3d pl = plan3d<float>(s, Fold3::kSoft);
  float* partial = static_cast<float*>(ws);
#define ECC_GO(TC, MANY)                                                                                          \
  hipLaunchKernelGGL((soft3d_fwd_kernel<TC, MANY>), layered(pl, s, T), dim3(256), kSoft3Lds, st, grid, (int)s.D, (int)s.H,      \
                     (int)s.W, s.N, pl.tl, pl.nseg, pl.planes_per_seg, u, alpha, tau, T,       \
                     kneg3d(lambda), partial)
  ECC_SOFT_VARIANT(tiltc, many_thresholds(T));
#undef ECC_GO
  double* mid = reinterpret_cast<double*>(static_cast<char*>(ws) + soft3d_partial_bytes(s, pl, T));
  const RedOut out = {chi, nullptr, nullptr, nullptr, nullptr, {}};
  launch_soft_reduce<1, true, -1>(partial, mid, (int)pl.grid.x * 4, s.batch, T, alpha, lambda, Origin3{pl.tl, pl.planes_per_seg}, out, st);
}

void launch_soft3d_bwd(const float* grid, const Shape& s, const float* u, float alpha, const float* tau, int T,
                       float lambda, const float* gup, float* grad_X, float* dtau, float* du, void* ws,
                       hipStream_t st, bool tiltc) {
  const Plan3d pl = plan3d<float>(s, Fold3::kSoft);
  float* partial = (dtau || du) ? static_cast<float*>(ws) : nullptr;
#define ECC_GO(TC, MANY)                                                                                          \
  hipLaunchKernelGGL((soft3d_bwd_kernel<TC, MANY>), pl.grid, dim3(256), kSoft3Lds, st, grid, (int)s.D, (int)s.H,      \
                     (int)s.W, s.N, pl.tl, pl.nseg, pl.planes_per_seg, u, alpha, tau, T,       \
                     kneg3d(lambda), lambda, gup, grad_X, partial)
  ECC_SOFT_VARIANT(tiltc, many_thresholds(T));
#undef ECC_GO
  if (partial) {
    double* mid = reinterpret_cast<double*>(static_cast<char*>(ws) + soft3d_partial_bytes(s, pl, T));
    const RedOut out = {nullptr, dtau, du, nullptr, nullptr, {}};
    launch_soft_reduce<4, false, 3>(partial, mid, (int)pl.grid.x * 4, s.batch, T, alpha, lambda, Origin3{pl.tl, pl.planes_per_seg}, out, st);
  }
}

// ---- forward that saves its critical vertices, backward from the saved lists ----------------
static unsigned state_cap3(const Shape& s, const Plan3d& pl) {
  // room for one vertex in eight of a unit's planes x 4 rows x 62 columns, rounded up to 64 entries; of twelve planes at least
  // in small launches, since the share of critical vertices varies the more the fewer there are (16 x 48 x 64 in segments of
  // eight planes ran over: backward pass from the grid, 41 us instead of 14).
  const Tiling3& tl = pl.tl;
  const bool small = (int64_t)pl.nseg * tl.nstrip * tl.ngroup4 * s.batch <= 4096;
  const unsigned planes = std::max(small ? 12u : 1u, (unsigned)pl.planes_per_seg);
  const unsigned cap = (planes * (unsigned)kRows3d * (unsigned)s3::kOut / 8u + 63u) / 64u * 64u;
  // The folded units of a narrow volume, whose unfolded ones had room for most of their few vertices, have room for one in
  // four, unless the launch is many rounds long (739 x 8 x 8 x 16 folded, a ninth of whose vertices is critical: 19 us, 27 from
  // the grid).
  if (tl.nstrip > 1 || tl.F == 1 || tl.ngroup * s.batch * s.D >= 160000) return cap;
  return std::max(cap, ((unsigned)tl.F * (unsigned)s.W * planes + 63u) / 64u * 64u);
}
static bool soft3d_saves(const Shape& s) { return soft3d_supported(s, 1) && s.N < ((int64_t)1 << 31); }
size_t soft3d_state_bytes(const Shape& s) {
  if (!soft3d_saves(s)) return 256;
  const Plan3d pl = plan3d<float>(s, Fold3::kSoft);
  return state_bytes(s.batch, (size_t)pl.grid.x * 4, state_cap3(s, pl));
}
bool soft3d_state_supported(const Shape& s, int T) { return soft3d_supported(s, T) && soft3d_saves(s); }

static SoftStateHeader state_header3(const Shape& s, const Plan3d& pl, bool tiltc) {
  SoftStateHeader h;
  h.magic = kSoftStateMagic;
  h.D = (int)s.D;
  h.H = (int)s.H;
  h.W = (int)s.W;
  h.batch = (int)s.batch;
  h.nstrip = pl.tl.nstrip;
  h.nseg = pl.nseg;
  h.rows_per_seg = pl.planes_per_seg;
  h.units = (int)pl.grid.x * 4;
  h.tiltc = tiltc ? 1 : 0;
  h.cap = state_cap3(s, pl);
  return h;
}

void launch_soft3d_fwd_save(const float* grid, const Shape& s, const float* u, float alpha, const float* tau, int T,
                            float lambda, float* chi, float* dtau, float* du, void* state, void* ws, hipStream_t st,
                            bool tiltc) {
  const Plan3d pl = plan3d<float>(s, Fold3::kSoft);
  const SoftStateHeader hdr = state_header3(s, pl, tiltc);
  const StateView sv = state_view(state, s.batch, (size_t)hdr.units);
  float* partial = static_cast<float*>(ws);
  double* mid = reinterpret_cast<double*>(static_cast<char*>(ws) + soft3d_partial_bytes(s, pl, T));
  const bool deriv = dtau || du;
#define ECC_GO3(TC, DV, MANY)                                                                                       \
  hipLaunchKernelGGL((soft3d_fwd_save_kernel<TC, DV, MANY>), layered(pl, s, T), dim3(256), kSoft3Lds, st, grid, (int)s.D, (int)s.H, \
                     (int)s.W, s.N, pl.tl, pl.nseg, pl.planes_per_seg, u, alpha, tau, T,         \
                     kneg3d(lambda), partial, sv, hdr.cap)
#define ECC_GO(TC, MANY) do { if (deriv) ECC_GO3(TC, true, MANY); else ECC_GO3(TC, false, MANY); } while (0)
  ECC_SOFT_VARIANT(tiltc, many_thresholds(T));
#undef ECC_GO3
#undef ECC_GO
  const RedOut out = {chi, dtau, du, sv.hdr, sv.gen, hdr};
  launch_soft_reduce<5, true, 3>(partial, mid, (int)pl.grid.x * 4, s.batch, T, alpha, lambda, Origin3{pl.tl, pl.planes_per_seg}, out, st);
}

void launch_soft3d_bwd_saved(const float* grid, const Shape& s, const float* u, float alpha, const float* tau, int T,
                             float lambda, const float* gup, float* grad_X, const void* state, hipStream_t st,
                             bool tiltc) {
  const Plan3d pl = plan3d<float>(s, Fold3::kSoft);
  const SoftStateHeader expect = state_header3(s, pl, tiltc);
  const StateView sv = state_view(const_cast<void*>(state), s.batch, (size_t)expect.units);
  launch_clear_f32(grad_X, s.N * s.batch, st);  // zero away from the critical vertices
  const dim3 g((unsigned)expect.units, (unsigned)s.batch);
  const size_t lds = (size_t)T * (soft_wide(T) ? sizeof(double) + sizeof(float) : 2 * sizeof(float));
#define ECC_GO(TC, WD)                                                                                            \
  hipLaunchKernelGGL((soft3d_bwd_saved_kernel<TC, WD>), g, dim3(256), lds, st, grid, (int)s.D, (int)s.H, (int)s.W, s.N, \
                     u, alpha, tau, T, kneg3d(lambda), lambda, gup, grad_X, sv, expect)
  ECC_SOFT_VARIANT(tiltc, soft_wide(T));
#undef ECC_GO
}

}  // namespace ecc
