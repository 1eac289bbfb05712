// Hard ECC, 3D: kernels and launchers around the tube sweep of ecc_sweep3d.h.
#include "ecc_sweep3d.h"

namespace ecc {

// Histogram mode; run_if (may be null): do nothing unless *run_if != 0.
template <int R, bool TLDS, int MODE>
__global__ __launch_bounds__(256) void sweep3d_kernel(
    const float* __restrict__ grid, int D, int H, int W, int64_t N, int bins, Tiling3 tl,
    int nseg, int planes_per_seg, const HardHeader* __restrict__ hdr,
    const float* __restrict__ table, HistOut hist,
    const unsigned* __restrict__ run_if, DirArgs dir) {
  if (run_if && *run_if == 0) return;
  extern __shared__ int smem[];
  // [2][4 waves][9][64] exchange words, [4 waves] queues (entries, tilts), histogram, table
  unsigned* xch = reinterpret_cast<unsigned*>(smem);
  uint2* qbuf = reinterpret_cast<uint2*>(smem + kXchInts) + (threadIdx.x >> 6) * kQueueCap;
  float* tbuf = reinterpret_cast<float*>(smem + kXchInts + 4 * kQueueCap * 2) + (threadIdx.x >> 6) * kQueueCap;
  int* lhist = smem + kXchInts + 4 * kQueueCap * 3;
  float* ltable = reinterpret_cast<float*>(lhist + bins);
  for (int b = threadIdx.x; b < bins; b += 256) {
    lhist[b] = 0;
    if (TLDS) ltable[b] = table[b];
  }
  __syncthreads();
  s3::TubeQueue<HistSink<false, mode_is_super(MODE)>> queue;
  queue.buf = qbuf;
  queue.tbuf = tbuf;
  queue.count = 0;
  queue.sink.lhist = lhist;
  queue.sink.table = TLDS ? ltable : table;
  queue.sink.bins = bins;
  queue.sink.lo = hdr->lo;
  queue.sink.scale = hdr->scale;
  WaveRange range;
  if constexpr (MODE == kTilted) {
    const int d = blockIdx.y / dir.batch, item = blockIdx.y - d * dir.batch;
    sweep3d_wave<float, R>(grid + (int64_t)item * N, D, H, W, N, tl, nseg, planes_per_seg, queue, xch,
                       range, load_tilt(dir, d));
  } else {
    sweep3d_wave<float, R>(grid + (int64_t)blockIdx.y * N, D, H, W, N, tl, nseg, planes_per_seg,
                       queue, xch, range, typename ModeTransform<MODE>::type());
  }
  __syncthreads();
  leave_histogram<256>(lhist, bins, hist);
}

// Single-pass mode: critical vertices to the item's list, min / max to the header.
template <int R, int MODE>
__global__ __launch_bounds__(256) void sweep3d_list_kernel(const float* __restrict__ grid, int D, int H, int W,
                                                           int64_t N, Tiling3 tl, int nseg,
                                                           int planes_per_seg, ListArgs la, DirArgs dir) {
  extern __shared__ int smem[];
  unsigned* xch = reinterpret_cast<unsigned*>(smem);
  uint2* qbuf = reinterpret_cast<uint2*>(smem + kXchInts) + (threadIdx.x >> 6) * kQueueCap;
  s3::TubeQueue<ListSink> queue;
  queue.buf = qbuf;
  queue.tbuf = reinterpret_cast<float*>(smem + kXchInts + 4 * kQueueCap * 2) + (threadIdx.x >> 6) * kQueueCap;
  queue.count = 0;
  __shared__ unsigned own[4];  // list per block: fill count, least / greatest key, overflow (never raised)
  if (la.heads) {              // (block-uniform)
    block_list_begin(la, queue.sink, own);
  } else {
    const unsigned sub = blockIdx.y * la.nsub + (blockIdx.x & (la.nsub - 1u));
    queue.sink.list = la.lists + (size_t)sub * la.cap;
    queue.sink.counter = la.counters + sub;
    queue.sink.overflow = &la.hdr->overflow;
  }
  queue.sink.cap = la.cap;
  WaveRange range;
  if constexpr (MODE == kTilted) {
    const int d = blockIdx.y / dir.batch, item = blockIdx.y - d * dir.batch;
    sweep3d_wave<float, R>(grid + (int64_t)item * N, D, H, W, N, tl, nseg, planes_per_seg, queue, xch,
                       range, load_tilt(dir, d));
  } else {
    sweep3d_wave<float, R>(grid + (int64_t)blockIdx.y * N, D, H, W, N, tl, nseg, planes_per_seg,
                       queue, xch, range, typename ModeTransform<MODE>::type());
  }
  if (la.heads) block_list_end(la, range, own);
  else range.commit(la.hdr);
}

static void launch3d(const float* p, const Shape& s, int bins, const HardHeader* hdr, const float* table,
                     const HistOut& hist, hipStream_t st, const unsigned* run_if, const DirArgs* dir, int conv) {
  constexpr int R = kRows3d;
  const Plan3d pl = plan3d<float>(s);
  const bool tlds = (size_t)bins * 8 + kFixedLds3d <= 60 * 1024;
  const size_t lds = kFixedLds3d + (size_t)bins * (tlds ? 8 : 4);
  const DirArgs none = {nullptr, 0.f, 1, 3};
#define ECC_GO(TL, TI)                                                                                    \
  hipLaunchKernelGGL((sweep3d_kernel<R, TL, TI>), pl.grid, dim3(256), lds, st, p, (int)s.D, (int)s.H,     \
                     (int)s.W, s.N, bins, pl.tl, pl.nseg, pl.planes_per_seg, hdr, table,   \
                     hist, run_if, dir ? *dir : none)
#define ECC_MODE(M)          \
  do {                       \
    if (tlds) ECC_GO(true, M); \
    else ECC_GO(false, M);   \
  } while (0)
  if (dir) {  // directional call
    ECC_MODE(kTilted);
    return;
  }
  switch (mode_of_conv(conv)) {
    case kTopCells: ECC_MODE(kTopCells); break;
    case kSuper: ECC_MODE(kSuper); break;
    case kTopSuper: ECC_MODE(kTopSuper); break;
    default: ECC_MODE(kPlain); break;
  }
#undef ECC_MODE
#undef ECC_GO
}

static void launch3d_list(const float* p, const Shape& s, const ListArgs& la, hipStream_t st, const DirArgs* dir,
                          int conv) {
  const Plan3d pl = plan3d<float>(s);
  const DirArgs none = {nullptr, 0.f, 1, 3};
#define ECC_LIST(M, DIR)                                                                                  \
  hipLaunchKernelGGL((sweep3d_list_kernel<kRows3d, M>), pl.grid, dim3(256), kFixedLds3d, st, p,           \
                     (int)s.D, (int)s.H, (int)s.W, s.N, pl.tl, pl.nseg, pl.planes_per_seg, la, \
                     DIR)
  if (dir) {
    ECC_LIST(kTilted, *dir);
    return;
  }
  switch (mode_of_conv(conv)) {
    case kTopCells: ECC_LIST(kTopCells, none); break;
    case kSuper: ECC_LIST(kSuper, none); break;
    case kTopSuper: ECC_LIST(kTopSuper, none); break;
    default: ECC_LIST(kPlain, none); break;
  }
#undef ECC_LIST
}

// dtype: float32, float16 or bfloat16 (the floating types whose range is found on the device)
void launch_sweep3d_list(const void* grid, int dtype, const Shape& s, const ListArgs& la, hipStream_t st,
                         const DirArgs* dir, int conv) {
  if (dtype != 2) launch_sweep3dp_list(grid, dtype, s, la, st, conv);
  else launch3d_list(static_cast<const float*>(grid), s, la, st, dir, conv);
}

unsigned sweep3d_shared_list_blocks(const Shape& s, int dtype) {
  return dtype == 2 ? plan3d<float>(s).grid.x : sweep3dp_shared_list_blocks(s);
}
unsigned sweep3d_hist_blocks(const Shape& s, int dtype, int bins) {
  return dtype == 2 ? plan3d<float>(s).grid.x : sweep3dp_hist_blocks(s, bins);
}
// blocks per item, and the most vertices of a block, of a launch with a list for each block
void sweep3d_list_plan(const Shape& s, int dtype, unsigned& per_item, unsigned& vertices) {
  if (dtype != 2) {
    sweep3dp_list_plan(s, per_item, vertices);
    return;
  }
  // four wave units of at most 62 columns x 4 rows (a folded unit: several row groups of fewer columns) x the segment's planes
  const Plan3d pl = plan3d<float>(s);
  per_item = pl.grid.x;
  vertices = 4u * (unsigned)s3::kOut * (unsigned)kRows3d * (unsigned)std::min<int64_t>(s.D, pl.planes_per_seg);
}

bool sweep3d_supported(const Shape& s, int bins) {
  // 32-bit element offsets inside a chunk of up to 31 planes (and so one plane stays far
  // below the 2^31 bytes a buffer resource can span)
  return bins <= 10240 && s.ndim == 3 && s.D >= 2 && s.W >= 8 && s.W <= (1 << 22) && s.H <= (1 << 22) &&
         s.H * s.W * 32 < ((int64_t)1 << 32) && s.D <= (1 << 30);
}

void launch_sweep3d(const void* grid, const Shape& s, int dtype, bool levels, int bins,
                    const HardHeader* hdr, const float* table, const HistOut& hist,
                    hipStream_t st, const unsigned* run_if, const DirArgs* dir, int conv) {
  if (dtype != 2) launch_sweep3dp(grid, s, dtype, levels, bins, hdr, table, hist, st, run_if, conv);
  else launch3d(static_cast<const float*>(grid), s, bins, hdr, table, hist, st, run_if, dir, conv);
}

// Coefficient map through the tube sweep: the critical vertices' c(p) written to an int8 map
// that the caller has cleared.  The same stencil, order and tie-break as every other
// tube-sweep kernel, made visible vertex by vertex.
template <int R>
__global__ __launch_bounds__(256) void coeff3d_kernel(const float* __restrict__ grid, int D, int H, int W, int64_t N,
                                                      Tiling3 tl, int nseg, int planes_per_seg,
                                                      int8_t* __restrict__ out) {
  extern __shared__ int smem[];
  unsigned* xch = reinterpret_cast<unsigned*>(smem);
  s3::TubeQueue<CoeffSink3d> queue;
  queue.buf = reinterpret_cast<uint2*>(smem + kXchInts) + (threadIdx.x >> 6) * kQueueCap;
  queue.tbuf = reinterpret_cast<float*>(smem + kXchInts + 4 * kQueueCap * 2) + (threadIdx.x >> 6) * kQueueCap;
  queue.count = 0;
  queue.sink.out = out + (int64_t)blockIdx.y * N;
  queue.sink.plane = (int64_t)H * W;
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int ox, oy;
  unit_origin3(unit, tl, planes_per_seg, R, ox, oy, queue.sink.oz);
  WaveRange range;
  sweep3d_wave<float, R>(grid + (int64_t)blockIdx.y * N, D, H, W, N, tl, nseg, planes_per_seg, queue, xch,
                         range, NoTilt());
}

void launch_coeff3d(const void* grid, const Shape& s, int dtype, int8_t* out, hipStream_t st) {
  if (dtype != 2) {
    launch_coeff3dp(grid, s, dtype, out, st);
    return;
  }
  const Plan3d pl = plan3d<float>(s);
  hipLaunchKernelGGL((coeff3d_kernel<kRows3d>), pl.grid, dim3(256), kFixedLds3d, st, static_cast<const float*>(grid),
                     (int)s.D, (int)s.H, (int)s.W, s.N, pl.tl, pl.nseg, pl.planes_per_seg, out);
}

}  // namespace ecc
