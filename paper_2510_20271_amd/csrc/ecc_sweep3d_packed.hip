// Hard ECC, 3D, one- and two-byte element types: kernels and launchers around the packed tube sweep of
// ecc_sweep3d_packed.h.
#include "ecc_sweep3d_packed.h"

#include <algorithm>
#include <cmath>

namespace ecc {

// Histogram mode; run_if (may be null): do nothing unless *run_if != 0.
template <typename T, bool LEVELS, bool TLDS, int MODE>
__global__ __launch_bounds__(256, 4) void sweep3dp_kernel(const T* __restrict__ grid, int D, int H, int W, int64_t N,
                                                       int bins, Tiling3 tl, int nseg, int planes_per_seg,
                                                       const HardHeader* __restrict__ hdr,
                                                       const float* __restrict__ table,
                                                       HistOut hist,
                                                       const unsigned* __restrict__ run_if) {
  if (run_if && *run_if == 0) return;
  extern __shared__ int smem[];
  // [4 waves] queues, histogram, table
  int* lhist = smem + 4 * kQueueCap * 2;
  float* ltable = reinterpret_cast<float*>(lhist + bins);
  for (int b = threadIdx.x; b < bins; b += 256) {
    lhist[b] = 0;
    if (TLDS) ltable[b] = table[b];
  }
  __syncthreads();
  s3::TubeQueue<HistSink<LEVELS, mode_is_super(MODE)>> queue;
  queue.buf = reinterpret_cast<uint2*>(smem) + (threadIdx.x >> 6) * kQueueCap;
  queue.tbuf = nullptr;
  queue.count = 0;
  queue.sink.lhist = lhist;
  queue.sink.table = TLDS ? ltable : table;
  queue.sink.bins = bins;
  queue.sink.lo = LEVELS ? 0.f : hdr->lo;
  queue.sink.scale = LEVELS ? 0.f : hdr->scale;
  WaveRange range;
  sweep3dp_wave<T, HistSink<LEVELS, mode_is_super(MODE)>, typename ModeTransform<MODE>::type>(
      grid + (int64_t)blockIdx.y * N, D, H, W, tl, nseg, planes_per_seg, queue, range);
  __syncthreads();
  leave_histogram<256>(lhist, bins, hist);
}

// Single-pass mode: critical vertices to the item's list, min / max to the header.
template <typename T, int MODE>
__global__ __launch_bounds__(256, 4) void sweep3dp_list_kernel(const T* __restrict__ grid, int D, int H, int W, int64_t N,
                                                            Tiling3 tl, int nseg, int planes_per_seg, ListArgs la) {
  extern __shared__ int smem[];
  s3::TubeQueue<ListSink> queue;
  queue.buf = reinterpret_cast<uint2*>(smem) + (threadIdx.x >> 6) * kQueueCap;
  queue.tbuf = nullptr;
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
  sweep3dp_wave<T, ListSink, typename ModeTransform<MODE>::type>(grid + (int64_t)blockIdx.y * N, D, H, W, tl, nseg,
                                                                 planes_per_seg, queue, range);
  if (la.heads) block_list_end(la, range, own);
  else range.commit(la.hdr);
}

template <typename T>
__global__ __launch_bounds__(256, 4) void coeff3dp_kernel(const T* __restrict__ grid, int D, int H, int W, int64_t N,
                                                       Tiling3 tl, int nseg, int planes_per_seg, int8_t* __restrict__ out) {
  extern __shared__ int smem[];
  s3::TubeQueue<CoeffSink3d> queue;
  queue.buf = reinterpret_cast<uint2*>(smem) + (threadIdx.x >> 6) * kQueueCap;
  queue.tbuf = nullptr;
  queue.count = 0;
  queue.sink.out = out + (int64_t)blockIdx.y * N;
  queue.sink.plane = (int64_t)H * W;
  queue.sink.oz = (int)(blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) / tl.units_seg * planes_per_seg;
  WaveRange range;
  sweep3dp_wave<T, CoeffSink3d, NoTilt>(grid + (int64_t)blockIdx.y * N, D, H, W, tl, nseg, planes_per_seg, queue, range);
}

constexpr size_t kQueueBytes3dp = (size_t)4 * kQueueCap * sizeof(uint2);

struct Plan3dp {
  Tiling3 tl;
  int nseg, planes_per_seg;
  dim3 grid;
};
enum class Feed3dp { kHist, kSharedLists, kBlockLists, kMap };
// entries of a block's list: its four wave units of 62 columns x 4 rows (a folded unit: several row groups of fewer columns)
static int64_t block_vertices3dp(const Shape& s, int planes) {
  return (int64_t)4 * s3::kOut * s3p::kR * std::min<int64_t>(s.D, planes);
}
// bins: of a histogram sweep
static Plan3dp plan3dp(const Shape& s, Feed3dp feed, int bins = 0) {
  Plan3dp p;
  const int D = (int)s.D, H = (int)s.H, W = (int)s.W;
  const Tiling3 tl = make_tiling3(D, H, W, s.batch, s3p::kR, Fold3::kAlways);
  p.tl = tl;
  const int64_t per_seg = (int64_t)tl.units_seg / 4 * s.batch;  // blocks
  // a segment's element offsets stay below 2^32 and its plane count below 2^24 (what the critical-vertex queue stores)
  int64_t fit = (((int64_t)1 << 32) - 1) / ((int64_t)H * W);
  fit = std::min<int64_t>(fit, (1 << 24) - 1) / s3p::kChunk * s3p::kChunk;  // (a supported plane has fewer than 2^27 elements)
  // Planes per segment, whole chunks (then segments of equal length): the least of what a launch was found to take (us).  A
  // wave's plane costs 0.35 us, and 0.21 for every wave on its SIMD (a block is a wave on each SIMD of a CU; between the mean
  // and the fullest CU); a segment has about five planes' worth of work besides its own; a block clears and merges its
  // histogram (1.4 us a million counters), and the blocks of an item meet at its counters, or at the rows that they share
  // (10 ns a block, of those that end together).  Over 500 histogram calls (2^17 to 2^26 vertices, 64 to 4096 bins, smooth
  // fields and noise) within 1.5 % of the best of 8 / 16 / 24 / 32 / 40 / 48 planes in the mean: 256^3 uint16 noise, 4096 bins
  // 58 / 44 / 37 / 41 / 38 / -; 193 x 229 x 193 int16, 1024 bins 23.8 / 24.6 / 26.1 / 28.5 / 30.4 / -.
  // Lists that blocks share: 32 planes.  A list that is full still costs every batch its reservation, and the fewer blocks
  // there are the fewer of them wait for one another: white noise of 220 x 376 x 465 bfloat16 5555 us with 8 planes, 4446 with
  // 24, 4201 with 32, smooth fields 93 / 77 / 75.
  // A list for each block: no more room than the float32 plan's lists have, which every type's workspace holds (shorter
  // segments of a ragged volume need more, and the call would take the shared lists: 7 x 73 x 94 x 93 bfloat16 40 us, 21 with
  // 16 planes).
  const size_t room = feed == Feed3dp::kBlockLists ? mid_workspace_bytes(s, 2) : 0;
  double least = 0.0;
  int64_t planes = 0;
  int last = 0;
  for (int aim = s3p::kChunk; feed != Feed3dp::kSharedLists && aim <= 48 && aim <= fit && last != 1; aim += s3p::kChunk) {
    const int segs = (D + aim - 1) / aim;
    if (segs == last) continue;  // (the same segments)
    last = segs;
    const int pl = (D + segs - 1) / segs;
    const int64_t blocks = segs * per_seg;
    if (room && list_room(blocks, block_vertices3dp(s, pl)) > room) continue;
    const int64_t of_item = (int64_t)segs * tl.units_seg / 4;
    const double meet = feed == Feed3dp::kHist ? 0.01 * (double)std::min<int64_t>(1024, of_item) / shared_rows(of_item, bins) : 0.0;
    const double cu = std::max(1.0, (double)blocks / 256.0);
    const double cost = (double)(pl + 5) * (0.35 + 0.105 * (cu + std::ceil(cu))) + meet + 1.4e-6 * (double)blocks * bins;
    if (planes == 0 || cost < least) {
      least = cost;
      planes = aim;
    }
  }
  if (planes == 0) planes = std::min<int64_t>(32, fit);  // (shared lists, or no list for each block: mid_supported)
  p.nseg = (int)((D + planes - 1) / planes);
  p.planes_per_seg = (D + p.nseg - 1) / p.nseg;
  p.grid = dim3((unsigned)(p.nseg * (int64_t)tl.units_seg / 4), (unsigned)s.batch);
  return p;
}
unsigned sweep3dp_shared_list_blocks(const Shape& s) { return plan3dp(s, Feed3dp::kSharedLists).grid.x; }
unsigned sweep3dp_hist_blocks(const Shape& s, int bins) { return plan3dp(s, Feed3dp::kHist, bins).grid.x; }
void sweep3dp_list_plan(const Shape& s, unsigned& per_item, unsigned& vertices) {
  const Plan3dp pl = plan3dp(s, Feed3dp::kBlockLists);
  per_item = pl.grid.x;
  vertices = (unsigned)block_vertices3dp(s, pl.planes_per_seg);
}

// LV: the type also comes with one bin per level (uint8 / uint16 grids without a range)
template <typename T, bool LV = false>
static void launch3dp_t(const void* grid, const Shape& s, bool levels, int bins, const HardHeader* hdr,
                        const float* table, const HistOut& hist, hipStream_t st, const unsigned* run_if, int conv) {
  const Plan3dp pl = plan3dp(s, Feed3dp::kHist, bins);
  const bool tlds = !levels && (size_t)bins * 8 + kQueueBytes3dp <= 60 * 1024;
  const size_t lds = kQueueBytes3dp + (size_t)bins * (tlds ? 8 : 4);
#define ECC_GO(LV, TL, M)                                                                                     \
  hipLaunchKernelGGL((sweep3dp_kernel<T, LV, TL, M>), pl.grid, dim3(256), lds, st, static_cast<const T*>(grid), \
                     (int)s.D, (int)s.H, (int)s.W, s.N, bins, pl.tl, pl.nseg, pl.planes_per_seg, hdr, table, hist, run_if)
#define ECC_MODE(M)                                  \
  do {                                               \
    if constexpr (LV) {                              \
      if (levels) { ECC_GO(true, false, M); break; } \
    }                                                \
    if (tlds) ECC_GO(false, true, M);                \
    else ECC_GO(false, false, M);                    \
  } while (0)
  switch (mode_of_conv(conv)) {
    case kTopCells: ECC_MODE(kTopCells); break;
    case kSuper: ECC_MODE(kSuper); break;
    case kTopSuper: ECC_MODE(kTopSuper); break;
    default: ECC_MODE(kPlain); break;
  }
#undef ECC_MODE
#undef ECC_GO
}

void launch_sweep3dp(const void* grid, const Shape& s, int dtype, bool levels, int bins, const HardHeader* hdr,
                     const float* table, const HistOut& hist, hipStream_t st, const unsigned* run_if, int conv) {
  switch (dtype) {
    case 0: launch3dp_t<uint8_t, true>(grid, s, levels, bins, hdr, table, hist, st, run_if, conv); break;
    case 1: launch3dp_t<uint16_t, true>(grid, s, levels, bins, hdr, table, hist, st, run_if, conv); break;
    case 3: launch3dp_t<F16>(grid, s, false, bins, hdr, table, hist, st, run_if, conv); break;
    case 6: launch3dp_t<Bf16>(grid, s, false, bins, hdr, table, hist, st, run_if, conv); break;
    default: launch3dp_t<int16_t>(grid, s, false, bins, hdr, table, hist, st, run_if, conv); break;
  }
}

template <typename T>
static void launch3dp_list_t(const void* grid, const Shape& s, const ListArgs& la, hipStream_t st, int conv) {
  const Plan3dp pl = plan3dp(s, la.heads ? Feed3dp::kBlockLists : Feed3dp::kSharedLists);
#define ECC_LIST(M)                                                                                             \
  hipLaunchKernelGGL((sweep3dp_list_kernel<T, M>), pl.grid, dim3(256), kQueueBytes3dp, st,                      \
                     static_cast<const T*>(grid), (int)s.D, (int)s.H, (int)s.W, s.N, pl.tl, pl.nseg, pl.planes_per_seg, la)
  switch (mode_of_conv(conv)) {
    case kTopCells: ECC_LIST(kTopCells); break;
    case kSuper: ECC_LIST(kSuper); break;
    case kTopSuper: ECC_LIST(kTopSuper); break;
    default: ECC_LIST(kPlain); break;
  }
#undef ECC_LIST
}
void launch_sweep3dp_list(const void* grid, int dtype, const Shape& s, const ListArgs& la, hipStream_t st, int conv) {
  if (dtype == 3) launch3dp_list_t<F16>(grid, s, la, st, conv);
  else launch3dp_list_t<Bf16>(grid, s, la, st, conv);
}

template <typename T>
static void launch_coeff3dp_t(const void* grid, const Shape& s, int8_t* out, hipStream_t st) {
  const Plan3dp pl = plan3dp(s, Feed3dp::kMap);
  hipLaunchKernelGGL((coeff3dp_kernel<T>), pl.grid, dim3(256), kQueueBytes3dp, st, static_cast<const T*>(grid),
                     (int)s.D, (int)s.H, (int)s.W, s.N, pl.tl, pl.nseg, pl.planes_per_seg, out);
}
void launch_coeff3dp(const void* grid, const Shape& s, int dtype, int8_t* out, hipStream_t st) {
  if (dtype == 0) launch_coeff3dp_t<uint8_t>(grid, s, out, st);
  else launch_coeff3dp_t<uint16_t>(grid, s, out, st);
}

}  // namespace ecc
