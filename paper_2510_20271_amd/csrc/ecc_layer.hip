// The two ends of a training step around the soft kernels: the unit direction from its angle(s), and the
// contraction of the uncontracted derivatives (Eq. 9 / Eq. 10 of the paper) with the upstream gradient.
//
// Both touch a few kilobytes to a few megabytes, so launches bound them.  Written as tensor operations the
// contraction of a step on 32 images with 128 thresholds was a matrix-vector product that the GEMM library ran
// in 62 us, a product, a sum and their copies (80 us in all), and the angles' part another dozen small launches
// of 4 to 5 us each; here each is one launch (two for large batches).
#include "ecc_device.h"
#include "ecc_internal.h"

#include <algorithm>

namespace ecc {

// The float32 functions and products that the elementwise tensor operations apply, so that the direction is
// the same to the bit: the order of a tilted field's vertices depends on it.
__global__ void direction_kernel(const float* __restrict__ theta, int ndim, float* __restrict__ u) {
  if (threadIdx.x != 0) return;
  const float t = theta[0];
  if (ndim == 2) {
    u[0] = cosf(t);
    u[1] = sinf(t);
  } else {
    const float p = theta[1], sp = sinf(p);
    u[0] = mul_rn(sp, cosf(t));
    u[1] = mul_rn(sp, sinf(t));
    u[2] = cosf(p);
  }
}

void launch_direction(const float* theta, int ndim, float* u, hipStream_t st) {
  hipLaunchKernelGGL(direction_kernel, dim3(1), dim3(kWave), 0, st, theta, ndim, u);
}

constexpr int kConBlock = 1024;
constexpr int kConWaves = kConBlock / kWave;
constexpr int64_t kConAlone = 32768;  // items x thresholds that one block takes by itself
constexpr int kConGroup = 64;         // thresholds of a block otherwise (fewer: the power of two that holds them)
constexpr int kConItems = 32;         // items a thread adds, about
constexpr int kConMost = 1024;        // blocks
constexpr int kConFinal = 256;

// gu: gradient with respect to the direction; writes it, or carries it on to the angles (theta not null)
__device__ __forceinline__ void contract_store(const double (&gu)[3], int ndim, const float* theta, float* out) {
  if (!theta) {
    for (int k = 0; k < ndim; ++k) out[k] = (float)gu[k];
    return;
  }
  const double t = (double)theta[0], st = sin(t), ct = cos(t);
  if (ndim == 2) {
    out[0] = (float)(ct * gu[1] - st * gu[0]);
  } else {
    const double p = (double)theta[1], sp = sin(p), cp = cos(p);
    out[0] = (float)(sp * (ct * gu[1] - st * gu[0]));
    out[1] = (float)(cp * (ct * gu[0] + st * gu[1]) - sp * gu[2]);
  }
}

// grad_tau[j] = sum_b g[b][j] dtau[b][j],  gu[k] = sum_b sum_j g[b][j] du[b][j][k], in float64 and in a fixed
// order.  A block takes `cols` thresholds (at most 1024) at a time, 1024 / cols threads on each, which share the items
// blockIdx.y per_block .. + per_block.  mid: three doubles a block (launches of several blocks), then [gridDim.y][T] sums
// (launches that split the items).
template <int ND>
__global__ __launch_bounds__(kConBlock) void contract_kernel(const float* __restrict__ g, const float* __restrict__ dtau,
                                                             const float* __restrict__ du,
                                                             const float* __restrict__ theta, int64_t batch, int T,
                                                             int cols, int64_t per_block, float* __restrict__ grad_tau,
                                                             float* __restrict__ grad_dir, double* __restrict__ mid) {
  __shared__ double part[kConBlock];
  __shared__ double wsum[ND][kConWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int slices = kConBlock / cols, col = tid % cols, slice = tid / cols;
  const int blocks = gridDim.x * gridDim.y;
  const int64_t begin = (int64_t)blockIdx.y * per_block, end = min(batch, begin + per_block);
  double gu[ND] = {};
  for (int j0 = blockIdx.x * cols; j0 < T; j0 += gridDim.x * cols) {  // (block-uniform)
    const int j = j0 + col;
    double gt = 0.0;
    if (j < T && slice < slices) {
#pragma unroll 4
      for (int64_t b = begin + slice; b < end; b += slices) {
        const int64_t i = b * T + j;
        const double gv = (double)g[i];
        if (dtau) gt += gv * (double)dtau[i];
        if (du) {
#pragma unroll
          for (int k = 0; k < ND; ++k) gu[k] += gv * (double)du[i * ND + k];
        }
      }
    }
    if (dtau) {
      part[tid] = gt;
      __syncthreads();
      if (slice == 0 && j < T) {
        for (int s = 1; s < slices; ++s) gt += part[s * cols + col];
        if (gridDim.y == 1) grad_tau[j] = (float)gt;
        else mid[(int64_t)blocks * 3 + (int64_t)blockIdx.y * T + j] = gt;
      }
      __syncthreads();
    }
  }
  if (!du) return;
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    double v = gu[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) wsum[k][wv] = v;
  }
  __syncthreads();
  if (tid == 0) {
    double r[3] = {0.0, 0.0, 0.0};
    for (int k = 0; k < ND; ++k)
      for (int w = 0; w < kConWaves; ++w) r[k] += wsum[k][w];
    if (blocks == 1) contract_store(r, ND, theta, grad_dir);
    else
      for (int k = 0; k < 3; ++k) mid[(blockIdx.y * gridDim.x + blockIdx.x) * 3 + k] = r[k];
  }
}

// Adds what the blocks left: a thread per threshold where the items were split in `parts` (> 1), the first block the
// direction's sums.
__global__ __launch_bounds__(kConFinal) void contract_final_kernel(const double* __restrict__ mid, int blocks, int parts,
                                                                   int T, int ndim, const float* __restrict__ theta,
                                                                   float* __restrict__ grad_tau,
                                                                   float* __restrict__ grad_dir) {
  __shared__ double sum[3][kConFinal];
  const int tid = threadIdx.x, j = blockIdx.x * kConFinal + tid;
  if (grad_tau && parts > 1 && j < T) {
    double v = 0.0;
    for (int q = 0; q < parts; ++q) v += mid[(int64_t)blocks * 3 + (int64_t)q * T + j];
    grad_tau[j] = (float)v;
  }
  if (!grad_dir || blockIdx.x != 0) return;  // (block-uniform)
  double r[3] = {0.0, 0.0, 0.0};
  for (int b = tid; b < blocks; b += kConFinal)
    for (int k = 0; k < 3; ++k) r[k] += mid[b * 3 + k];
  for (int k = 0; k < 3; ++k) sum[k][tid] = r[k];
  __syncthreads();
  for (int o = kConFinal / 2; o > 0; o >>= 1) {
    if (tid < o)
      for (int k = 0; k < 3; ++k) sum[k][tid] += sum[k][tid + o];
    __syncthreads();
  }
  if (tid == 0) {
    for (int k = 0; k < 3; ++k) r[k] = sum[k][0];
    contract_store(r, ndim, theta, grad_dir);
  }
}

// One block up to kConAlone products a derivative (32 a thread: 7 us at 16 x 512; a second launch would cost 4 to
// 5 us).  Beyond, blocks of 64 thresholds, or of all of them when there are fewer, that also split the items, so that a
// thread adds about 32 of them, and a closing launch (65535 items, T = 64: 3.7 ms with the thresholds split alone, 70 us so).
struct ContractPlan {
  int cols, groups, parts;
  int64_t per_block;
};
static ContractPlan contract_plan(int64_t batch, int T) {
  ContractPlan p;
  p.cols = kConGroup;
  while (p.cols > 1 && p.cols / 2 >= T) p.cols /= 2;
  if (batch * T <= kConAlone) {
    if (T > kConGroup) p.cols = std::min(kConBlock, (T + kWave - 1) / kWave * kWave);
    p.groups = p.parts = 1;
    p.per_block = batch;
    return p;
  }
  p.groups = (T + p.cols - 1) / p.cols;
  const int64_t each = (int64_t)(kConBlock / p.cols) * kConItems;
  const int64_t parts = std::max<int64_t>(1, std::min<int64_t>((batch + each - 1) / each, kConMost / p.groups));
  p.per_block = (batch + parts - 1) / parts;
  p.parts = (int)((batch + p.per_block - 1) / p.per_block);
  return p;
}
size_t contract_workspace_bytes(int64_t batch, int T) {
  const ContractPlan p = contract_plan(batch, T);
  const size_t n = (size_t)p.groups * p.parts * 3 + (p.parts > 1 ? (size_t)p.parts * T : 0);
  return (n * sizeof(double) + 255) / 256 * 256;
}

hipError_t launch_contract(const float* g, const float* dtau, const float* du, const float* theta, int64_t batch, int T,
                           int ndim, float* grad_tau, float* grad_dir, void* ws, hipStream_t st) {
  const ContractPlan p = contract_plan(batch, T);
  const int blocks = p.groups * p.parts;
  double* mid = static_cast<double*>(ws);
#define ECC_GO(ND)                                                                                                \
  hipLaunchKernelGGL(contract_kernel<ND>, dim3((unsigned)p.groups, (unsigned)p.parts), dim3(kConBlock), 0, st, g, dtau, \
                     du, theta, batch, T, p.cols, p.per_block, grad_tau, grad_dir, mid)
  if (ndim == 2) ECC_GO(2);
  else ECC_GO(3);
#undef ECC_GO
  if (blocks > 1 && (du || p.parts > 1)) {
    const unsigned nb = grad_tau && p.parts > 1 ? (unsigned)((T + kConFinal - 1) / kConFinal) : 1u;
    hipLaunchKernelGGL(contract_final_kernel, dim3(nb), dim3(kConFinal), 0, st, mid, blocks, p.parts, T, ndim, theta,
                       grad_tau, grad_dir);
  }
  return hipGetLastError();
}

}  // namespace ecc
