// Device code of libsprnn: the forward instantiations of the persistent kernel (sprnn_persistent.h), the
// per-timestep comparison kernel and small helpers.
#include <algorithm>

#include "sprnn_persistent.h"

namespace sprnn {

// ------------------------------------------------------------------------------------------------
// Per-timestep comparison kernel: one launch per step, CSR weights re-read from device memory,
// one wavefront per weight row (vanilla) or per hidden unit (LSTM: its four gate rows in turn).
template <int B, bool LSTM>
__global__ __launch_bounds__(256) void stepwise_kernel(const StepArgs p) {
  const int lane = threadIdx.x & 63;
  const int unit = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int H = p.hidden;
  if (unit >= H) return;
  constexpr int G = LSTM ? 4 : 1;
  float pre[G][B];
#pragma unroll
  for (int q = 0; q < G; ++q) {
    const int row = q * H + unit;
    float acc[B];
#pragma unroll
    for (int b = 0; b < B; ++b) acc[b] = 0.0f;
    for (int k = p.row_ptr[row] + lane; k < p.row_ptr[row + 1]; k += 64) {
      const float wv = half_bits_to_float(p.val[k]);
      const int c = p.col[k];
#pragma unroll
      for (int b = 0; b < B; ++b) acc[b] = fmaf(wv, p.h_prev ? p.h_prev[(size_t)b * H + c] : 0.0f, acc[b]);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      float v = acc[b];
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
      pre[q][b] = v + p.x_t[(size_t)b * (G * H) + row];
    }
  }
  if (lane != 0) return;
#pragma unroll
  for (int b = 0; b < B; ++b) {
    if constexpr (LSTM) {
      const float cp = p.c_prev ? p.c_prev[(size_t)b * H + unit] : 0.0f;
      const float c = sigmoidf_(pre[1][b]) * cp + sigmoidf_(pre[0][b]) * tanhf_(pre[2][b]);
      p.c_cur[(size_t)b * H + unit] = c;
      p.h_cur[(size_t)b * H + unit] = sigmoidf_(pre[3][b]) * tanhf_(c) + 0.0f;
    } else {
      p.h_cur[(size_t)b * H + unit] = activate(p.act, pre[0][b]);
    }
  }
}

// Fill a device buffer with one 32-bit pattern (used instead of a memset node so that callers may capture it).
__global__ void fill_kernel(uint32_t* dst, uint32_t value, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) dst[i] = value;
}

__global__ void exchange_reset_kernel(uint32_t* ring, size_t slot_words, size_t used_words, int slots, uint32_t* ctrl, int ctrl_words) {
  const size_t first = blockIdx.x * (size_t)blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = first; i < slot_words * (size_t)slots; i += stride) ring[i] = (i % slot_words) < used_words ? kSentinelBits : 0u;
  for (size_t i = first; i < (size_t)ctrl_words; i += stride) ctrl[i] = 0u;
}

// ------------------------------------------------------------------------------------------------
const void* persistent_kernel_for(int batch, int template_words, int cell, bool timeline) {
  const int kind = cell == SPRNN_CELL_LSTM ? 1 : (cell == SPRNN_CELL_GRU ? 2 : 0);
  const bool forward = cell >= SPRNN_ACT_RELU && cell <= SPRNN_CELL_GRU;
  if (timeline) {   // the phase timeline is built for the forward pass of the vanilla and LSTM cells only
    if (!forward || kind == 2) return nullptr;
    return persistent_timeline_kernel_for(batch, template_words, kind == 1);
  }
  if (cell == kCellBackward || cell == kCellBackwardGrad) return persistent_backward_kernel_for(batch, template_words, cell);
  if (!forward) return persistent_gated_backward_kernel_for(batch, template_words, cell);
  if (kind == 2) return pick_b<2, false>(batch, template_words);
  return kind == 1 ? pick_b<1, false>(batch, template_words) : pick_b<0, false>(batch, template_words);
}

hipError_t launch_stepwise(int batch, bool lstm, const StepArgs& a, hipStream_t stream) {
  const int waves_per_block = 4;
  dim3 grid((a.hidden + waves_per_block - 1) / waves_per_block), block(waves_per_block * 64);
#define SPRNN_LAUNCH_STEP(BB)                                                                          \
  if (lstm) hipLaunchKernelGGL((stepwise_kernel<BB, true>), grid, block, 0, stream, a);              \
  else hipLaunchKernelGGL((stepwise_kernel<BB, false>), grid, block, 0, stream, a);
  switch (batch) {
    case 1: SPRNN_LAUNCH_STEP(1) break;
    case 2: SPRNN_LAUNCH_STEP(2) break;
    case 4: SPRNN_LAUNCH_STEP(4) break;
    case 8: SPRNN_LAUNCH_STEP(8) break;
    default: return hipErrorInvalidValue;
  }
#undef SPRNN_LAUNCH_STEP
  return hipGetLastError();
}

hipError_t launch_fill(uint32_t* dst, uint32_t value, size_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const int block = 256;
  const int grid = (int)((n + block - 1) / block < 1024 ? (n + block - 1) / block : 1024);
  hipLaunchKernelGGL(fill_kernel, dim3(grid), dim3(block), 0, stream, dst, value, n);
  return hipGetLastError();
}

hipError_t launch_exchange_reset(uint32_t* ring, size_t slot_words, size_t used_words, int slots, uint32_t* ctrl, int ctrl_words,
                                 hipStream_t stream) {
  const size_t n = std::max(slot_words * (size_t)slots, (size_t)ctrl_words);
  const int block = 256;
  const int grid = (int)std::min<size_t>((n + block - 1) / block, 256);
  hipLaunchKernelGGL(exchange_reset_kernel, dim3(std::max(grid, 1)), dim3(block), 0, stream, ring, slot_words, used_words, slots, ctrl, ctrl_words);
  return hipGetLastError();
}

}  // namespace sprnn
