// Weight gradient on the sparsity pattern, dU[p] = sum_m a[m][row(p)] * b[m][col(p)] over m = (timestep, sample): the
// non-recurrent half of the backward pass, a dense product of two tall matrices sampled at the nonzeros.
//
// On this chip the dense product on the matrix cores is the faster way to it for matrices up to about 4000 x 4000 whatever
// their density: the multiply-adds of the nonzeros alone on the vector units, with h and delta in LDS, took 1.6 times as
// long at 30 % and no less at 2 % (there the fetch of the operands bounds both).  Wider matrices, whose dense elements
// outgrow what a step costs otherwise, and very short calls go to sprnn_wgrad_lanes.hip (see sprnn_wgrad_rule.h).
//
// Both operands are binary32 and stay so: each is split, while it is staged, into three bfloat16 numbers (round to nearest)
// whose sum is the number exactly, 3 x 8 bits (times a power of two that keeps the parts of the smallest numbers normal, 1-4 %
// of the call; what is too large for that, and infinities, are added up again at the end of the kernel); six of the nine
// products go through v_mfma_f32_16x16x32_bf16 with binary32 sums, the three that are left out are below 2^-26 of the product
// of the two numbers, a quarter of the rounding of one binary32 product (measured against binary64: 4.8e-7 of the gradient's
// norm over 1024 vectors, a chain of binary32 multiply-adds 5.7e-7).
//
// A workgroup of sixteen wavefronts (4 x 4 over the tile) owns a tile of TM rows x TN columns of dU and walks m in slabs
// of 32.  The operands are [m][row] and [m][column]: a lane fetches eight consecutive m of one column (128 consecutive
// bytes per half wavefront, any alignment), splits them, and each part is one 16-byte LDS write in the layout the matrix
// instructions read ([row][m], see piece_at).  Two LDS stages; while slab s is multiplied, slab s + 1 is split and stored
// and slabs s + 2, s + 3 are in flight from memory in two register sets.  At the end the tile goes through LDS and every
// row's nonzeros are picked out of it and stored in CSR order.
//
// Measured (one call, before: every workgroup brought all of h into LDS in every timestep): 2304 x 2304 at 30 %, 1024
// vectors 288 -> 73 us; 4096 x 1024 at 20 %, 1024 vectors 177 -> 52; 1792 at 10 % 247 -> 50; 701 at 15 %, 154 vectors
// 76 -> 13.  Matrix instructions are busy 45 % of the launch (2304 x 2304), with 135 other vector instructions (most of them
// the split) to 36 of theirs per wavefront and slab: a
// workgroup's wavefronts meet at a barrier per slab, and around it neither runs.
#include <algorithm>

#include "sprnn_persistent.h"
#include "sprnn_wgrad.h"

namespace sprnn {
namespace {

typedef __bf16 bfloatx8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kSlab = 32;                      // m per slab
constexpr int kPitch = kSlab * 2;              // bytes of one row of one part in LDS: four 16-byte pieces
constexpr float kOperandScale = 0x1p24f;       // both operands, so sums carry its square: with it every binary32 number,
constexpr float kSumScale = 0x1p-48f;          // the smallest included, is three normal bfloat16 numbers
constexpr int plane_bytes(int tm, int tn) { return (tm + tn) * kPitch; }
constexpr int stage_bytes(int tm, int tn) { return 3 * plane_bytes(tm, tn); }
constexpr int lds_bytes(int tm, int tn) { return std::max(2 * stage_bytes(tm, tn), tm * (tn + 4) * 4); }

// Where piece q (eight m) of a row sits in the row.  Rows of 64 bytes repeat their banks every four rows, so the pieces
// change places with bits 1 to 3 of the row: the sixteen lanes that one LDS cycle serves when a matrix instruction's
// operand is read (16 rows x 4 pieces) then hit all sixteen 16-byte groups of the 64 banks, and the eight lanes of a write
// (8 rows x one piece) all eight groups of 32 banks.
__device__ __forceinline__ int piece_at(int row, int q) {
  const int g = (row >> 2) & 3;
  return q ^ ((((g ^ (g >> 1)) & 1) << 1) | (g >> 1)) ^ ((row >> 1) & 1);
}

// A buffer whose address is the same for the whole wavefront, said in a way that the compiler sees.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_buffer(const void* base, int bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(lo | hi << 32), 0, __builtin_amdgcn_readfirstlane(bytes), kBufWord3);
}
__device__ __forceinline__ bool is_finite(float v) { return (__builtin_bit_cast(uint32_t, v) & 0x7f800000u) != 0x7f800000u; }
__device__ __forceinline__ float load_f32(__amdgpu_buffer_rsrc_t buf, uint32_t byte) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(buf, (int)byte, 0, 0));
}

// (x0, x1) rounded to bfloat16, packed; x0 and x1 become what is left of them (exactly)
__device__ __forceinline__ uint32_t take_bf16(float& x0, float& x1) {
  typedef __bf16 bfloatx2 __attribute__((ext_vector_type(2)));
  bfloatx2 v;
  v[0] = (__bf16)x0;
  v[1] = (__bf16)x1;
  const uint32_t bits = __builtin_bit_cast(uint32_t, v);
  x0 -= __builtin_bit_cast(float, bits << 16);
  x1 -= __builtin_bit_cast(float, bits & 0xffff0000u);
  return bits;
}

// Vector m's element of one row or column.
__device__ __forceinline__ float element(const WGradOperand& o, int m, int at) {
  if (m >= o.shift) return o.x[(size_t)(m - o.shift) * o.ld + at];
  return o.first ? o.first[(size_t)m * o.ld + at] : 0.0f;
}

__device__ __forceinline__ float column_element(const WGradArgs& p, int m, int at) {
  const float v = element(p.b, m, at);
  return p.gate && at >= p.gate_from ? v * p.gate[(size_t)m * p.gate_ld + at - p.gate_from] : v;
}

// GATED: the column side is multiplied by p.gate while it is staged (the GRU's recurrent gradient out of dL/db' and the reset
// gate, for callers who do not keep it).  The second register set holds the gate then, so one slab is in flight, not two:
// about as fast, and the recurrence has one output less to write (GRU 1100 at 30 %, batch 4, 128 steps, whole call 355 us
// against 371 with that output and 414 with the sums inside the recurrence).
template <int TM, int TN, bool GATED>
__global__ __launch_bounds__(kThreads) void weight_grad_kernel(const WGradArgs p, const TileGrid grid) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int kPlane = plane_bytes(TM, TN), kStage = stage_bytes(TM, TN);
  constexpr int MI = TM / 64, NI = TN / 64;    // 16 x 16 blocks of one wavefront along rows and columns
  constexpr int kUnits = (TM + TN) / 32 * 2;   // fetch units of a slab: 32 columns x 16 m
  constexpr int kMine = (kUnits + kWaves - 1) / kWaves;      // ... of one wavefront
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
  // Workgroups are dealt round-robin to the eight XCDs.  Each XCD takes a rectangle of the grid of tiles, so that the rows
  // and columns its tiles share come out of its own L2 (the launch has room for the largest rectangle eight times).
  const int xcd = (int)blockIdx.x % 8, turn = (int)blockIdx.x / 8, xr = xcd % grid.parts_m, xc = xcd / grid.parts_m;
  const int parts_n = 8 / grid.parts_m;
  const int m_lo = xr * grid.tiles_m / grid.parts_m, m_n = (xr + 1) * grid.tiles_m / grid.parts_m - m_lo;
  const int n_lo = xc * grid.tiles_n / parts_n, n_n = (xc + 1) * grid.tiles_n / parts_n - n_lo;
  if (turn >= m_n * n_n) return;
  const int r0 = (m_lo + turn % m_n) * TM, tile_c = n_lo + turn / m_n, c0 = tile_c * TN;
  const int rows = p.a.ld, cols = p.b.ld;

  // ---- the nonzeros this lane will store: half wavefronts take one row of the tile each, TM / 32 turns
  constexpr int kTurns = TM / 32;
  int first[kTurns], last[kTurns];
  auto find_nonzeros = [&]() {
#pragma unroll
    for (int i = 0; i < kTurns; ++i) {
      const int r = r0 + i * 32 + wave * 2 + (lane >> 5);
      first[i] = r < rows ? p.starts[(size_t)tile_c * rows + r] : 0;
      last[i] = r < rows ? p.starts[(size_t)(tile_c + 1) * rows + r] : 0;
    }
  };
  if constexpr (!GATED) find_nonzeros();

  // ---- fetch: unit u of a slab is 32 rows (or, beyond TM / 32 * 2 units, columns) x half of its m; a lane takes eight m
  struct Source { uint32_t from, to, gate; };
  Source src[kMine];
  auto unit_of = [&](int i) { return wave + kWaves * i; };
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    const int u = unit_of(i), slot = (u >> 1) * 32 + (lane & 31);        // row of the LDS planes
    const bool row_side = slot < TM;
    const int x = row_side ? r0 + slot : c0 + slot - TM, ld = row_side ? rows : cols;
    const int k8 = (u & 1) * 2 + (lane >> 5);
    src[i].from = x < ld ? (uint32_t)(k8 * 8 * ld + x) * 4u : (uint32_t)kOutOfRange;
    src[i].to = (uint32_t)(slot * kPitch + piece_at(slot, k8) * 16);
    if constexpr (GATED)
      src[i].gate = !row_side && x >= p.gate_from && x < ld ? (uint32_t)(k8 * 8 * p.gate_ld + x - p.gate_from) * 4u : (uint32_t)kOutOfRange;
  }
  // The buffer of a slab starts at the slab's first vector that exists in memory and ends with its last one: offsets
  // before or beyond it (rows of h_0, the end of the sequence, lanes without a column) read zero.
  float pre[2][kMine][8];
  auto fetch = [&](float (&v)[kMine][8], int m0, auto is_first) {
    constexpr bool kFirst = decltype(is_first)::value;   // slab 0: the only one that may begin with vectors of `first`
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      if (kUnits % kWaves != 0 && unit_of(i) >= kUnits) continue;
      const bool row_side = (unit_of(i) >> 1) * 32 < TM;
      const float* const x = row_side ? p.a.x : p.b.x;
      const float* const head = row_side ? p.a.first : p.b.first;
      const int ld = row_side ? rows : cols, shift = row_side ? p.a.shift : p.b.shift;
      const int start = kFirst ? 0 : m0 - shift, have = kFirst ? min(p.vectors, kSlab) - shift : min(p.vectors - m0, kSlab);
      const __amdgpu_buffer_rsrc_t buf = uniform_buffer(x + (size_t)start * ld, max(have, 0) * ld * 4);
      const uint32_t step = (uint32_t)ld * 4u;
      uint32_t at = src[i].from - (kFirst ? (uint32_t)shift * step : 0u);
      asm volatile("" : "+v"(at));             // (else the compiler keeps all offsets in registers for the whole loop)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[i][e] = load_f32(buf, at + e * step);
      if (kFirst && head) {                   // (where one of the two buffers ends the other begins: zero bits merge)
        const __amdgpu_buffer_rsrc_t hbuf = uniform_buffer(head, shift * ld * 4);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[i][e] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v[i][e]) | __builtin_bit_cast(uint32_t, load_f32(hbuf, src[i].from + e * step)));
      }
    }
  };
  auto fetch_gate = [&](float (&g)[kMine][8], int m0) {
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      if ((kUnits % kWaves != 0 && unit_of(i) >= kUnits) || (unit_of(i) >> 1) * 32 < TM) continue;
      const __amdgpu_buffer_rsrc_t buf = uniform_buffer(p.gate + (size_t)m0 * p.gate_ld, max(min(p.vectors - m0, kSlab), 0) * p.gate_ld * 4);
      uint32_t at = src[i].gate;
      asm volatile("" : "+v"(at));
#pragma unroll
      for (int e = 0; e < 8; ++e) g[i][e] = load_f32(buf, at + e * (uint32_t)p.gate_ld * 4u);
    }
  };
  auto store = [&](float (&v)[kMine][8], int i, int stage) {
    if (kUnits % kWaves != 0 && unit_of(i) >= kUnits) return;
    if constexpr (GATED) {
      if ((unit_of(i) >> 1) * 32 >= TM) {
        const bool gated = src[i].gate != (uint32_t)kOutOfRange;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[i][e] *= gated ? pre[1][i][e] : 1.0f;
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[i][e] *= kOperandScale;
#pragma unroll
    for (int part = 0; part < 3; ++part) {
      i32x4 q;
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] = (int)take_bf16(v[i][2 * e], v[i][2 * e + 1]);
      *reinterpret_cast<i32x4*>(lds + stage * kStage + part * kPlane + src[i].to) = q;
    }
  };

  // ---- multiply: this wavefront's blocks of the tile
  const int wm = wave & 3, wn = wave >> 2;
  const uint32_t a_at = (uint32_t)((wm * (TM / 4) + (lane & 15)) * kPitch + piece_at(lane, lane >> 4) * 16);
  const uint32_t b_at = (uint32_t)((TM + wn * (TN / 4) + (lane & 15)) * kPitch + piece_at(lane, lane >> 4) * 16);
  f32x4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto part_of = [&](uint32_t at, int stage, int part, int block) {
    return *reinterpret_cast<const bfloatx8*>(lds + stage * kStage + part * kPlane + at + block * 16 * kPitch);
  };

  const int slabs = (p.vectors + kSlab - 1) / kSlab;
  auto step = [&](float (&v)[kMine][8], int s) {
    const int stage = s & 1;
    bfloatx8 b[3][NI];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int j = 0; j < NI; ++j) b[q][j] = part_of(b_at, stage, q, j);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      bfloatx8 a[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) a[q] = part_of(a_at, stage, q, i);
      // smallest products first
      constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[pa[q]], b[pb[q]][j], acc[i][j], 0, 0, 0);
      if (i < kMine) store(v, i, stage ^ 1);   // slab s + 1, split in the shadow of the products
    }
#pragma unroll
    for (int i = MI; i < kMine; ++i) store(v, i, stage ^ 1);
    fetch(v, (s + (GATED ? 2 : 3)) * kSlab, std::false_type());   // (beyond the last slab this reads nothing)
    if constexpr (GATED) fetch_gate(pre[1], (s + 2) * kSlab);
    // one matrix instruction, then vector instructions in its shadow
#pragma unroll
    for (int q = 0; q < 6 * MI * NI; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
    }
    lds_barrier();
  };
  if constexpr (GATED) {
    if (slabs > 0) {
      fetch(pre[0], 0, std::true_type());
      fetch_gate(pre[1], 0);
#pragma unroll
      for (int i = 0; i < kMine; ++i) store(pre[0], i, 0);
      fetch(pre[0], kSlab, std::false_type());
      fetch_gate(pre[1], kSlab);
      lds_barrier();
      for (int s = 0; s < slabs; ++s) step(pre[0], s);
    }
  } else if (slabs > 0) {
    fetch(pre[0], 0, std::true_type());
    fetch(pre[1], kSlab, std::false_type());
#pragma unroll
    for (int i = 0; i < kMine; ++i) store(pre[0], i, 0);
    fetch(pre[0], 2 * kSlab, std::false_type());
    lds_barrier();
    int s = 0;
    for (; s + 2 <= slabs; s += 2) {
      step(pre[1], s);
      step(pre[0], s + 1);
    }
    if (s < slabs) step(pre[1], s);
  }

  if constexpr (GATED) find_nonzeros();      // (at the start they would cost registers that the gate needs)

  // ---- the tile through LDS, rows of TN + 4 floats; then the nonzeros of each row in CSR order
  float* const tile = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        tile[(wm * (TM / 4) + i * 16 + (lane >> 4) * 4 + v) * (TN + 4) + wn * (TN / 4) + j * 16 + (lane & 15)] = acc[i][j][v];
  const __amdgpu_buffer_rsrc_t colbuf = uniform_buffer(p.col, p.nnz * 4), out = uniform_buffer(p.dU, p.nnz * 4);
  constexpr int kPieces = TN / 32;
  int col[kTurns][kPieces];
#pragma unroll
  for (int i = 0; i < kTurns; ++i)
#pragma unroll
    for (int q = 0; q < kPieces; ++q) {
      const int k = first[i] + q * 32 + (lane & 31);
      col[i][q] = __builtin_amdgcn_raw_buffer_load_b32(colbuf, k < last[i] ? k * 4 : kOutOfRange, 0, 0);
    }
  lds_barrier();
  bool odd = false;
#pragma unroll
  for (int i = 0; i < kTurns; ++i)
#pragma unroll
    for (int q = 0; q < kPieces; ++q) {
      const int k = first[i] + q * 32 + (lane & 31);
      const bool mine = k < last[i];
      const float v = tile[(i * 32 + wave * 2 + (lane >> 5)) * (TN + 4) + (mine ? col[i][q] - c0 : 0)];
      const bool good = is_finite(v);
      odd |= mine && !good;
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v * kSumScale), out, mine && good ? k * 4 : kOutOfRange, 0, 0);
    }

  // ---- sums that left the range of the split (an infinite or NaN operand, one of 2^104 or more, a sum of 2^80 or more):
  // the same lanes add them up again, one multiply-add per vector, which is what the numbers themselves give
  if (!__any(odd)) return;
#pragma unroll 1
  for (int i = 0; i < kTurns; ++i) {
    const int r = r0 + i * 32 + wave * 2 + (lane >> 5);
    if (r >= rows) continue;
    const int end = p.starts[(size_t)(tile_c + 1) * rows + r];
    for (int k = p.starts[(size_t)tile_c * rows + r] + (lane & 31); k < end; k += 32) {
      const int c = p.col[k];
      if (is_finite(tile[(r - r0) * (TN + 4) + c - c0])) continue;
      float sum = 0.0f;
      for (int m = 0; m < p.vectors && sum == sum; ++m) sum = fmaf(element(p.a, m, r), column_element(p, m, c), sum);
      p.dU[k] = sum;
    }
  }
}

__global__ __launch_bounds__(256) void tile_starts_kernel(const int32_t* row_ptr, const int32_t* col, int rows, int tile_cols, int entries, int32_t* starts) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= entries) return;
  const int r = i % rows, limit = i / rows * tile_cols;
  int lo = row_ptr[r], hi = row_ptr[r + 1];
  while (lo < hi) {
    const int mid = lo + (hi - lo) / 2;
    if (col[mid] < limit) lo = mid + 1;
    else hi = mid;
  }
  starts[i] = lo;
}

template <bool GATED>
const void* kernel_of(WGradTile t) {
  switch (t.rows * 1000 + t.cols) {
    case 64064: return (const void*)weight_grad_kernel<64, 64, GATED>;
    case 64128: return (const void*)weight_grad_kernel<64, 128, GATED>;
    case 128128: return (const void*)weight_grad_kernel<128, 128, GATED>;
    case 128192: return (const void*)weight_grad_kernel<128, 192, GATED>;
    default: return nullptr;
  }
}

}  // namespace

hipError_t launch_tile_starts(const int32_t* row_ptr, const int32_t* col, int rows, int cols, int tile_cols, int32_t* starts,
                              hipStream_t stream) {
  int entries = rows * ((cols + tile_cols - 1) / tile_cols + 1);
  void* a[] = {(void*)&row_ptr, (void*)&col, (void*)&rows, (void*)&tile_cols, (void*)&entries, (void*)&starts};
  return hipLaunchKernel((const void*)tile_starts_kernel, dim3((entries + 255) / 256), dim3(256), a, 0, stream);
}

hipError_t launch_weight_gradient(const WGradArgs& args, WGradTile tile, hipStream_t stream) {
  const void* const kernel = args.gate ? kernel_of<true>(tile) : kernel_of<false>(tile);
  if (!kernel) return hipErrorInvalidValue;
  int most = 0;
  TileGrid grid = tile_grid(args.a.ld, args.b.ld, tile, &most);
  void* a[] = {(void*)&args, (void*)&grid};
  return hipLaunchKernel(kernel, dim3((unsigned)most * 8), dim3(kThreads), a, (size_t)lds_bytes(tile.rows, tile.cols), stream);
}

hipError_t prepare_weight_gradient(WGradTile tile, bool gated) {   // two stages exceed the 64 KB of LDS a launch may ask for by default
  const void* const kernel = gated ? kernel_of<true>(tile) : kernel_of<false>(tile);
  return kernel ? hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(tile.rows, tile.cols)) : hipErrorInvalidValue;
}

}  // namespace sprnn
