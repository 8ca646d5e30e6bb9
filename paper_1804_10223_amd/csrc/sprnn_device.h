// Declarations shared by the device code (sprnn_kernels.hip) and the C ABI (sprnn_api.hip).
#ifndef SPRNN_DEVICE_H_
#define SPRNN_DEVICE_H_

#include <hip/hip_runtime.h>

#include <cstdint>

#include "sprnn.h"

namespace sprnn {

constexpr int kRingSlotsDev = 4;                  // exchange ring depth (power of two)
constexpr uint32_t kSentinelBits = 0x80000000u;   // -0.0f marks a ring element that is not written yet
constexpr int kCtrlStatus = 0;                    // ctrl[0]: non-zero once a spin watchdog tripped
constexpr int kCtrlBarrier = 32;                  // grid-barrier mode: ctrl[32] top counter, ctrl[32 + 16 (1 + g)] counter of group g (64 bytes apart)
constexpr int kCtrlPlacement = kCtrlBarrier + 16 * 9;   // one-XCD mode: two sets (launch parity) of 16 words: workgroups seen per XCD [0..7]
constexpr int kCtrlWords = kCtrlPlacement + 32;
constexpr int kPlacementStride = 16;              // words between the counters of two XCDs where there is room for it, behind a handle's own control words: two share a 128-byte line
constexpr int kOwnCtrlWords = kCtrlWords + 2 * 8 * kPlacementStride;
constexpr uint32_t kStatusWatchdog = 1u, kStatusPlacement = 2u;   // bits of the status word
constexpr int kCellBackward = 100;                // persistent_kernel_for: backward pass of a vanilla cell
constexpr int kCellBackwardGrad = 101;            // the same with the weight gradient fused in
constexpr int kCellLstmBackwardGrad = 102;        // backward pass of the LSTM with the weight gradient fused in
constexpr int kCellGruBackwardGrad = 103;         // backward pass of the GRU with the weight gradient fused in
constexpr int kSoloCopyBytes = 32768;             // single workgroup, form without options: distance of the two LDS copies of h
constexpr int kTimelineSlots = 16;                // 64-bit accumulators per workgroup in the phase timeline
constexpr int kLdsTailBytes = 16 + 8 * kTimelineSlots;   // LDS after h: abort flags, timeline sums

struct KernelArgs {
  const uint32_t* words;      // [grid][NW][block] packed <index,value> words
  const int32_t* lane_row;    // [grid][block]
  const int32_t* wave_words;  // [grid][waves]
  const uint32_t* fill_src;   // column compaction: [grid][fill_rows][block] copy list, or null
  const int32_t* wg_plane;    // column compaction: [grid] bytes of one plane of the workgroup's LDS copy
  const int32_t* wave_early;  // two-part copy: [grid][waves] leading slots of a wavefront's lanes that read only the first part, or null
  const int32_t* lane_sum;    // lane-pool layout: [grid][block] for an output lane: first group of its row | groups << 16
  uint32_t* ring;             // [parts][4][h_bytes / 4]
  uint32_t* ctrl;             // [kCtrlWords]
  const float* x;             // [T][B][R]
  const float* h0;            // [B][H] or null
  const float* c0;            // [B][H] or null (LSTM)
  const float* b_hn;          // [H] or null (GRU: recurrent bias of the candidate)
  const float* aux;           // backward pass: forward outputs h_t, [T][B][H]; LSTM backward: gate values, [T][B][4H]
  float* dh0;                 // backward pass: dL/dh_0, [B][H], or null
  const float* bwd_h0;        // backward pass with weight gradient: h_0, [B][H], or null (zeros)
  const float* side_src;      // backward pass with weight gradient: forward outputs h_t, [T][B][H]
  const int32_t* word_src;    // backward pass with weight gradient: packed word -> CSR position (of the handle's matrix)
  float* dU;                  // backward pass with weight gradient: [nnz] sums, in the handle's CSR order
  float* h_out;               // [T][B][H]
  float* c_out;               // [T][B][H] (LSTM; its backward pass reads the forward cell states from here)
  float* gates_out;           // LSTM forward: [T][B][4H] gate values after their activations, or null (not kept)
  float* dc0;                 // LSTM backward: dL/dc_0, [B][H], or null
  unsigned long long* timeline;  // [grid][16] phase accumulators in wall-clock ticks, or null (off)
  int hidden, T, lanes_per_row, act, h_bytes, poll_delay, spin_limit, sync;
  int fill_rows;              // rounds in the copy list (column compaction)
  int lds_h_bytes;            // bytes of one LDS copy of h (= h_bytes without column compaction)
  int jitter;                 // test aid: seed of pseudo-random pauses (0 = none)
  int tl_wave;                // phase timeline: the wavefront of every workgroup that records it
  int one_xcd;                // 1: the launch has 8 x part_grid workgroups, those of one XCD per part take the work (see persistent_kernel)
  int batch;                  // samples of the call: the layout's batch x parts (x, h_out, ... hold this many per timestep)
  int parts;                  // groups of workgroups that each advance their share of the samples: 1, 2, 4 or 8
  int part_grid;              // workgroups of a part
  uint32_t* placement;        // one-XCD mode: two sets of max(16, 8 placement_stride) words, XCD x's workgroups counted in word x * placement_stride
  int placement_stride;
  uint32_t placement_enough;  // workgroups that an XCD must have received to take a part: part_grid (or, test aid, more than there are)
  uint32_t launch_epoch;      // launches of this handle so far (parity selects the placement counters)
  int seg_rounds;             // > 0: the copy of h is consumed in two parts, its first seg_rounds rounds first (see persistent_kernel)
  int gather_waves;           // lane-pool layout: wavefronts of a workgroup that hold weights (the others own the outputs)
  int index_shift;            // LDS byte offset of a packed word = (word >> 16) << index_shift
  uint32_t step_base;         // global index of the first step of this call (ring slot = index mod 4)
  uint32_t barrier_base;      // grid barriers completed before this call (step t waits at barrier number barrier_base + t)
};

struct StepArgs {
  const int32_t* row_ptr;
  const int32_t* col;
  const uint16_t* val;
  const float* x_t;     // [B][R]
  const float* h_prev;  // [B][H] or null
  const float* c_prev;  // [B][H] or null
  float* h_cur;         // [B][H]
  float* c_cur;         // [B][H]
  int hidden, act;
};

const void* persistent_kernel_for(int batch, int template_words, int cell, bool timeline);   // cell: SPRNN_ACT_* / SPRNN_CELL_*
// (the instantiations live in translation units of their own; persistent_kernel_for forwards to some of these)
const void* persistent_timeline_kernel_for(int batch, int template_words, bool lstm);        // forward pass with the phase timeline
const void* persistent_overlap_kernel_for(int batch, int template_words, bool timeline);     // vanilla forward with the copy of h consumed in two parts (batch <= 4; timeline: batch 4)
// Without run-time options (tagged hand-off, h copied whole among several workgroups, no pauses), for a copy of one, two, three, four
// and more rounds: forward passes, kCellBackward, SPRNN_CELL_*_BACKWARD.  (More than 32 words per lane: from three rounds up.)
const void* persistent_plain1_kernel_for(int batch, int template_words, int cell, bool half);
const void* persistent_plain2_kernel_for(int batch, int template_words, int cell, bool half);
const void* persistent_plain3_kernel_for(int batch, int template_words, int cell, bool half);
const void* persistent_plain4_kernel_for(int batch, int template_words, int cell, bool half);
const void* persistent_plain5_kernel_for(int batch, int template_words, int cell, bool half);
const void* persistent_solo_kernel_for(int batch, int template_words, int cell);              // the same for a single workgroup (per part): forward passes, h of at most kSoloCopyBytes - 16
const void* persistent_half_kernel_for(int batch, int template_words);                       // vanilla forward with h exchanged as binary16 (batch 4, 8)
const void* persistent_narrow_kernel_for(int batch, int template_words);                     // vanilla forward, batch 4, 4-byte gathers (ablation)
const void* persistent_backward_kernel_for(int batch, int template_words, int cell);         // kCellBackward, kCellBackwardGrad
const void* persistent_gated_backward_kernel_for(int batch, int template_words, int cell);   // SPRNN_CELL_*_BACKWARD, kCell{Lstm,Gru}BackwardGrad
hipError_t launch_stepwise(int batch, bool lstm, const StepArgs& a, hipStream_t stream);
// b'[m][n] = sum_k x[m][k] W[n][k] + bias[n] (bias may be null); x [M][K] float32, w [N][K] binary16 bits, out [M][N] float32.
hipError_t launch_project(const float* x, const uint16_t* w, const float* bias, float* out, int M, int N, int K,
                          hipStream_t stream);
const void* pool_kernel_for(int batch, int template_words, int cell, bool timeline = false);                         // lane-pool layout: SPRNN_ACT_*, kCellBackward, kCellBackwardGrad
hipError_t launch_fill(uint32_t* dst, uint32_t value, size_t n, hipStream_t stream);
// Put an exchange ring and its control words into the state a new handle starts from: the first `used_words` 32-bit
// elements of each of the `slots` slots (of `slot_words` each) carry the "not written" mark, the rest of a slot is
// zero, the control words are zero.
hipError_t launch_exchange_reset(uint32_t* ring, size_t slot_words, size_t used_words, int slots, uint32_t* ctrl, int ctrl_words,
                                 hipStream_t stream);

}  // namespace sprnn
#endif
