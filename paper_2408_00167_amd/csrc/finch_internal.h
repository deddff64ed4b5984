// Internal declarations shared by the host driver and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "finch.h"

namespace finch {

// Keys handled by one workgroup of the fp32 scoring kernels.
constexpr int kTileKeys = 256;
// Prompt rows staged in LDS at a time (larger R is processed in several chunks).
constexpr int kMaxRowChunk = 512;
// bf16 two-pass scoring: threads per workgroup, and the number of slices the keys
// of a problem are cut into (one workgroup streams one slice of about 2400 keys).
constexpr int kStreamThreads = 512;
constexpr int kDefaultSliceKeys = 2400;
__host__ __device__ inline int stream_slices(int n_keys, int slice_keys) {
  const int s = (n_keys + slice_keys / 2) / slice_keys;
  return s < 1 ? 1 : s;
}
// One-workgroup-per-problem path: most prompt rows staged per pass over the keys.
constexpr int kOwnerMaxRowChunk = 256;
// Most LDS the one-workgroup-per-problem kernels keep behind their selection scratch: kept indices
// and order keys of a step with 12000 candidates fit beside 256 prompt rows of 256 bytes.
constexpr size_t kOwnerSelectBytes = 60 * 1024;
// Most kept rows a workgroup of these kernels ranks by score (a bitonic network in registers).
constexpr int kOwnerRankRows = 2048;
// Most problems per layer run that the one-workgroup-per-problem kernels select for together.
constexpr int kOwnerMaxLayer = 16;
// Several workgroups per problem in one launch (cluster_bf16.hip): most workgroups of a launch,
// most key blocks of 32 and candidates per problem, and most prompt rows (their statistics
// are held per workgroup in the workspace).
constexpr int kMaxClusterGrid = 256;
constexpr int kClusterSliceBlocks = 128;
constexpr int kClusterMaxKeys = 15872;  // what a 512-thread selection holds in registers
constexpr int kClusterMaxRows = 4096;
// Words in which the workgroups of such a launch meet.
constexpr int kClusterMeetWords = 32 + 18 * kMaxClusterGrid;
// A workgroup that has waited for others this long in all (100 MHz ticks) does their work itself:
// 0.1 ms, and 1 us for every tile of 32 keys x 32 rows of a slice.  Both passes over a tile take
// 0.22 us (128 channels, 304 tiles: 66 us), so slices that differ in length, or workgroups that
// start late, do not make the others do work that is being done.
constexpr int64_t kClusterHelpTicks = 10000;
constexpr int64_t kClusterHelpTicksPerTile = 100;
// Most LDS a workgroup of the selection kernels asks for.
constexpr size_t kSelLdsBytes = 144 * 1024;
// Rows copied by one workgroup of the compaction kernels.
constexpr int kGatherRows = 64;
// Most kept rows per problem when slots go by score rank (their order keys are held
// in LDS by every workgroup of the problem).
constexpr int kRankMaxRows = 32768;

// Everything the scoring / selection / compaction kernels need besides the
// descriptors.  Passed by value.
struct LaunchParams {
  const finch_problem* probs;  // device descriptors
  int32_t n_problems;
  int32_t group;               // G
  int32_t tiles_max;           // most partial-statistics records of any problem:
                               // ceil(max_p (c+m) / tile_keys), or stream_slices(max) if
                               // tile_keys == 0
  int32_t tile_keys;           // kTileKeys for the fp32 kernels, 0 for the bf16 ones
  int32_t slice_keys;          // target keys per slice of the bf16 kernels
  int32_t merge_in_pass2;      // bf16: pass 2 merges the slice statistics itself (no lse kernel)
  int32_t rpad_max;            // max_p round_up(G*n_que, 32)
  int32_t row_chunk;           // rows staged per pass over the keys (multiple of 32)
  int32_t score_stride;        // floats per problem in ws_scores
  float scale_log2;            // log2(e) / sqrt(d_k)
  float2* stats;               // [P][tiles_max][rpad_max] partial (max, sum) per tile
  float* lse;                  // [P][rpad_max] log2-domain log-sum-exp per prompt row
  float* ws_scores;            // [P][score_stride] used when desc.scores == NULL
  uint32_t lds_bytes;          // dynamic LDS of the launch
  // re-positioning inside the one-workgroup-per-problem kernels (ascending slots)
  int32_t rope_pairing;        // FINCH_ROPE_OFF / _HALF / _INTERLEAVED
  int32_t rank_order;          // kept rows go to the slot of their score's rank (else ascending slots)
  double rope_log2_base;       // log2 of the rotary base
  // layer-wise selection inside the one-workgroup-per-problem kernels: the L workgroups of
  // a run of problems meet through two counters per run (scores out / scores read) and
  // share one error word behind them; zeroed before the launch
  int32_t layer_group;         // L (1: every problem selects for itself)
  int32_t* layer_sync;         // [2 * runs]
  int32_t* layer_err;          // one word behind them
  // several workgroups per problem (cluster_bf16.hip): slices of a problem, the meeting words (what
  // a launch that has ended has left in them, or zeros), and how long a workgroup waits before it helps
  int32_t cluster_slices;
  int32_t* meet;
  int64_t help_ticks;
  int32_t stay_rows;           // whole loop: most kept rows a step may leave where they are (0: none; room for as many notes, 8
                               // bytes each, follows the lds_bytes)
  int32_t est_words;           // whole loop: 4-byte words of LDS for RowEstimates, behind the notes (0: every step makes both passes)
  int32_t* ways;               // whole loop with est_words: one word per step and slot for how the step selected (kWay...), or null
  int64_t spin_ticks;          // longest wait for the other workgroups, in 100 MHz ticks
};

// Launchers; each returns hipGetLastError() after the launch.
unsigned score_grid(const LaunchParams& p);
hipError_t launch_rowstats_bf16(int head_dim, const LaunchParams& p, size_t lds, hipStream_t s);
hipError_t launch_colsum_bf16(int head_dim, const LaunchParams& p, size_t lds, hipStream_t s);
hipError_t launch_rowstats_f32(int head_dim, const LaunchParams& p, size_t lds, hipStream_t s);
hipError_t launch_colsum_f32(int head_dim, const LaunchParams& p, size_t lds, hipStream_t s);
hipError_t launch_lse(const LaunchParams& p, hipStream_t s);
hipError_t launch_select(LaunchParams p, int n_max, hipStream_t s);
hipError_t launch_select_layer(LaunchParams p, int group, float* layer_scores, int n_max, hipStream_t s);
hipError_t set_max_lds_select(size_t bytes);
hipError_t launch_gather(const LaunchParams& p, int row_bytes, int r_max, hipStream_t s);
constexpr int kEstExtraWords = 32;  // words of RowEstimates beside one per prompt row
// how a step of those loops selected: on bounds from one pass (kWayOnce), which settled all keys, or left a list of keys, or
// left all of them (too small for bounds) to the exact scores, or was of no use (its step made both passes: the rows' sums out of range,
// or keys open with rows in several chunks).  0: both passes from the start.
enum : int32_t { kWayOnce = 1, kWaySettled = 2, kWayList = 4, kWayAll = 8, kWayRange = 16, kWayAgain = 32 };
constexpr int kEstMaxRows = 1024;   // most prompt rows it is kept for (4 KB of LDS)
size_t owner_lds_bytes(int head_dim, int row_chunk, int n_max, int r_max, bool rank_order, bool stages);
hipError_t launch_prompt_lse(const LaunchParams& p, int head_dim, bool bf16, int rows_max, hipStream_t s);
hipError_t launch_reposition(const LaunchParams& p, int row_bytes, bool bf16, int r_max, int pairing,
                             bool rank, double base, hipStream_t s);
hipError_t set_max_lds_reposition(size_t bytes);
hipError_t launch_owner_bf16(int head_dim, const LaunchParams& p, int stages, hipStream_t s);
hipError_t launch_owner_loop_bf16(int head_dim, const LaunchParams& p, const int* step_first,
                                  int n_steps, int n_slots, hipStream_t s);
hipError_t set_max_lds_owner(size_t bytes);
hipError_t launch_owner_loop_once_bf16(int head_dim, const LaunchParams& p, const int* step_first,
                                       int n_steps, int n_slots, hipStream_t s);
hipError_t set_max_lds_owner_once(size_t bytes);
// one workgroup per problem for fp32 inputs (prompt rows and rows of the chunk's own tokens)
size_t owner_f32_lds_bytes(int head_dim);
hipError_t launch_owner_f32(int head_dim, const LaunchParams& p, int stages, hipStream_t s);
hipError_t launch_owner_loop_f32(int head_dim, const LaunchParams& p, const int* step_first, int n_steps,
                                 int n_slots, hipStream_t s);
hipError_t set_max_lds_owner_f32(size_t bytes);
// several workgroups per problem, one launch
size_t cluster_lds_bytes(int head_dim, int row_chunk, int slice_blocks, int n_max, int r_max);
hipError_t launch_cluster_bf16(int head_dim, const LaunchParams& p, int n_max, int stages, hipStream_t s);
hipError_t set_max_lds_cluster(size_t bytes);
hipError_t launch_zero_words(int32_t* words, int n, int32_t* one_more, hipStream_t s);
// the same with rows of the chunk's own tokens (desc.q_doc)
hipError_t launch_owner_doc_bf16(int head_dim, const LaunchParams& p, int stages, hipStream_t s);
hipError_t launch_owner_loop_doc_bf16(int head_dim, const LaunchParams& p, const int* step_first,
                                      int n_steps, int n_slots, hipStream_t s);
hipError_t set_max_lds_owner_doc(size_t bytes);
// Raise the dynamic-LDS limit of the scoring kernels of one dtype to `bytes`.
hipError_t set_max_lds_bf16(size_t bytes);
hipError_t set_max_lds_f32(size_t bytes);


// Descriptor pointers are generic; telling the compiler they are global memory
// turns flat loads/stores into global ones (which do not tie up the LDS counter).
#define FINCH_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ const FINCH_GLOBAL T* as_global(const void* p) {
  return (const FINCH_GLOBAL T*)(p);
}
template <typename T>
__device__ __forceinline__ FINCH_GLOBAL T* as_global_mut(void* p) {
  return (FINCH_GLOBAL T*)(p);
}

}  // namespace finch
