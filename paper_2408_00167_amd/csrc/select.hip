// Selection kernel: exact top-r of the per-key scores of one problem (Method:
// t = top-r(A_agg, r)), ties to the lower index, output in ascending index order.
//
// One workgroup per problem; the algorithm is in select_common.h.  Problems whose order keys
// fit into the launch's LDS (prm.lds_bytes) take it there; larger ones re-read their
// scores (L2) in every round.
#include "select_common.h"

namespace finch {

namespace {

// LDS of a selection over at most n_max candidates: scratch and order keys, or the scratch
// alone if they do not fit.
size_t select_lds_bytes(int n_max) {
  const size_t all = sizeof(SelLds) + static_cast<size_t>(n_max) * 4;
  return n_max <= kSelThreads * kSelRegKeys && all <= kSelLdsBytes ? all : sizeof(SelLds);
}

// Top-r of `score_of` into idx by the whole workgroup, 0 < r < N.
__device__ __forceinline__ void select_problem(const LaunchParams& prm, char* smem, const FINCH_GLOBAL float* scores, int N,
                                               int r, FINCH_GLOBAL int* idx, int tid, int lane, int wave) {
  SelLds* lds = reinterpret_cast<SelLds*>(smem);
  const OneScoreVector src = {scores};
  if (sizeof(SelLds) + static_cast<size_t>(N) * 4 <= prm.lds_bytes && N <= kSelThreads * kSelRegKeys) {
    unsigned* keys = reinterpret_cast<unsigned*>(smem + sizeof(SelLds));
    sel_stage_keys<kSelThreads>(src, N, keys, tid);
    __syncthreads();
    select_keys_any<kSelThreads, false>(keys, N, r, idx, nullptr, lds, tid, lane, wave);
  } else {
    select_generic<kSelThreads>(src, N, r, idx, nullptr, lds, tid, lane, wave);
  }
}

}  // namespace

__global__ __launch_bounds__(kSelThreads) void select_topr(LaunchParams prm) {
  extern __shared__ __align__(16) char smem[];
  const int p = blockIdx.x;
  const finch_problem pb = prm.probs[p];
  const int N = pb.c + pb.m;
  const int r = min(pb.r, N);
  if (r <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const FINCH_GLOBAL float* scores = as_global<float>(
      pb.scores ? pb.scores : prm.ws_scores + static_cast<size_t>(p) * prm.score_stride);
  FINCH_GLOBAL int* idx = as_global_mut<int>(pb.idx);
  if (r >= N) {  // nothing to decide: keep every candidate
    for (int i = tid; i < N; i += kSelThreads) idx[i] = i;
    return;
  }
  select_problem(prm, smem, scores, N, r, idx, tid, lane, wave);
}

// Layer-wise selection (Method: "Sum over heads" - the scores of all heads of a layer
// are added before ONE top-r per layer): the problems of a batch come in runs of
// `group` consecutive descriptors, the KV heads of one layer, with the same c, m
// and r.  One workgroup per run adds the run's score vectors head by head (a
// fixed order), keeps the sum in `layer_scores` (one slot of prm.score_stride floats
// per run), selects on it and writes the same indices to every problem of the run.
__global__ __launch_bounds__(kSelThreads) void select_layer(LaunchParams prm, int group,
                                                            float* layer_scores) {
  extern __shared__ __align__(16) char smem[];
  const int run = blockIdx.x;
  const int p0 = run * group;
  const finch_problem pb0 = prm.probs[p0];
  const int N = pb0.c + pb0.m;
  const int r = min(pb0.r, N);
  if (r <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (r >= N) {  // nothing to decide: every head keeps every candidate
    for (int g = 0; g < group; ++g) {
      FINCH_GLOBAL int* idx = as_global_mut<int>(prm.probs[p0 + g].idx);
      for (int i = tid; i < N; i += kSelThreads) idx[i] = i;
    }
    return;
  }
  FINCH_GLOBAL float* total = as_global_mut<float>(layer_scores + static_cast<size_t>(run) * prm.score_stride);
  for (int g = 0; g < group; ++g) {  // head by head; a thread only ever touches its own elements
    const finch_problem pb = prm.probs[p0 + g];
    const FINCH_GLOBAL float* sc = as_global<float>(
        pb.scores ? pb.scores : prm.ws_scores + static_cast<size_t>(p0 + g) * prm.score_stride);
    for (int i = tid; i < N; i += kSelThreads) total[i] = g == 0 ? sc[i] : total[i] + sc[i];
  }
  __syncthreads();  // the sums this workgroup wrote are read back by other threads below
  FINCH_GLOBAL int* idx0 = as_global_mut<int>(pb0.idx);
  select_problem(prm, smem, total, N, r, idx0, tid, lane, wave);
  __syncthreads();
  for (int g = 1; g < group; ++g) {
    FINCH_GLOBAL int* idx = as_global_mut<int>(prm.probs[p0 + g].idx);
    for (int t = tid; t < r; t += kSelThreads) idx[t] = idx0[t];
  }
}

hipError_t launch_select_layer(LaunchParams p, int group, float* layer_scores, int n_max, hipStream_t s) {
  if (p.n_problems == 0) return hipSuccess;
  p.lds_bytes = static_cast<uint32_t>(select_lds_bytes(n_max));
  hipLaunchKernelGGL(select_layer, dim3(p.n_problems / group), dim3(kSelThreads), p.lds_bytes, s, p, group,
                     layer_scores);
  return hipGetLastError();
}

hipError_t launch_select(LaunchParams p, int n_max, hipStream_t s) {
  if (p.n_problems == 0) return hipSuccess;
  p.lds_bytes = static_cast<uint32_t>(select_lds_bytes(n_max));
  hipLaunchKernelGGL(select_topr, dim3(p.n_problems), dim3(kSelThreads), p.lds_bytes, s, p);
  return hipGetLastError();
}

hipError_t set_max_lds_select(size_t bytes) {
  if (bytes < kSelLdsBytes) return hipErrorInvalidValue;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&select_topr),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kSelLdsBytes));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&select_layer), hipFuncAttributeMaxDynamicSharedMemorySize,
                             static_cast<int>(kSelLdsBytes));
}

}  // namespace finch
