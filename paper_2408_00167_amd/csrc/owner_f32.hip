// One workgroup per problem for fp32 Q/K/V: both scoring passes
// (Background, attention equation; Method: prompt-guided sub-matrix, sum over heads and
// prompt rows), then the top-r and the compaction of owner_body.h, for one step or for
// the whole chunk loop in one launch (Method: Document Segmentation).  Rows come from the
// prompt and, with desc.q_doc, from the chunk's own tokens under the causal mask with the
// Method's normalisation step read per row.
//
// Rows go through in chunks of 16, keys in tiles of 16: a tile of logits is one chain of fp64
// matrix instructions (v_mfma_f64_16x16x4: every fp32 product is exact there, sums are fp64),
// which leaves one row and four keys to a lane.  The softmax runs in fp32 in the log2 domain
// with a running (maximum, sum) per row and lane, merged over the workgroup.  Logits of up to
// kHeldTiles tiles (1024 candidates) wait in LDS for the second pass; beyond that they are
// formed again.  This serves fp32 problems of modest size, where a step is
// latency: 320 candidates and 16 rows of 64 channels take 10 us (40 with a key per thread on the
// vector ALU, where every fp64 multiply-add came with two conversions); large ones are better
// off spread over the chip by the kernels per stage.
#include "owner_body.h"

namespace finch {

namespace {

constexpr int kRowChunk = 16;  // rows at a time
constexpr int kTile = 16;      // keys of a tile
constexpr int kHeldTiles = 64; // tiles whose logits are kept from pass 1 to pass 2

typedef double f64x4 __attribute__((ext_vector_type(4)));

struct F32Lds {
  float4* held;    // [kHeldTiles][64 lanes]
  float* lse;      // [kRowChunk]
  float2* wred;    // [waves][kRowChunk]
  char* sel;       // selection scratch
};

__device__ __forceinline__ F32Lds f32_lds(char* smem) {
  F32Lds l;
  l.held = reinterpret_cast<float4*>(smem);
  smem += sizeof(float4) * 64 * kHeldTiles;
  l.lse = reinterpret_cast<float*>(smem);
  l.wred = reinterpret_cast<float2*>(smem + sizeof(float) * kRowChunk);
  l.sel = smem + ((sizeof(float) * kRowChunk + sizeof(float2) * kOwnWaves * kRowChunk + 15) & ~size_t{15});
  return l;
}

// A lane's share of an operand of the fp64 matrix instructions: row `lane & 15` of sixteen, the
// (lane >> 4)-th quarter of its channels (which k-step takes which channel is free as long as
// both operands agree).
template <int D>
__device__ __forceinline__ void f32_load_quarter(const float* row, int lane, u32x4 (&x)[D / 16]) {
  const FINCH_GLOBAL u32x4* rp = as_global<u32x4>(row + (lane >> 4) * (D / 4));
#pragma unroll
  for (int s = 0; s < D / 16; ++s) x[s] = rp[s];
}
template <int D>
__device__ __forceinline__ void f32_load_keys(const finch_problem& pb, int N, int tile, int lane, u32x4 (&x)[D / 16]) {
  const int key = min(tile * kTile + (lane & 15), N - 1);
  const float* base = static_cast<const float*>(key < pb.c ? pb.k_cache : pb.k_chunk);
  f32_load_quarter<D>(base + static_cast<size_t>(key < pb.c ? key : key - pb.c) * D, lane, x);
}

// Dot products of 16 keys and 16 rows: element v of a lane is key 4 v + (lane >> 4), row lane & 15.
template <int D>
__device__ __forceinline__ void f32_dots(const u32x4 (&k)[D / 16], u32x4 (&q)[D / 16], float (&dot)[4]) {
  if (D > 64) {  // (128 channels of a row as fp64 would not fit for good: they are widened tile by tile)
#pragma unroll
    for (int s = 0; s < D / 16; ++s) asm volatile("" : "+v"(q[s]));
  }
  f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int s = 0; s < D / 4; ++s)
    acc[s & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(__uint_as_float(k[s >> 2][s & 3])),
                                                      static_cast<double>(__uint_as_float(q[s >> 2][s & 3])), acc[s & 1], 0, 0, 0);
#pragma unroll
  for (int v = 0; v < 4; ++v) dot[v] = static_cast<float>(acc[0][v] + acc[1][v]);
}

// Sum over the 16 lanes of a row of lanes (lane ^ 8, ^ 7, ^ 2, ^ 1 through DPP; fixed order).
__device__ __forceinline__ float sum_over16(float x) {
  x += from_lane_dpp<0x128>(x);
  x += from_lane_dpp<0x141>(x);
  x += from_lane_dpp<0x4E>(x);
  x += from_lane_dpp<0xB1>(x);
  return x;
}

// One step of one problem by the whole workgroup; see own_step_body for `step_probs`,
// `epoch` and the return value.
template <int D, bool ROT>
__device__ __forceinline__ bool own_step_body_f32(const LaunchParams& prm, const finch_problem& pb, int slot,
                                                  int stages, char* smem, const finch_problem* step_probs,
                                                  int epoch) {
  const int N = pb.c + pb.m;
  if (N == 0) return false;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const F32Lds l = f32_lds(smem);
  const float sc = prm.scale_log2;
  float* gscores = pb.scores ? pb.scores : prm.ws_scores + static_cast<size_t>(slot) * prm.score_stride;
  FINCH_GLOBAL float* dst = as_global_mut<float>(gscores);
  const int L = prm.layer_group;
  const bool layered = stages && L > 1 && pb.r > 0 && pb.r < N;
  int* const sync_words = (stages && L > 1) ? prm.layer_sync + 2 * (slot / L) : nullptr;
  if (sync_words && epoch > 0) {
    // (see own_step_body: the scores of the step before may still be read by the layer's other workgroups)
    if (tid == 0) {
      const long long t0 = wall_clock64();
      while (__hip_atomic_load(sync_words + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < L * epoch) {
        __builtin_amdgcn_s_sleep(8);
        if (wall_clock64() - t0 > prm.spin_ticks) {
          atomicOr(prm.layer_err, 1);
          break;
        }
      }
    }
    __syncthreads();
  }
  const size_t sel_bytes = prm.lds_bytes - static_cast<size_t>(l.sel - smem);
  unsigned* const lkeys = (stages && pb.r > 0 && pb.r < N) ? own_sel_keys(l.sel, sel_bytes, 0, N, pb.r) : nullptr;
  // rows: the prompt's (they see every key), then those of the chunk's own tokens, head by head
  const int Rp = pb.q ? prm.group * pb.n_que : 0;
  const int Rd = (pb.q_doc && pb.m > 0) ? prm.group * pb.m : 0;
  const int n_rows = Rp + Rd;
  const int n_tiles = (N + kTile - 1) / kTile;
  const bool hold = n_tiles <= kHeldTiles;
  const int col = lane & 15, part = lane >> 4;
  u32x4 kf[D / 16], kn[D / 16];
  for (int row0 = 0; row0 < n_rows; row0 += kRowChunk) {
    const int rows = min(kRowChunk, n_rows - row0);
    // this lane's row: its keys end at `lim` (a row past the end sees none)
    const int row = row0 + min(col, rows - 1);
    const int lim = col >= rows ? 0 : row < Rp ? N : min(N, pb.c + (row - Rp) % pb.m + 1);
    if (wave < n_tiles) f32_load_keys<D>(pb, N, wave, lane, kf);
    u32x4 q[D / 16];
    f32_load_quarter<D>(row < Rp ? static_cast<const float*>(pb.q) + static_cast<size_t>(row) * D
                                 : static_cast<const float*>(pb.q_doc) + static_cast<size_t>(row - Rp) * D,
                        lane, q);
    // ---- pass 1: running (maximum, sum exp2) of this lane's row over its keys
    float m = -kInf, z = 0.f;
    auto tile_stats = [&](const float (&dot)[4], int tile) {
      float s[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) s[v] = tile * kTile + 4 * v + part < lim ? dot[v] * sc : -kInf;
      const float mn = fmaxf(fmaxf(fmaxf(m, s[0]), fmaxf(s[1], s[2])), s[3]);
      const float mu = mn == -kInf ? 0.f : mn;
      z = z * fast_exp2(m - mu) + (fast_exp2(s[0] - mu) + fast_exp2(s[1] - mu)) + (fast_exp2(s[2] - mu) + fast_exp2(s[3] - mu));
      m = mn;
    };
    for (int tile = wave; tile < n_tiles; tile += kOwnWaves) {
      if (tile + kOwnWaves < n_tiles) f32_load_keys<D>(pb, N, tile + kOwnWaves, lane, kn);
      float dot[4];
      f32_dots<D>(kf, q, dot);
      if (hold) l.held[tile * 64 + lane] = make_float4(dot[0], dot[1], dot[2], dot[3]);
      tile_stats(dot, tile);
#pragma unroll
      for (int s = 0; s < D / 16; ++s) kf[s] = kn[s];
    }
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float m2 = __shfl_xor(m, o);
      const float z2 = __shfl_xor(z, o);
      merge_stats(m, z, m2, z2);
    }
    if (lane < kRowChunk) l.wred[wave * kRowChunk + lane] = make_float2(m, z);
    if (!hold) f32_load_keys<D>(pb, N, wave, lane, kf);
    __syncthreads();
    if (tid < kRowChunk) {
      float lse = kInf;  // rows past the end add exp2(-inf) = 0
      if (tid < rows) {
        float2 a = l.wred[tid];
#pragma unroll
        for (int w = 1; w < kOwnWaves; ++w) {
          const float2 c = l.wred[w * kRowChunk + tid];
          merge_stats(a.x, a.y, c.x, c.y);
        }
        lse = a.x + fast_log2(a.y);
        if (row < Rp) {
          if (pb.lse_extra) lse = widen_lse(lse, as_global<float>(pb.lse_extra)[row]);
        } else {
          // normalisation step: the row's weights times (keys it sees) / (c + m)
          lse -= fast_log2(static_cast<float>(lim) / static_cast<float>(N));
        }
      }
      l.lse[tid] = lse;
    }
    __syncthreads();
    // ---- pass 2: this chunk's rows added to the scores of the keys
    const float lse = l.lse[col];
    auto tile_sums = [&](const float (&dot)[4], int tile) {
      float mine = 0.f;  // lane col == v takes the sum of key 4 v + part
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float w = tile * kTile + 4 * v + part < lim ? fast_exp2(__builtin_fmaf(dot[v], sc, -lse)) : 0.f;
        const float u = sum_over16(w);
        mine = col == v ? u : mine;
      }
      const int key = tile * kTile + 4 * col + part;
      if (col < 4 && key < N) {
        const float val = row0 == 0 ? mine : dst[key] + mine;
        if (layered) __hip_atomic_store(dst + key, val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else dst[key] = val;
        if (lkeys) lkeys[key] = order_key(val);
      }
    };
    if (hold) {  // (a wave reads back what it has written itself)
      for (int tile = wave; tile < n_tiles; tile += kOwnWaves) {
        const float4 h = l.held[tile * 64 + lane];
        const float dot[4] = {h.x, h.y, h.z, h.w};
        tile_sums(dot, tile);
      }
    } else {
      for (int tile = wave; tile < n_tiles; tile += kOwnWaves) {
        if (tile + kOwnWaves < n_tiles) f32_load_keys<D>(pb, N, tile + kOwnWaves, lane, kn);
        float dot[4];
        f32_dots<D>(kf, q, dot);
        tile_sums(dot, tile);
#pragma unroll
        for (int s = 0; s < D / 16; ++s) kf[s] = kn[s];
      }
    }
    __syncthreads();  // after the last chunk: the scores are out
  }
  if (n_rows == 0) own_no_rows(gscores, lkeys, N, tid);
  if (!stages) return false;
  KeptRows kept;
  own_finish_step<D / 4, 4, ROT>(prm, pb, slot, N, dst, l.sel, sel_bytes, lkeys, step_probs, epoch, layered, sync_words, tid, kept);
  return layered;
}

template <int D, bool ROT>
__global__ __launch_bounds__(kOwnThreads) void owner_step_f32(LaunchParams prm, int stages) {
  extern __shared__ __align__(16) char smem[];
  const int p = own_slot_of(blockIdx.x, gridDim.x, stages ? prm.layer_group : 1);
  const finch_problem pb = load_problem(prm.probs + p);
  own_step_body_f32<D, ROT>(prm, pb, p, stages, smem, prm.probs, 0);
}

template <int D, bool ROT>
__global__ __launch_bounds__(kOwnThreads) void owner_loop_f32(LaunchParams prm, const int* step_first, int n_steps) {
  extern __shared__ __align__(16) char smem[];
  const int slot = own_slot_of(blockIdx.x, gridDim.x, prm.layer_group);
  int epoch = 0;
  for (int s = 0; s < n_steps; ++s) {
    const int first = step_first[s];
    if (slot >= step_first[s + 1] - first) break;  // slots are filled from the front
    const finch_problem pb = load_problem(prm.probs + uni(first + slot));
    if (own_step_body_f32<D, ROT>(prm, pb, slot, /*stages=*/1, smem, prm.probs + first, epoch)) ++epoch;
    // the rows this step wrote are the next step's cache: complete before it reads
    __syncthreads();
  }
}

template <typename F>
bool with_f32_step_kernel(int head_dim, bool rot, F f) {
  if (head_dim == 128) rot ? f(&owner_step_f32<128, true>) : f(&owner_step_f32<128, false>);
  else if (head_dim == 64) rot ? f(&owner_step_f32<64, true>) : f(&owner_step_f32<64, false>);
  else return false;
  return true;
}
template <typename F>
bool with_f32_loop_kernel(int head_dim, bool rot, F f) {
  if (head_dim == 128) rot ? f(&owner_loop_f32<128, true>) : f(&owner_loop_f32<128, false>);
  else if (head_dim == 64) rot ? f(&owner_loop_f32<64, true>) : f(&owner_loop_f32<64, false>);
  else return false;
  return true;
}

}  // namespace

size_t owner_f32_lds_bytes(int head_dim) {
  (void)head_dim;
  const size_t fixed = sizeof(float4) * 64 * kHeldTiles + sizeof(float) * kRowChunk + sizeof(float2) * kOwnWaves * kRowChunk + 16;
  return fixed + sizeof(SelLds) + kOwnerSelectBytes;
}

hipError_t launch_owner_f32(int head_dim, const LaunchParams& p, int stages, hipStream_t s) {
  if (p.n_problems <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(p.n_problems)), block(kOwnThreads);
  const bool ok = with_f32_step_kernel(head_dim, p.rope_pairing != FINCH_ROPE_OFF || p.rank_order, [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, p.lds_bytes, s, p, stages);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_owner_loop_f32(int head_dim, const LaunchParams& p, const int* step_first, int n_steps,
                                 int n_slots, hipStream_t s) {
  if (n_slots <= 0 || n_steps <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(n_slots)), block(kOwnThreads);
  const bool ok = with_f32_loop_kernel(head_dim, p.rope_pairing != FINCH_ROPE_OFF || p.rank_order, [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, p.lds_bytes, s, p, step_first, n_steps);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t set_max_lds_owner_f32(size_t bytes) {
  hipError_t err = hipSuccess;
  auto set = [&](auto kern) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
    if (e != hipSuccess) err = e;
  };
  for (int d = 0; d < 2; ++d)
    for (int rot = 0; rot < 2; ++rot) {
      with_f32_step_kernel(d ? 128 : 64, rot != 0, set);
      with_f32_loop_kernel(d ? 128 : 64, rot != 0, set);
    }
  return err;
}

}  // namespace finch
