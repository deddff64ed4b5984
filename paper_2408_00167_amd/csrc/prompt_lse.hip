// The prompt's share of the softmax denominator (Method: in the model's input the
// prompt follows the context, so a prompt token attends to the context keys and,
// causally, to the prompt tokens up to itself; Background, attention equation).
// For every prompt row i = g*n_que + t of a problem this kernel writes
//   lse_extra[i] = log sum_{j <= t} exp(q_i . kq_j / sqrt(d_k))
// over the prompt's own keys kq, which the scoring kernels add to the row's
// denominator over the context keys.
//
// The work is tiny (R * n_que / 2 dot products per problem), so what counts is that nothing
// runs one after the other: a workgroup takes 16 rows, its waves (four, or one or two for
// prompts of at most 16 or 32 tokens, whose waves would have nothing to do otherwise: 1024 problems of
// 64 rows and 16 prompt keys 33.8 us with four waves, 16.6 with one) share out the blocks
// of 16 prompt keys, and a block's 256 logits are one chain of fp64 matrix instructions
// (every product is exact, sums are fp64).  Each lane then holds the logits of one key
// against four rows; maxima and sums stay in fp64.  One layer of 8 KV heads, 256 rows and 64
// prompt keys each: 38 us with one row per four lanes and the keys one after the other, 6.4 us
// now (most of it the first loads' latency).
#include "finch_internal.h"

namespace finch {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kRowsPerGroup = 16, kMaxLseWaves = 4;

// Element e of a run of 16-byte pieces as fp64 (exact); E = elements per piece.
template <int E>
__device__ __forceinline__ double element(const u32x4* v, int e) {
  if (E == 4) return static_cast<double>(__uint_as_float(v[e >> 2][e & 3]));
  const unsigned w = v[e >> 3][(e & 7) >> 1];
  return static_cast<double>(__uint_as_float((e & 1) ? (w & 0xFFFF0000u) : (w << 16)));
}

}  // namespace

template <int D, int E, int kLseWaves>
__global__ __launch_bounds__(64 * kLseWaves) void prompt_lse_rows(LaunchParams prm, int blocks_per_problem) {
  __shared__ double red[2][kLseWaves][kRowsPerGroup];  // maxima and sums per wave
  const int p = blockIdx.x / blocks_per_problem;
  const finch_problem pb = prm.probs[p];
  const int n_que = pb.n_que;
  const int R = prm.group * n_que;
  const int row0 = (blockIdx.x - p * blocks_per_problem) * kRowsPerGroup;
  if (row0 >= R) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, part = lane >> 4;
  // v_mfma_f64_16x16x4: lane (col, part) gives row / key `col`, k-element `part` of a step, and
  // receives rows 4 v + part, key `col`.  The order of the k-elements is free as long as both
  // sides share it: part p takes the p-th quarter of the channels, read as whole pieces.
  constexpr int kSteps = D / 4, kPieces = kSteps / E;
  const FINCH_GLOBAL u32x4* qp =
      as_global<u32x4>(pb.q) + static_cast<size_t>(min(row0 + col, R - 1)) * (D / E) + part * kPieces;
  u32x4 q[kPieces];
#pragma unroll
  for (int i = 0; i < kPieces; ++i) q[i] = qp[i];
  int lim[4];  // last key each of this lane's rows sees
  int last = 0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    lim[v] = min(row0 + 4 * v + part, R - 1) % n_que;
    last = max(last, lim[v]);
  }
  last = max(last, __shfl_xor(last, 16));
  last = max(last, __shfl_xor(last, 32));
  const double scale = 1.0 / sqrt(static_cast<double>(D));
  double m[4], z[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    m[v] = -__builtin_inf();
    z[v] = 0.0;
  }
  for (int key0 = wave * 16; key0 <= last; key0 += 16 * kLseWaves) {
    const int key = key0 + col;
    const FINCH_GLOBAL u32x4* kp =
        as_global<u32x4>(pb.k_que) + static_cast<size_t>(min(key, n_que - 1)) * (D / E) + part * kPieces;
    u32x4 k[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) k[i] = kp[i];
    f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
      acc[s & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(element<E>(q, s), element<E>(k, s), acc[s & 1], 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (key <= lim[v]) {
        const double s = (acc[0][v] + acc[1][v]) * scale;
        const double mn = fmax(m[v], s);
        z[v] = z[v] * exp(m[v] - mn) + exp(s - mn);  // exp(-inf) = 0 on the first key
        m[v] = mn;
      }
    }
  }
  // over the 16 keys of a row, then over the waves
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    double mx = m[v];
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    double zs = m[v] == -__builtin_inf() ? 0.0 : z[v] * exp(m[v] - mx);
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) zs += __shfl_xor(zs, o);
    if (col == 0) {
      red[0][wave][4 * v + part] = mx;
      red[1][wave][4 * v + part] = zs;
    }
  }
  __syncthreads();
  if (tid < kRowsPerGroup && row0 + tid < R) {
    double mx = red[0][0][tid];
#pragma unroll
    for (int w = 1; w < kLseWaves; ++w) mx = fmax(mx, red[0][w][tid]);
    double zs = 0.0;  // (every row sees at least key 0, so mx is finite)
#pragma unroll
    for (int w = 0; w < kLseWaves; ++w) zs += red[1][w][tid] * exp(red[0][w][tid] - mx);
    as_global_mut<float>(pb.lse_extra)[row0 + tid] = static_cast<float>(mx + log(zs));
  }
}

namespace {

template <int kLseWaves>
hipError_t launch_with_waves(const LaunchParams& p, int head_dim, bool bf16, int rows_max, hipStream_t s) {
  const int bpp = (rows_max + kRowsPerGroup - 1) / kRowsPerGroup;
  const dim3 block(64 * kLseWaves);
  // (a launch has fewer than 2^32 threads: enormous batches go in several)
  const int per_launch = (1 << 23) / bpp > 0 ? (1 << 23) / bpp : 1;
  for (int first = 0; first < p.n_problems; first += per_launch) {
    LaunchParams q = p;
    q.probs = p.probs + first;
    const int n = p.n_problems - first < per_launch ? p.n_problems - first : per_launch;
    const dim3 grid(static_cast<unsigned>(bpp) * static_cast<unsigned>(n));
    if (bf16 && head_dim == 128) {
      hipLaunchKernelGGL((prompt_lse_rows<128, 8, kLseWaves>), grid, block, 0, s, q, bpp);
    } else if (bf16 && head_dim == 64) {
      hipLaunchKernelGGL((prompt_lse_rows<64, 8, kLseWaves>), grid, block, 0, s, q, bpp);
    } else if (!bf16 && head_dim == 128) {
      hipLaunchKernelGGL((prompt_lse_rows<128, 4, kLseWaves>), grid, block, 0, s, q, bpp);
    } else if (!bf16 && head_dim == 64) {
      hipLaunchKernelGGL((prompt_lse_rows<64, 4, kLseWaves>), grid, block, 0, s, q, bpp);
    } else {
      return hipErrorInvalidValue;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_prompt_lse(const LaunchParams& p, int head_dim, bool bf16, int rows_max, hipStream_t s) {
  if (p.n_problems == 0 || rows_max <= 0) return hipSuccess;
  const int key_blocks = (rows_max / p.group + 15) / 16;  // of the longest prompt
  if (key_blocks <= 1) return launch_with_waves<1>(p, head_dim, bf16, rows_max, s);
  if (key_blocks <= 2) return launch_with_waves<2>(p, head_dim, bf16, rows_max, s);
  return launch_with_waves<kMaxLseWaves>(p, head_dim, bf16, rows_max, s);
}

}  // namespace finch
