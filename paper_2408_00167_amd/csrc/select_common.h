// Exact top-r of the per-key scores of one problem by one workgroup of NT = 512 or
// 1024 threads (Method: t = top-r(A_agg, r)): ties to the lower index, output in
// ascending index order.  Shared by the selection kernel and the
// one-workgroup-per-problem step kernel.
//
// The r-th largest value T is found over order-preserving 32-bit keys with LDS histograms.
// The kept set is { key > T } plus the first (r - #greater) candidates with key == T in
// index order, and an ordered scan gives each kept index its output slot, so nothing is
// sorted.
#pragma once

#include <type_traits>

#include "finch_internal.h"

namespace finch {

constexpr int kSelThreads = 1024;          // threads of the selection kernel
constexpr int kSelMaxWaves = 16;           // most waves of any workgroup that selects
// select_keys keeps up to this many candidates per thread in registers
constexpr int kSelRegKeys = 31;
// its histograms: 2048 bins, 32 per lane; a lane's bins stand together, 4 words apart from
// the next lane's, so that the 16-byte reads of neighbouring lanes fall into different banks
constexpr int kSelBinBits = 11;
constexpr int kSelLaneWords = 36;
constexpr int kSelHistWords = 64 * kSelLaneWords;
constexpr int kSelIdxPad = 32;
constexpr int kSelCand = 16;  // a bin with at most this many candidates is resolved directly
__device__ __forceinline__ int sel_hist_at(unsigned bin) { return static_cast<int>(bin + (bin >> 5) * 4u); }

// Monotone map float -> uint32 (larger float <=> larger key); -0 counts as +0.
__device__ __forceinline__ unsigned order_key(float f) {
  const unsigned u = __float_as_uint(f + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The float of an order key.
__device__ __forceinline__ float order_value(unsigned key) {
  return __uint_as_float((key & 0x80000000u) ? key & 0x7fffffffu : ~key);
}

// Inclusive prefix sum over the 64 lanes of a wave without a trip through LDS: shifts
// by 1, 2, 4, 8 inside each row of 16 lanes (zeros shifted in), then lane 15 of every
// even row is added to the row above it and lane 31 to the upper half.
__device__ __forceinline__ int wave_inclusive_scan(int x) {
  int v = x;
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
  return v;
}

// Maximum over the 64 lanes of a wave, the same way.
__device__ __forceinline__ unsigned wave_max_u32(unsigned x) {
  int v = static_cast<int>(x);
  auto mx = [](int a, int b) { return static_cast<unsigned>(a) > static_cast<unsigned>(b) ? a : b; };
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));
  return static_cast<unsigned>(__builtin_amdgcn_readlane(v, 63));
}

constexpr int kSelMaxLayer = 16;  // most score vectors a selection inside a workgroup adds up

struct SelLds {  // LDS scratch of a selection
  alignas(16) int hist[2][kSelHistWords];
  alignas(16) unsigned cand[kSelCand];
  int wave_tot[2][kSelMaxWaves];
  unsigned wave_max[2][kSelMaxWaves];  // largest key and largest complement of a key per wave
  int n_cand;
  int digit[4], remaining[4];
  const float* layer_src[kSelMaxLayer];  // LayerScores: the score vectors of a layer's heads
  int layer_gave_up;                     // the wait for the layer's other workgroups expired
};

// What a selection may be asked beside its result: which candidates lie within a factor `room` of the r-th
// largest score, for non-negative scores.  thr_lo is the order key of the least score / room, thr_hi
// that of the most that score can be * room; n_lo candidates are not below the one, n_hi above the other.
struct SelBand {
  float room;
  unsigned thr_lo = 0u, thr_hi = 0u;
  int n_lo = 0, n_hi = 0;
  float least = 0.f;  // the r-th largest score is not below this
};

// Where a selection takes the score of candidate i from: one vector ...
struct OneScoreVector {
  const FINCH_GLOBAL float* p;
  __device__ __forceinline__ float operator()(int i) const { return p[i]; }
};
// ... or the sum of the L vectors of a layer's heads, added head by head in fp32 (Method:
// "Sum over heads"; the order is that of select_layer, so both give the same bits).  The
// vectors come from other workgroups: they are read past this compute unit's caches.
// W: at least L; all W loads go out together (those past L repeat the last one), so keep it small.
template <int W>
struct LayerScores {
  const float* const* src;  // LDS table of L pointers
  int L;
  __device__ __forceinline__ float operator()(int i) const {
    float v[W];
#pragma unroll
    for (int g = 0; g < W; ++g)
      v[g] = __hip_atomic_load((const FINCH_GLOBAL float*)src[min(g, L - 1)] + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    float t = v[0];
#pragma unroll
    for (int g = 1; g < W; ++g) t = g < L ? t + v[g] : t;
    return t;
  }
};

// Wave 0 only: lane L owns bins 4L..4L+3 of `hist`; finds the bin where the count
// from the top reaches `remaining` and writes that bin and the rank left inside it.
__device__ __forceinline__ void sel_pick_digit(const int* hist, int remaining, int lane, int* digit_out,
                                               int* left_out) {
  const int h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2], h3 = hist[4 * lane + 3];
  const int mine = h0 + h1 + h2 + h3;
  const int prefix = wave_inclusive_scan(mine);
  const int total = __builtin_amdgcn_readlane(prefix, 63);
  const int suffix = total - prefix + mine;  // inclusive sum over lanes >= this one
  const int above = suffix - mine;  // keys in bins of higher lanes
  if (above < remaining && remaining <= suffix) {
    int left = remaining - above;  // >= 1
    int digit;
    if (left <= h3) {
      digit = 3;
    } else if (left <= h3 + h2) {
      digit = 2;
      left -= h3;
    } else if (left <= h3 + h2 + h1) {
      digit = 1;
      left -= h3 + h2;
    } else {
      digit = 0;
      left -= h3 + h2 + h1;
    }
    *digit_out = 4 * lane + digit;
    *left_out = left;
  }
}

// By every wave for itself (all waves read the same histogram and get the same answer, so
// nothing has to be handed round through LDS and no barrier follows): the bin of a
// kSelHistWords histogram where the count from the top reaches `remaining`, the rank left
// inside it and the number of keys in it.  0 < remaining <= number of keys counted.
__device__ __forceinline__ void sel_pick_bin_wave(const int* hist, int remaining, int lane, unsigned& bin_out,
                                                  int& left_out, int& count_out) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const i32x4* mine4 = reinterpret_cast<const i32x4*>(hist + lane * kSelLaneWords);
  i32x4 x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = mine4[i];
  const i32x4 y = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
  const int mine = (y[0] + y[1]) + (y[2] + y[3]);
  const int prefix = wave_inclusive_scan(mine);
  const int total = __builtin_amdgcn_readlane(prefix, 63);
  // keys in the bins of lanes >= this one: total - prefix + mine; the lane that holds the bin
  // is the highest one where that reaches `remaining`
  const unsigned long long m = __ballot(total - prefix + mine >= remaining);
  const int src = m ? 63 - __builtin_clzll(m) : 0;
  const int left = remaining - (total - __builtin_amdgcn_readlane(prefix, src));
  // that lane's 32 bins, one per lane (the upper half of the lanes holds a copy)
  const int h = hist[src * kSelLaneWords + (lane & 31)];
  const int v = wave_inclusive_scan(lane < 32 ? h : 0);
  const int tot32 = __builtin_amdgcn_readlane(v, 31);
  const unsigned m32 = static_cast<unsigned>(__ballot(tot32 - v + h >= left));
  const int b = m32 ? 31 - __builtin_clz(m32) : 0;
  bin_out = static_cast<unsigned>(32 * src + b);
  left_out = left - (tot32 - __builtin_amdgcn_readlane(v, b));
  count_out = __builtin_amdgcn_readlane(h, b);
}

// Exclusive rank of `flag` among the workgroup's threads in thread order, and the
// total.  Two barriers; every thread must call it.
template <int NT>
__device__ __forceinline__ int sel_block_rank(bool flag, int* wave_tot, int lane, int wave, int& total) {
  const unsigned long long b = __ballot(flag);
  const int below = __popcll(b & ((1ull << lane) - 1ull));
  if (lane == 0) wave_tot[wave] = __popcll(b);
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const int x = wave_tot[w];
    if (w < wave) base += x;
    tot += x;
  }
  __syncthreads();
  total = tot;
  return base + below;
}

// Any N: scores are taken from `score_of` again each round.  Writes idx to `gidx` and, if `lidx` is
// not null, also to LDS.  0 < r < N.  Whole workgroup; starts and ends without a barrier.
template <int NT, class Src = OneScoreVector>
__device__ __forceinline__ void select_generic(const Src& score_of, int N, int r, FINCH_GLOBAL int* gidx, int* lidx, SelLds* f,
                                               int tid, int lane, int wave) {
  auto key_at = [&](int i) -> unsigned { return order_key(score_of(i)); };
  unsigned prefix = 0, mask = 0;
  int remaining = r;
  int* hist = f->hist[0];
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int i = tid; i < N; i += NT) {
      const unsigned key = key_at(i);
      if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
    }
    __syncthreads();
    if (wave == 0) sel_pick_digit(hist, remaining, lane, &f->digit[0], &f->remaining[0]);
    __syncthreads();
    prefix |= static_cast<unsigned>(f->digit[0]) << shift;
    mask |= 255u << shift;
    remaining = f->remaining[0];
    __syncthreads();
  }
  const unsigned T = prefix;
  const int need_eq = remaining;  // candidates equal to T that are kept (>= 1)
  int carry_eq = 0, carry_keep = 0;
  for (int base = 0; base < N; base += NT) {
    const int i = base + tid;
    const bool valid = i < N;
    const unsigned key = valid ? key_at(i) : 0u;
    const bool gt = valid && key > T;
    const bool eq = valid && key == T;
    int tot_eq, tot_keep;
    const int eq_rank = carry_eq + sel_block_rank<NT>(eq, f->wave_tot[0], lane, wave, tot_eq);
    const bool keep = gt || (eq && eq_rank < need_eq);
    const int pos = carry_keep + sel_block_rank<NT>(keep, f->wave_tot[0], lane, wave, tot_keep);
    // (pos < r always when the scores hold still; if another workgroup is overwriting them -
    // a layer's workgroup whose bounded wait has expired - the rounds may have counted
    // different values, and nothing may be written past the r places of the output)
    if (keep && pos < r) {
      gidx[pos] = i;
      if (lidx) lidx[pos] = i;
    }
    carry_eq += tot_eq;
    carry_keep += tot_keep;
  }
}

// N <= NT * KMAX.  `keys` (LDS) holds the candidates' order keys, complete before a barrier
// that precedes the call; thread t owns the candidates [t K, (t + 1) K) in registers, K odd
// (so that the lanes of a wave read different LDS banks), and what it keeps goes to
// consecutive places that one scan over the threads hands out.  The histogram bins divide
// the range between the smallest and the largest key evenly, 2048 to a round, so that
// scores of any spread fill them (fixed bits of a key would put nearly all scores of a
// problem into one bin of the first rounds, and LDS atomics on one word take turns).  A
// round narrows the range to the bin the r-th largest falls into; after one or two rounds
// that bin holds few keys, which every wave ranks against each other directly.
// What this is bound by is latency (barriers and dependent LDS reads), so rounds are few
// and every wave reads the histogram for itself.  5500 scores of which 1400 are kept, 512
// threads: 8400 clocks (3.5 us) against 19300 of a four-round radix select with a branch per
// candidate; a third of that is the three barriers and the reads of the histogram.
// Writes the kept indices in ascending order to `lidx` (LDS, kSelIdxPad words more than r) or
// to `gidx`.  0 < r < N.  Whole workgroup; ends without a barrier.
template <int NT, int KMAX, bool LDS_OUT>
__device__ __forceinline__ void select_keys(const unsigned* keys, int N, int r, FINCH_GLOBAL int* gidx, int* lidx,
                                            SelLds* f, int tid, int lane, int wave, SelBand* band = nullptr) {
  constexpr int kWavesNT = NT / 64;
  const int K = ((N + NT - 1) / NT) | 1;
  const int i0 = tid * K;
  const int nk = max(0, min(K, N - i0));  // candidates of this thread
  // order keys of finite scores lie strictly between 0 and the largest unsigned value;
  // registers without a candidate hold 0
  // (no branches per candidate below: a lane without one, or one that has nothing to do, takes
  // the same LDS access to a word that nobody reads)
  unsigned key[KMAX];
  unsigned hi = 0u, nlo = 0u;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) key[k] = keys[min(i0 + k, N - 1)];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    key[k] = k < nk ? key[k] : 0u;
    hi = max(hi, key[k]);
    nlo = max(nlo, key[k] ? ~key[k] : 0u);
  }
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 zero4 = {0, 0, 0, 0};
  for (int i = tid; i < 2 * kSelHistWords / 4; i += NT) reinterpret_cast<i32x4*>(&f->hist[0][0])[i] = zero4;
  if (tid < kSelCand) f->cand[tid] = 0u;
  if (tid == 0) f->n_cand = 0;
  hi = wave_max_u32(hi);
  nlo = wave_max_u32(nlo);
  if (lane == 0) {
    f->wave_max[0][wave] = hi;
    f->wave_max[1][wave] = nlo;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWavesNT; ++w) {
    hi = max(hi, f->wave_max[0][w]);
    nlo = max(nlo, f->wave_max[1][w]);
  }
  // keys [lo, lo + range] are left, `remaining` of them (from the top) are kept
  unsigned lo = ~nlo, range = hi - lo;
  int remaining = r;
  unsigned T = lo;           // keys above T are kept,
  int need_eq = remaining;   // and the first need_eq of those equal to it
  unsigned kth_hi = lo;      // most that the r-th largest key can be
  for (int round = 0; range != 0u; ++round) {
    int* hist = f->hist[round & 1];
    if (round >= 2) {  // (everyone has read it: the barrier of the round before lies between)
      for (int i = tid; i < kSelHistWords; i += NT) hist[i] = 0;
      __syncthreads();
    }
    const int shift = max(0, 32 - __builtin_clz(range) - kSelBinBits);
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      // (keys below lo, and 0, wrap around to more than range; the last words of a lane's kSelLaneWords are padding)
      const unsigned off = key[k] - lo;
      atomicAdd(&hist[off <= range ? sel_hist_at(off >> shift) : lane * kSelLaneWords + 32], 1);
    }
    __syncthreads();
    unsigned bin;
    int count;
    sel_pick_bin_wave(hist, remaining, lane, bin, remaining, count);
    lo += bin << shift;
    range = min((1u << shift) - 1u, range - (bin << shift));
    if (count == remaining) {  // the whole bin is kept
      T = lo - 1u;
      need_eq = 0;
      kth_hi = lo + range;
      break;
    }
    T = lo;
    need_eq = remaining;
    kth_hi = lo;
    if (range != 0u && count <= kSelCand) {
      unsigned in_bin = 0u;
#pragma unroll
      for (int k = 0; k < KMAX; ++k) in_bin |= key[k] - lo <= range ? 1u << k : 0u;
      int at = in_bin ? atomicAdd(&f->n_cand, __popc(in_bin)) : 0;
      while (in_bin) {  // (few lanes have any, hardly one more than one)
        const int k1 = __ffs(static_cast<int>(in_bin)) - 1;
        f->cand[at++ & (kSelCand - 1)] = keys[i0 + k1];
        in_bin &= in_bin - 1u;
      }
      __syncthreads();
      // every row of 16 lanes holds all of them (unused places hold 0) and ranks its own by
      // turning the row
      const unsigned mine = f->cand[lane & (kSelCand - 1)];
      int above = 0, upto = 1;  // keys above this lane's, and not below it
      auto turned = [&](auto ctrl) {
        const unsigned o = static_cast<unsigned>(
            __builtin_amdgcn_update_dpp(0, static_cast<int>(mine), decltype(ctrl)::value, 0xF, 0xF, true));
        above += o > mine ? 1 : 0;
        upto += o >= mine ? 1 : 0;
      };
#define FINCH_TURN(i) turned(std::integral_constant<int, 0x120 + i>{});  /* row_ror:i */
      FINCH_TURN(1) FINCH_TURN(2) FINCH_TURN(3) FINCH_TURN(4) FINCH_TURN(5) FINCH_TURN(6) FINCH_TURN(7) FINCH_TURN(8)
      FINCH_TURN(9) FINCH_TURN(10) FINCH_TURN(11) FINCH_TURN(12) FINCH_TURN(13) FINCH_TURN(14) FINCH_TURN(15)
#undef FINCH_TURN
      const unsigned long long m = __ballot(mine != 0u && above < remaining && remaining <= upto);
      const int src = m ? __ffsll(static_cast<long long>(m)) - 1 : 0;
      T = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(mine), src));
      need_eq = remaining - __builtin_amdgcn_readlane(above, src);
      kth_hi = T;
      break;
    }
  }
  // candidates above T in the low and equal to T in the high half-word
  int mine = 0;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) mine += (key[k] > T ? 1 : 0) + (key[k] == T ? 0x10000 : 0);
  const int incl = wave_inclusive_scan(mine);
  if (band) {
    band->least = order_value(T);
    band->thr_lo = order_key(band->least / band->room);
    band->thr_hi = order_key(order_value(kth_hi) * band->room);
    int in = 0;  // (registers without a candidate hold 0: below any score)
#pragma unroll
    for (int k = 0; k < KMAX; ++k) in += (key[k] >= band->thr_lo ? 1 : 0) + (key[k] > band->thr_hi ? 0x10000 : 0);
    in = wave_inclusive_scan(in);
    if (lane == 63) f->wave_tot[1][wave] = in;
  }
  if (lane == 63) f->wave_tot[0][wave] = incl;
  __syncthreads();
  if (band) {
#pragma unroll
    for (int w = 0; w < kWavesNT; ++w) {
      const int x = f->wave_tot[1][w];
      band->n_lo += x & 0xFFFF;
      band->n_hi += x >> 16;
    }
  }
  int before = incl - mine;
#pragma unroll
  for (int w = 0; w < kWavesNT; ++w) {
    const int x = f->wave_tot[0][w];
    before += w < wave ? x : 0;
  }
  int eq_rank = before >> 16;
  int pos = (before & 0xFFFF) + min(eq_rank, need_eq);
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    const int eq = key[k] == T ? 1 : 0;
    const int keep = (key[k] > T ? 1 : 0) | (eq_rank < need_eq ? eq : 0);
    if (LDS_OUT) {
      lidx[keep ? min(pos, r) : r + (lane & 31)] = i0 + k;
    } else if (keep && pos < r) {
      gidx[pos] = i0 + k;
    }
    pos += keep;
    eq_rank += eq;
  }
}

// select_keys with as many registers as the problem needs.
template <int NT, bool LDS_OUT>
__device__ __forceinline__ void select_keys_any(const unsigned* keys, int N, int r, FINCH_GLOBAL int* gidx, int* lidx,
                                                SelLds* f, int tid, int lane, int wave, SelBand* band = nullptr) {
  if (N <= NT * 3) select_keys<NT, 3, LDS_OUT>(keys, N, r, gidx, lidx, f, tid, lane, wave, band);
  else if (N <= NT * 7) select_keys<NT, 7, LDS_OUT>(keys, N, r, gidx, lidx, f, tid, lane, wave, band);
  else if (N <= NT * 11) select_keys<NT, 11, LDS_OUT>(keys, N, r, gidx, lidx, f, tid, lane, wave, band);
  else select_keys<NT, kSelRegKeys, LDS_OUT>(keys, N, r, gidx, lidx, f, tid, lane, wave, band);
}

// Puts the order keys of the N scores into LDS (no barrier).
// BATCH: candidates whose loads are in flight per thread.
template <int NT, int BATCH, class Src>
__device__ __forceinline__ void sel_stage_keys_batch(const Src& score_of, int N, unsigned* keys, int tid) {
  constexpr int kBatch = BATCH;
  for (int i0 = tid; i0 < N; i0 += NT * kBatch) {
    float v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) v[u] = score_of(min(i0 + u * NT, N - 1));
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (i0 + u * NT < N) keys[i0 + u * NT] = order_key(v[u]);
  }
}

template <int NT, class Src>
__device__ __forceinline__ void sel_stage_keys(const Src& score_of, int N, unsigned* keys, int tid) {
  sel_stage_keys_batch<NT, 8>(score_of, N, keys, tid);
}
// The sums over the L vectors of a layer.
template <int NT>
__device__ __forceinline__ void sel_stage_layer_keys(const float* const* src, int L, int N, unsigned* keys, int tid) {
  if (L <= 8) sel_stage_keys_batch<NT, 4>(LayerScores<8>{src, L}, N, keys, tid);
  else sel_stage_keys_batch<NT, 2>(LayerScores<kSelMaxLayer>{src, L}, N, keys, tid);
}

}  // namespace finch
