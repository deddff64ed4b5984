// One workgroup per problem for a whole prefill step, bf16 Q/K/V on gfx950: scoring
// pass 1, the merge of the row statistics, scoring pass 2, top-r and compaction
// (Method: attention of the prompt rows over cache + chunk keys, sum over heads and
// prompt rows, t = top-r(A_agg, r), Managing the Cache) run back to back inside the
// workgroup that owns the problem.
//
// Nothing is exchanged between workgroups, so there are no kernel boundaries, no
// atomics on device memory and no waits (but for layer groups, whose workgroups exchange
// scores): the row statistics are merged in LDS, and the scores' order keys and the kept
// indices stay there for top-r and compaction where they fit; else the workgroup reads back
// what it wrote itself.  The keys are read a second time right after the first pass, while
// the memory-side cache still holds most of them.  Workgroups are 8 waves (two per
// SIMD, up to 256 registers each), one per CU; the batch should have about as many problems as the chip has CUs (or a
// multiple), which the host checks before it picks this path.
//
// The arithmetic (and therefore every output bit of scores given the same block
// assignment rules) follows the two-pass kernels: MFMA 32x32x16 bf16 with one
// prompt row per lane, log2-domain softmax, pass 1 with a fixed assignment of key
// blocks to waves, pass 2 with key blocks handed out by an LDS counter.
//
// Templates of the one-workgroup-per-problem kernels; instantiated by
// owner_bf16.hip (prompt rows only) and owner_doc_bf16.hip (rows of the chunk's own
// tokens as well).
#pragma once

#include "reposition_common.h"
#include "score_common.h"
#include "select_common.h"

namespace finch {

namespace {

// Phase timers, compiled in only with -DFINCH_PHASE_TIMERS (the build script's --phase-timers
// writes that variant to a library of its own; the normal library has none of this).  Thread 0
// of every workgroup adds the ticks of the 100 MHz wall clock it spent between two marks to
// the phase's total: 0 staging of the prompt rows, 1 pass 1 of wave 0, 2 wave 0's wait at the
// barrier after pass 1, 3 merge of the row statistics, 4 pass 2 of wave 0, 5 its wait at the
// barrier after pass 2, 6 top-r, 7 compaction.  Each translation unit has its own totals.
#ifdef FINCH_PHASE_TIMERS
static __device__ unsigned long long finch_phase_ticks[8];
#define FINCH_PHASE_BEGIN() unsigned long long phase_last_ = wall_clock64()
#define FINCH_PHASE(i)                                        \
  do {                                                        \
    if (threadIdx.x == 0) {                                   \
      const unsigned long long now_ = wall_clock64();         \
      atomicAdd(&finch_phase_ticks[i], now_ - phase_last_);   \
      phase_last_ = now_;                                     \
    }                                                         \
  } while (0)
#else
#define FINCH_PHASE_BEGIN() do { } while (0)
#define FINCH_PHASE(i) do { } while (0)
#endif

constexpr int kOwnThreads = 512;
constexpr int kOwnWaves = kOwnThreads / 64;

// The thread's index, through an empty asm: in the whole-loop kernels the compiler would otherwise compute
// everything that depends only on it once for all steps, and keep it in registers through every
// phase.  So each phase asks for it anew.
__device__ __forceinline__ int own_thread() {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  return tid;
}

__device__ __forceinline__ int own_next_block(int* counter, int lane) {
  int v = 0;
  if (lane == 0) v = atomicAdd(counter, 1);
  return __builtin_amdgcn_readfirstlane(v);
}

// Rows that stay where they are.  Inside the whole-loop kernels a step need not move the rows it
// keeps if a later step overwrites all of its k_out / v_out and the step in between is the only
// one to read them (owner_loop_bf16 decides; the host has checked that nothing else of the
// slot touches those buffers): it only notes in LDS where each kept row lies, and the next step
// reads its cache there.  Kept rows are moved when they are wanted in their place, at the end of
// the loop.  With re-positioning that holds for the values only: a key is rounded every time
// it moves.
struct KeptRows {
  int* at = nullptr;         // LDS: kept row t lies at[t] 16-byte pieces behind k0, and at[cap + t] behind v0
  int cap = 0;
  const char* k0 = nullptr;
  const char* v0 = nullptr;
  bool mapped = false;       // the cache rows of this step are where `at` says, not in k_cache / v_cache
  bool stay = false;         // this step leaves its kept rows where they are
};

// Keys that stay open cost their part of the second pass, and finding them and another selection 5 to 6 us: the
// time of 500 (192 rows, long steps) to 1200 keys (32 rows) there.  So a step is worth trying while both come to well less
// than that pass; half of it for what they may come to, as what is open is known from the step before only.  est_fixed is in
// keys of one row block.  Loops of 256 problems, time : with two passes at every step, keys spread evenly and relevant keys that
// stand clear: with this 0.86 to 1.05 and 0.71 to 0.94; with 600 whatever the rows 0.86 to 1.07 and 0.71 to 0.95; with 3000 (6000
// for 64 channels) 0.87 to 1.05 and 0.72 to 0.98, as tries are left out that would have settled all but a few keys.
template <int D>
__device__ constexpr int est_fixed(int qb) {
  return (300 + 200 * qb) * 128 / D;
}
constexpr float kEstRoom = 1.15f;      // factor around the r-th largest score in which a slot without experience looks for others
constexpr float kEstSpread = 16.f;     // log2 of the largest spread that is of use
// Largest |log2 z_i|: sums of 1024 rows stay below 2^70, and the terms below 2^-126 that a row's sum of 2^-60 and more has
// lost are less than 2^-52 of it.
constexpr float kEstReach = 60.f;
constexpr float kEstLeast = 0x1p-60f;  // smaller key sums may have lost terms below the least exponent

// Selection on one pass over the keys.  The weight of row i at key j is exp2(logit - lse_i), and lse_i is only known
// when all keys have been seen: hence two passes.  But with any guess g_i of it, one pass gives S_j = sum_i
// exp2(logit - g_i) for every key and z_i = 2^(lse_i - g_i) for every row; all terms are
// positive, so the true score of every key lies between S_j / max_i z_i and S_j / min_i z_i.  Keys
// further from the r-th largest S than that spread are in or out whatever their exact scores
// are; only the others, often none, are scored exactly and chosen among.  The selection is that of two passes, but for open
// keys whose exact scores differ by no more than rounding: the log-sum-exps behind them are sums over another
// reference, and may differ from those of two passes in the last bit.
// As guesses serve the log-sum-exps of the slot's step before (the same rows over most of the same heavy
// keys).  The scores themselves are not formed, so this is for steps whose scores nobody can see:
// the next step of the call overwrites all of them (the host has checked that nothing else of the
// slot touches them), or there is no place to put them.
// What bounds these loops is the chip's power: with 192 rows a launch runs at 1.72 GHz, at 1.92 GHz with the same
// cycles when its keys come from L2, at 2.13 GHz without key loads.  So what counts is work not done: one
// pass has half the matrix instructions, LDS operands and key bytes of two and two thirds of their
// vector instructions.  Loops of 256 problems, 128 channels, two passes at every step and this: 192 rows, 4096-token
// chunks of 131072 tokens, no key near the line 4790 -> 2920 us, keys spread evenly 4820 -> 3610 (open keys scored
// exactly; rows in several chunks, with which open keys start the step over, 360 rows, 2048-token chunks of 32768: 2565 ->
// 1670 and 2575); 256 rows, 2048-token chunks 1965 -> 1325 and 1985; 1024 problems of 32 rows, 512-token chunks 952 -> 900.
// Steps that do not pay (est_fixed) make both passes with code of their own (kOnceNote), which differs from the kernels without
// this by noting the guesses and how many keys are near the line: 0.6 to 1.4 us a step, 2 where both ways were one code.  A
// try that turns out of no use costs its pass beside the two, so tries are left out for longer with each that is (pause): log-sum-exps
// that move apart at every step, 192 rows, 8 steps 1184 us with two passes, 1257, 1604 with a try at every step.
enum : int { kOnceNote = 1, kOnceTry = 2 };
struct RowEstimates {
  float* lse = nullptr;      // LDS: one guess per row (`cap` of them) ...
  int cap = 0;
  int* words = nullptr;      // ... and kEstExtraWords words behind them: [0, 16) extremes per wave, [16] counter
  const void* q = nullptr;   // the rows they are for
  int rows = 0;
  float room = kEstRoom;     // how far from the r-th largest score keys are taken to stay open: as in the last step that tried, less with every one that does not
  bool dense = true;         // too many keys are that close (by the last step's scores): not worth trying
  bool hidden = false;       // this step's scores are not seen by anybody
  int pause = 0;             // steps worth trying that are still left at two passes after tries of no use ...
  int longest = 3;           // ... and how many were the last time: 7, 15, 31, ... as long as none is of use
  int way = 0;               // how this step selects (kWay...)
  const int* ask = nullptr;  // (no estimate: memory that a later step begins with)
};

// Copy rows idx[t0..t1) of [cache ; chunk] of K and V into k_out / v_out by NT threads
// (`tid` = index among them), t1 <= the rows kept.  `lidx` (LDS) or `gidx` (memory, written by this
// workgroup) holds the indices; with `identity` row t is simply candidate t.
template <int SEGS, int NT = kOwnThreads, int kUnroll = 8>
__device__ __forceinline__ void own_gather(const finch_problem& pb, int N, const int* lidx,
                                           const FINCH_GLOBAL int* gidx, bool identity, int tid, int t0,
                                           int t1, const KeptRows& kept = KeptRows{}) {
  const FINCH_GLOBAL u32x4* kc = as_global<u32x4>(kept.mapped ? kept.k0 : pb.k_cache);
  const FINCH_GLOBAL u32x4* kk = as_global<u32x4>(pb.k_chunk);
  const FINCH_GLOBAL u32x4* vc = as_global<u32x4>(kept.mapped ? kept.v0 : pb.v_cache);
  const FINCH_GLOBAL u32x4* vk = as_global<u32x4>(pb.v_chunk);
  FINCH_GLOBAL u32x4* ko = as_global_mut<u32x4>(pb.k_out);
  FINCH_GLOBAL u32x4* vo = as_global_mut<u32x4>(pb.v_out);
  constexpr int kRowsPerIter = NT / SEGS;
  const int seg = tid % SEGS, sub = tid / SEGS;
  for (int row0 = t0; row0 < t1; row0 += kRowsPerIter * kUnroll) {
    u32x4 kv[kUnroll], vv[kUnroll];
#pragma unroll
    for (int it = 0; it < kUnroll; ++it) {
      const int t = min(row0 + it * kRowsPerIter + sub, t1 - 1);
      int j = identity ? t : (lidx ? lidx[t] : gidx[t]);
      j = min(max(j, 0), N - 1);
      const bool cached = j < pb.c;
      if (kept.mapped) {
        long long ko_at = static_cast<long long>(j - pb.c) * SEGS, vo_at = ko_at;
        if (cached) {
          ko_at = kept.at[j];
          vo_at = kept.at[kept.cap + j];
        }
        kv[it] = (cached ? kc : kk)[ko_at + seg];
        vv[it] = (cached ? vc : vk)[vo_at + seg];
        continue;
      }
      const size_t off = static_cast<size_t>(cached ? j : j - pb.c) * SEGS + seg;
      kv[it] = (cached ? kc : kk)[off];
      vv[it] = (cached ? vc : vk)[off];
    }
#pragma unroll
    for (int it = 0; it < kUnroll; ++it) {
      const int t = row0 + it * kRowsPerIter + sub;
      if (t < t1) {
        ko[static_cast<size_t>(t) * SEGS + seg] = kv[it];
        vo[static_cast<size_t>(t) * SEGS + seg] = vv[it];
      }
    }
  }
}

// The same with the kept keys re-positioned: slot p takes kept row t = p (the ascending
// order), or, with `ranked` (LDS; see own_rank_kept), the kept row whose record stands
// at place p of the sorted records; the key is turned by p - idx[t] positions while it
// is copied (not at all with pairing FINCH_ROPE_OFF).  A thread owns two pieces of a
// row, d/2 channels apart, i.e. both partners of its channel pairs.  (Values may stay where
// they are; keys do not.)
template <int SEGS, int NT = kOwnThreads, int E = 8, int kUnroll = 4>
__device__ __forceinline__ void own_gather_rot(const finch_problem& pb, int N, int r, const int* lidx,
                                               const FINCH_GLOBAL int* gidx, bool identity, int pairing,
                                               double log2_base, int tid, const unsigned long long* ranked,
                                               int t0, int t1, const KeptRows& kept = KeptRows{}) {
  constexpr int kHalf = SEGS / 2;
  const FINCH_GLOBAL u32x4* kc = as_global<u32x4>(pb.k_cache);
  const FINCH_GLOBAL u32x4* kk = as_global<u32x4>(pb.k_chunk);
  const FINCH_GLOBAL u32x4* vc = as_global<u32x4>(kept.mapped ? kept.v0 : pb.v_cache);
  const FINCH_GLOBAL u32x4* vk = as_global<u32x4>(pb.v_chunk);
  FINCH_GLOBAL u32x4* ko = as_global_mut<u32x4>(pb.k_out);
  FINCH_GLOBAL u32x4* vo = as_global_mut<u32x4>(pb.v_out);
  constexpr int kRowsPerIter = NT / kHalf;
  const int seg = tid % kHalf, sub = tid / kHalf;
  double th[E];
  pair_thetas<E, kHalf>(pairing, seg, log2_base, th);
  for (int row0 = t0; row0 < t1; row0 += kRowsPerIter * kUnroll) {
    u32x4 ka[kUnroll], kb[kUnroll], va[kUnroll], vb[kUnroll];
    int shift[kUnroll], slot[kUnroll];
#pragma unroll
    for (int it = 0; it < kUnroll; ++it) {
      const int p = min(row0 + it * kRowsPerIter + sub, t1 - 1);
      const int t = ranked ? min(static_cast<int>(~static_cast<unsigned>(ranked[p])), r - 1) : p;
      int j = identity ? t : (lidx ? lidx[t] : gidx[t]);
      j = min(max(j, 0), N - 1);
      slot[it] = p;
      shift[it] = p - j;
      const bool cached = j < pb.c;
      const size_t off = static_cast<size_t>(cached ? j : j - pb.c) * SEGS + seg;
      ka[it] = (cached ? kc : kk)[off];
      kb[it] = (cached ? kc : kk)[off + kHalf];
      if (!kept.stay) {
        long long voff = static_cast<long long>(off);
        if (kept.mapped && cached) voff = static_cast<long long>(kept.at[kept.cap + j]) + seg;
        va[it] = (cached ? vc : vk)[voff];
        vb[it] = (cached ? vc : vk)[voff + kHalf];
      }
    }
#pragma unroll
    for (int it = 0; it < kUnroll; ++it) {
      if (row0 + it * kRowsPerIter + sub < t1) {
        if (pairing != FINCH_ROPE_OFF && shift[it] != 0) rotate_pieces<E>(pairing, th, shift[it], ka[it], kb[it]);
        const size_t o = static_cast<size_t>(slot[it]) * SEGS + seg;
        ko[o] = ka[it];
        ko[o + kHalf] = kb[it];
        if (!kept.stay) {
          vo[o] = va[it];
          vo[o + kHalf] = vb[it];
        }
      }
    }
  }
}

// Notes where the r rows that this step keeps lie (KeptRows::stay).  In place: kept row t is candidate
// idx[t] >= t, so that a turn of NT rows only reads places that no turn before it has written.
// Whole workgroup; the notes are complete at the next barrier.
template <int SEGS>
__device__ __forceinline__ void own_note_rows(const finch_problem& pb, int r, const int* lidx, const FINCH_GLOBAL int* gidx,
                                              bool identity, int tid, const KeptRows& kept) {
  auto pieces = [](const void* p, const char* base) { return static_cast<int>((static_cast<const char*>(p) - base) / 16); };
  const int kc = pieces(pb.k_cache, kept.k0), vc = pieces(pb.v_cache, kept.v0);
  const int kk = pieces(pb.k_chunk, kept.k0), vk = pieces(pb.v_chunk, kept.v0);
  for (int t0 = 0; t0 < r; t0 += kOwnThreads) {
    const int t = t0 + tid, u = min(t, r - 1);
    const int j = identity ? u : (lidx ? lidx[u] : gidx[u]);
    const bool cached = j < pb.c;
    const int off = (cached ? j : j - pb.c) * SEGS;
    int k_at = (cached ? kc : kk) + off, v_at = (cached ? vc : vk) + off;
    if (kept.mapped && cached) {
      k_at = kept.at[j];
      v_at = kept.at[kept.cap + j];
    }
    __syncthreads();
    if (t < r) {
      kept.at[t] = k_at;
      kept.at[kept.cap + t] = v_at;
    }
  }
}

}  // namespace

// Kept rows by relevance: one 64-bit record per kept row t < r - order key of its score
// in the upper half, ~t in the lower - sorted in descending order by a bitonic network
// over npad = max(64, next power of two) records (padding records are zero and end up
// last), so that place p holds the row with the p-th highest score, equal scores in index
// order.  `ranked` needs 8 * npad bytes of LDS.  Whole workgroup; ends with a barrier.
// A wave owns a part of max(64, npad / 8) consecutive records and keeps them in registers,
// record lane + 64 s of the part in slot s of the lane: partners less than 64 apart are
// exchanged by lane shuffles, partners 64 or 128 apart sit in the same lane, and only the
// stages whose partners lie in different parts go through LDS and workgroup barriers.
constexpr int kRankSlots = 4;  // records per lane: parts of at most 256 records = 2048 kept rows
__device__ __forceinline__ int own_rank_pad(int r) {
  int npad = 64;
  while (npad < r) npad <<= 1;
  return npad;
}
__device__ __forceinline__ void own_rank_kept(unsigned long long* ranked, int r, const FINCH_GLOBAL float* scores,
                                              const int* lidx, bool identity, int tid) {
  const int npad = own_rank_pad(r);
  const int lane = tid & 63, wave = tid >> 6;
  const int part = max(64, npad / kOwnWaves);
  const int slots = part >> 6;  // 1, 2 or 4
  const bool active = wave * part < npad;
  const int e0 = wave * part + lane;  // slot s holds record e0 + 64 s
  unsigned long long rec[kRankSlots];
#pragma unroll
  for (int sl = 0; sl < kRankSlots; ++sl) {
    rec[sl] = 0ull;
    const int u = e0 + 64 * sl;
    if (active && sl < slots && u < r)
      rec[sl] = (static_cast<unsigned long long>(order_key(scores[identity ? u : lidx[u]])) << 32) | static_cast<unsigned>(~u);
  }
  // the record that stays at position e after the exchange with position e ^ j in the stage (k, j)
  auto keep = [](unsigned long long mine, unsigned long long other, int e, int j, int k) {
    const bool want_max = ((e & k) == 0) == ((e & j) == 0);
    return want_max ? (mine > other ? mine : other) : (mine < other ? mine : other);
  };
  bool in_lds = false;  // the current order is in `ranked`, not in the registers
  for (int k = 2; k <= npad; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j >= part) {
        if (!in_lds) {
#pragma unroll
          for (int sl = 0; sl < kRankSlots; ++sl)
            if (active && sl < slots) ranked[e0 + 64 * sl] = rec[sl];
        }
        __syncthreads();
        for (int q = tid; q < (npad >> 1); q += kOwnThreads) {
          const int i = ((q & ~(j - 1)) << 1) | (q & (j - 1));
          const unsigned long long a = ranked[i], b = ranked[i + j];
          if (((i & k) == 0) ? a < b : a > b) {
            ranked[i] = b;
            ranked[i + j] = a;
          }
        }
        in_lds = true;
        continue;
      }
      if (in_lds) {
        __syncthreads();
#pragma unroll
        for (int sl = 0; sl < kRankSlots; ++sl)
          if (active && sl < slots) rec[sl] = ranked[e0 + 64 * sl];
        in_lds = false;
      }
      if (j >= 64) {
        // partner in the same lane, j / 64 slots away (1 or 2)
        unsigned long long nxt[kRankSlots];
#pragma unroll
        for (int sl = 0; sl < kRankSlots; ++sl) {
          const unsigned long long other = (j == 64) ? rec[sl ^ 1] : rec[sl ^ 2];
          nxt[sl] = keep(rec[sl], other, e0 + 64 * sl, j, k);
        }
#pragma unroll
        for (int sl = 0; sl < kRankSlots; ++sl)
          if (sl < slots) rec[sl] = nxt[sl];
      } else {
#pragma unroll
        for (int sl = 0; sl < kRankSlots; ++sl) {
          const unsigned long long other = __shfl_xor(rec[sl], j);
          rec[sl] = keep(rec[sl], other, e0 + 64 * sl, j, k);
        }
      }
    }
  }
  if (in_lds) {
    __syncthreads();
  } else {
    // (nobody reads `ranked` before the barrier below, and the last stage that wrote it
    // was followed by a barrier and a reload)
#pragma unroll
    for (int sl = 0; sl < kRankSlots; ++sl)
      if (active && sl < slots) ranked[e0 + 64 * sl] = rec[sl];
    __syncthreads();
  }
}

// Where the candidates' order keys go in the LDS scratch `sel` of sel_bytes: behind the
// selection's own words and the kept indices, and behind the first `busy` bytes (what is still
// in use while scores are being written).  Null if there is no room.
__device__ __forceinline__ unsigned* own_sel_keys(char* sel, size_t sel_bytes, size_t busy, int N, int r) {
  const size_t mine = sizeof(SelLds) + (static_cast<size_t>(r) + kSelIdxPad) * 4;
  const size_t off = ((mine > busy ? mine : busy) + 15) & ~size_t{15};
  if (N > kOwnThreads * kSelRegKeys || off + static_cast<size_t>(N) * 4 > sel_bytes) return nullptr;
  return reinterpret_cast<unsigned*>(sel + off);
}

// Scores of a step without any row (document rows only, and no chunk): empty sums.  Whole
// workgroup; a barrier at the end.
__device__ __forceinline__ void own_no_rows(float* scores, unsigned* lkeys, int N, int tid) {
  for (int i = tid; i < N; i += kOwnThreads) {
    __hip_atomic_store((FINCH_GLOBAL float*)scores + i, 0.f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lkeys) lkeys[i] = order_key(0.f);
  }
  __syncthreads();
}

// What a step keeps: its rows' indices in LDS (null: only in pb.idx), all rows in their order
// (identity), nothing (a wait has expired, or r is 0).
struct Selected {
  int* lidx;
  bool identity, ok;
};

// Top-r (Method: t = top-r(A_agg, r); with `layered` on the sum over the
// layer's heads) once this workgroup's scores are in memory (and a barrier has been passed since).
// `sel` is LDS scratch of sel_bytes (owner_lds_bytes); `dst` the
// scores of this problem; `lkeys` what own_sel_keys said, with the order keys of these scores
// in it already (not those of the layer's sum).  The indices are in LDS at the end (a barrier has been
// passed), and in memory already if they were not chosen by `lkeys`.
__device__ __forceinline__ Selected own_select(const LaunchParams& prm, const finch_problem& pb, int slot, int N,
                                               FINCH_GLOBAL float* dst, char* sel, size_t sel_bytes,
                                               unsigned* lkeys, const finch_problem* step_probs, int epoch,
                                               bool layered, int* sync_words, int tid, SelBand* band = nullptr) {
  const int lane = tid & 63, wave = tid >> 6;
  const int L = prm.layer_group;
  const int r = min(pb.r, N);
  if (r <= 0) return {nullptr, false, false};
  FINCH_GLOBAL int* gidx = as_global_mut<int>(pb.idx);
  const bool identity = r >= N;
  SelLds* fl = reinterpret_cast<SelLds*>(sel);
  int* lidx = nullptr;
  if (!identity) {
    if (sizeof(SelLds) + (static_cast<size_t>(r) + kSelIdxPad) * 4 <= sel_bytes)
      lidx = reinterpret_cast<int*>(sel + sizeof(SelLds));
    if (layered) {
      // this workgroup's scores are out (stored past the caches, and every thread has waited
      // for its own stores at the barrier after pass 2); wait until all L workgroups of the
      // run say the same
      const int run = slot / L;
      if (tid == 0) {
        __hip_atomic_fetch_add(sync_words, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const long long t0 = wall_clock64();
        int gave_up = 0;
        while (__hip_atomic_load(sync_words, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < L * (epoch + 1)) {
          __builtin_amdgcn_s_sleep(8);
          if (wall_clock64() - t0 > prm.spin_ticks) {
            atomicOr(prm.layer_err, 1);
            gave_up = 1;
            break;
          }
        }
        fl->layer_gave_up = gave_up;
      }
      if (tid < L) {
        const finch_problem pg = step_probs[run * L + tid];
        fl->layer_src[tid] = pg.scores ? pg.scores
                                       : prm.ws_scores + static_cast<size_t>(run * L + tid) * prm.score_stride;
      }
      __syncthreads();
      if (fl->layer_gave_up) {
        // Scores that other workgroups are still writing must not be selected on (a
        // selection that reads them twice could count differently each time): this
        // workgroup leaves the step's indices and cache rows unwritten.  It still says
        // that it will not read the others' scores any more.
        if (tid == 0) __hip_atomic_fetch_add(sync_words + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return {nullptr, false, false};
      }
    }
    const LayerScores<kSelMaxLayer> layer_sum = {fl->layer_src, L};
    const OneScoreVector own = {dst};
    if (lkeys) {  // (then there is room for the indices as well)
      if (layered) {
        sel_stage_layer_keys<kOwnThreads>(fl->layer_src, L, N, lkeys, tid);
        __syncthreads();
      }
      select_keys_any<kOwnThreads, true>(lkeys, N, r, gidx, lidx, fl, tid, lane, wave, band);
    } else {
      __syncthreads();
      if (layered) select_generic<kOwnThreads>(layer_sum, N, r, gidx, lidx, fl, tid, lane, wave);
      else select_generic<kOwnThreads>(own, N, r, gidx, lidx, fl, tid, lane, wave);
    }
    __syncthreads();  // idx complete
    // (the other workgroups' scores have been read for the last time)
    if (layered && tid == 0) __hip_atomic_fetch_add(sync_words + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return {lidx, identity, true};
}

// The rest of a step once it is known what it keeps: the indices, and compaction (Method: Managing the
// Cache) of rows of SEGS 16-byte pieces with E elements each.
template <int SEGS, int E, bool ROT>
__device__ __forceinline__ void own_compact(const LaunchParams& prm, const finch_problem& pb, int N, const Selected& chosen,
                                            FINCH_GLOBAL float* dst, char* sel, bool in_lds, int tid, KeptRows& kept) {
  const int r = min(pb.r, N);
  KeptRows mine = kept;
  kept.mapped = false;  // (of the next step's cache; a step that gives up leaves none)
  if (!chosen.ok) return;
  FINCH_PHASE_BEGIN();
  FINCH_GLOBAL int* gidx = as_global_mut<int>(pb.idx);
  const bool identity = chosen.identity;
  int* const lidx = chosen.lidx;
  if (identity) {
    for (int i = tid; i < N; i += kOwnThreads) gidx[i] = i;
  } else if (in_lds) {
    for (int t = tid; t < r; t += kOwnThreads) gidx[t] = lidx[t];
  }
  if (ROT) {
    // slots by relevance (Method: Managing the Cache, the worked example): the rank of a kept
    // row's score among the kept ones, highest first, equal scores by index.  The host
    // sends such batches here only if the indices and the records of all kept rows fit
    // behind the selection scratch.
    unsigned long long* ranked = nullptr;
    if (prm.rank_order) {
      __syncthreads();  // (the identity case has not been through a barrier since the scores)
      ranked = reinterpret_cast<unsigned long long*>(sel + sizeof(SelLds) + ((static_cast<size_t>(r) * 4 + 7) & ~size_t{7}));
      own_rank_kept(ranked, r, dst, lidx, identity, tid);
    }
    own_gather_rot<SEGS, kOwnThreads, E>(pb, N, r, lidx, gidx, identity, prm.rope_pairing, prm.rope_log2_base, tid, ranked, 0, r,
                                         mine);
  } else if (!mine.stay) {
    own_gather<SEGS>(pb, N, lidx, gidx, identity, tid, 0, r, mine);
  }
  if (mine.stay) {
    own_note_rows<SEGS>(pb, r, lidx, gidx, identity, tid, mine);
    kept.mapped = true;
  }
  FINCH_PHASE(7);
}

// Both.
template <int SEGS, int E, bool ROT>
__device__ __forceinline__ void own_finish_step(const LaunchParams& prm, const finch_problem& pb, int slot, int N,
                                                FINCH_GLOBAL float* dst, char* sel, size_t sel_bytes,
                                                unsigned* lkeys, const finch_problem* step_probs, int epoch,
                                                bool layered, int* sync_words, int tid, KeptRows& kept) {
  FINCH_PHASE_BEGIN();
  const Selected chosen = own_select(prm, pb, slot, N, dst, sel, sel_bytes, lkeys, step_probs, epoch, layered, sync_words, tid);
  FINCH_PHASE(6);
  own_compact<SEGS, E, ROT>(prm, pb, N, chosen, dst, sel, lkeys != nullptr, tid, kept);
}

// Few rows of 64 channels: 128 registers are enough for a step, and two workgroups share a compute unit.
constexpr bool own_lean(int d, int qbt, bool rot, bool doc) { return d == 64 && qbt == 2 && !rot && !doc; }

// Calls f(number of row blocks) with the number as a constant if it is one of those a kernel for up
// to QBT has the code without branches for; what f says, or false.
template <int QBT, typename F>
__device__ __forceinline__ bool own_whole(int qb, F f) {
  if (qb == QBT) return f(std::integral_constant<int, QBT>{});
  if (qb == QBT - 1) return f(std::integral_constant<int, QBT - 1>{});
  return false;
}

// The same for every number of row blocks up to QBT.
template <int QBT, typename F>
__device__ __forceinline__ bool own_any(int qb, F f) {
  if (qb == QBT) return f(std::integral_constant<int, QBT>{});
  if constexpr (QBT > 1) return own_any<QBT - 1>(qb, f);
  else return false;
}

// One step of one problem by the whole workgroup.  QBT = row blocks (of 32 prompt
// rows) per pass over the keys the code is compiled for; prm.row_chunk <= 32 * QBT.
// stages: 0 = scores only, 1 = scores, top-r and compaction.  `staged_q` names the
// prompt block whose rows are in LDS from the previous step of the same launch (or
// nullptr); inputs do not change during a launch, so the same pointer and row
// count mean the same rows and the copy is skipped.  Ends with every thread past
// its last access to LDS only after the next barrier: callers that go on to
// another step must put a barrier in between.
// With prm.layer_group = L > 1 the L workgroups of a run of slots (a layer's KV heads)
// select together (Method: "Sum over heads", then one top-r per layer): each publishes
// its scores, waits for the others (bounded: a wait that runs out sets the error word and
// the workgroup leaves the step's indices and rows unwritten), adds the L vectors up in the same order
// and selects on the sum, so that all L arrive at the same indices on their own.
// `step_probs` are the descriptors of this step, `epoch` counts the exchanges this
// workgroup has been through in this launch; returns true if the step made one.
// ONCE (RowEstimates): kOnceTry selects on one pass, if that is worth trying; true if the step is done, else it
// is to be made with kOnceNote, which makes both passes and leaves what the next try needs.
template <int D, int QBT, bool ROT, bool DOC, bool LOOP, int ONCE>
__device__ __forceinline__ bool own_step_body(const LaunchParams& prm, const finch_problem& pb, int slot,
                                              int stages, char* smem, const void*& staged_q,
                                              int& staged_rows, const finch_problem* step_probs,
                                              int epoch, KeptRows& kept, RowEstimates& est) {
  const int N = pb.c + pb.m;
  if (N == 0) {
    kept.mapped = false;
    return ONCE == kOnceTry;
  }
  FINCH_PHASE_BEGIN();
  const int Rp = (DOC && !pb.q) ? 0 : prm.group * pb.n_que;  // prompt rows
  const int tid = own_thread();
  // (DOC kernels: in a scalar register, so that the loops over a wave's key blocks are uniform.  A key buffer
  // there lives on past both exits of such a loop; with a loop that lanes may leave at different times the
  // compiler keeps what either exit hands on in registers of its own, 32 more than there are: up to
  // 56 spilled, 789 us in place of 604 for the loop of 256 problems, 200-token chunks, with
  // re-positioning, 808 and 743 for a step of 256 problems of 512 + 1024 candidates.)
  const int wave = DOC || ONCE ? uni(tid >> 6) : tid >> 6;
  constexpr int kStride = D * 2 + 16;
  const int RC = prm.row_chunk;
  char* lds_q = smem;
  float2* wstats = reinterpret_cast<float2*>(smem + RC * kStride);                 // [waves][RC]
  float* lds_lse = reinterpret_cast<float*>(smem + RC * (kStride + kOwnWaves * 8));  // [RC]
  int* sh_next = reinterpret_cast<int*>(smem + RC * (kStride + kOwnWaves * 8 + 4));
  // (keys that are re-positioned lie in the cache)
  const bool mapped = !ROT && kept.mapped;
  const KeySource ks = {mapped ? kept.k0 : static_cast<const char*>(pb.k_cache), static_cast<const char*>(pb.k_chunk), pb.c,
                        mapped, kept.at};
  const int nb = (N + 31) >> 5;
  const float sc = prm.scale_log2;
  float* gscores = pb.scores ? pb.scores : prm.ws_scores + static_cast<size_t>(slot) * prm.score_stride;
  FINCH_GLOBAL float* dst = as_global_mut<float>(gscores);
  const int L = prm.layer_group;
  const bool layered = stages && L > 1 && pb.r > 0 && pb.r < N;  // the same in every workgroup of the run
  // selection scratch lies behind the staged prompt rows, over the statistics of pass 1; the
  // scores' order keys go there from pass 2 (past what pass 2 still reads)
  char* const sel = smem + RC * kStride;
  const size_t sel_bytes = prm.lds_bytes - static_cast<size_t>(RC) * kStride;
  unsigned* const lkeys = (stages && pb.r > 0 && pb.r < N)
                              ? own_sel_keys(sel, sel_bytes, static_cast<size_t>(RC) * (kOwnWaves * 8 + 4) + 16, N, pb.r)
                              : nullptr;
  int* const sync_words = (stages && L > 1) ? prm.layer_sync + 2 * (slot / L) : nullptr;
  if (sync_words && epoch > 0) {
    // nobody of the run may still be adding up the scores of the step before when this
    // step's scores start to overwrite them
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

  // (two workgroups a compute unit have no registers for it)
  constexpr bool WHOLE = !own_lean(D, QBT, ROT, DOC) || LOOP;
  auto whole = [](int qb, auto f) { return own_whole<QBT>(qb, f); };

  // Row chunks: the prompt rows first (they see every key, so they initialise all
  // scores), then, in DOC kernels, the rows of the chunk's own tokens, head by head
  // and from the last tokens to the first (the last ones see every key as well).
  const int n_pchunks = (Rp + RC - 1) / RC;
  const int dper = (DOC && pb.q_doc && pb.m > 0) ? (pb.m + RC - 1) / RC : 0;
  const int n_chunks = n_pchunks + prm.group * dper;
  // With several chunks the sums so far stay in LDS, as the order keys that the selection wants there, and go
  // to memory at the end: a wave that asked memory for a sum would wait for its next key block, which is on the
  // way before, as well.  (The loop of 256 problems, 192 rows and 1024-token chunks with document rows: 2295 us, 2225
  // with the sums in LDS.)
  const bool lkeys_sum = lkeys && !layered && n_chunks > 1;
  struct RowChunk {
    const void* qsrc;
    int R, row0, lim0, lim_step;
  };
  // rows [row0, row0 + RC) of `qsrc` (R rows in all); row i of the chunk sees the
  // keys below lim0 + lim_step * i
  auto row_chunk = [&](int ch) -> RowChunk {
    if (!DOC || ch < n_pchunks) return {pb.q, Rp, ch * RC, N, 0};
    const int dc = ch - n_pchunks;
    const int g = dc / dper;
    const int row0 = (dper - 1 - (dc - g * dper)) * RC;
    return {static_cast<const char*>(pb.q_doc) + static_cast<size_t>(g) * pb.m * (D * 2), pb.m, row0, pb.c + row0 + 1, 1};
  };
  // Key blocks a wave works on and the ones under way.  In DOC kernels, whose passes are a few key
  // blocks long, a buffer is never left idle: beside the last key block of pass 1 the first of
  // pass 2 is under way, beside the last of pass 2 this thread's pieces of the next chunk's
  // rows (a thread's share of 256 rows is exactly as large as its share of a key block).
  // 256 problems of 192 rows, 1024-token chunks, 17 chunks of rows a step: the loop takes 2216 us,
  // 2346 where every chunk asks for its rows when its turn has come (64 channels, 256 rows: 1569 and 1669).
  bf16x8 ka[D / 16], kb[D / 16];
  static_assert(!ONCE || (LOOP && !DOC));
  if (ONCE == kOnceTry) {
    if (!est.hidden || est.q != pb.q || est.rows != Rp || Rp > est.cap || !lkeys || est.dense) return false;
    if (est.pause > 0) {
      --est.pause;
      return false;
    }
    est.way = kWayOnce;
  }
  auto no_use = [&](int why) {
    est.way |= why;
    est.pause = est.longest = 2 * est.longest + 1;
  };
  unsigned most = 0u, least = 0u;  // largest order key of any row's log2 z, and the smallest one's complement
  Selected chosen = {nullptr, false, false};
  int asked;  // (asked for beside the first key block)
  for (int ch = 0; ch < n_chunks; ++ch) {
    const int tid = own_thread(), lane = tid & 63, t = lane & 31, h = lane >> 5;
    const RowChunk rc = row_chunk(ch);
    const void* const qsrc = rc.qsrc;
    const int R = rc.R, row0 = rc.row0, lim0 = rc.lim0, lim_step = rc.lim_step;
    const int rows = min(RC, round_up32(R - row0));
    const int QB = rows >> 5;
    const bool first_chunk = ch == 0;
    // key blocks any row of the chunk sees
    const int nbc = DOC ? (min(N, lim0 + lim_step * (min(row0 + rows, R) - 1 - row0)) + 31) >> 5 : nb;
    // smallest and largest limit of row block q, and this lane's own in it
    auto lim_lo = [&](int q) { return lim0 + lim_step * (q * 32); };
    auto lim_hi = [&](int q) { return lim0 + lim_step * (q * 32 + 31); };
    auto lim_mine = [&](int q) { return min(N, lim0 + lim_step * (q * 32 + t)); };
    int b = wave;
    if (DOC && ch > 0) {
      // (requested, like the rows in kb, at the end of the chunk before)
      stage_q_held<D, kOwnThreads>(kb, R, row0, rows, lds_q, tid);
      __syncthreads();
    } else {
      load_k_block<D>(ks, N, b << 5, lane, ka);  // requested before Q is staged
      if (LOOP && ch == 0) asked = *as_global<int>(est.ask);
      if (!(R <= RC && staged_q == qsrc && staged_rows == R)) {
        stage_q<D, kOwnThreads>(qsrc, R, row0, rows, lds_q, tid);
        __syncthreads();
      }
    }
    staged_q = nullptr;
    FINCH_PHASE(0);

    // ---- the only pass (RowEstimates): row sums and key sums of exp2(logit - guess), fixed block assignment
    float spread = 0.f;  // log2 of max_i z_i / min_i z_i
    if (ONCE == kOnceTry) {
      const int tid = own_thread(), lane = tid & 63, t = lane & 31, h = lane >> 5;
      float z_run[QBT], g[QBT];
#pragma unroll
      for (int q = 0; q < QBT; ++q) {
        z_run[q] = 0.f;
        g[q] = q < QB ? est.lse[row0 + q * 32 + t] : kInf;
      }
      auto put = [&](float tot, int kbase) {
        const int key = kbase + acc_key(t >> 1, h);
        if ((t & 1) == 0 && key < N) lkeys[key] = order_key(first_chunk ? tot : order_value(lkeys[key]) + tot);
      };
      auto process = [&](const bf16x8(&kf)[D / 16], int blk) {
        const int kbase = blk << 5;
        float u[16];
        auto whole_block = [&](auto qb) {
          constexpr int QBC = decltype(qb)::value;
          float z[QBC];
          for_block_logits<D, QBC>(kf, lds_q, lane, [&](int q, int v, float a) {
            const float e = fast_exp2(__builtin_fmaf(a, sc, -g[q]));
            z[q] = v == 0 ? e : z[q] + e;
            u[v] = q == 0 ? e : u[v] + e;
          });
#pragma unroll
          for (int q = 0; q < QBC; ++q) z_run[q] += z[q];
          return true;
        };
        if (kbase + 32 > N) {
#pragma unroll
          for (int v = 0; v < 16; ++v) u[v] = 0.f;
#pragma unroll
          for (int q = 0; q < QBT; ++q) {
            if (q < QB) {
              bf16x8 qf[D / 16];
              load_q_frags<D>(lds_q, q, lane, qf);
              const f32x16 a = mfma_block<D>(kf, qf);
              float z = 0.f;
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                const float e = kbase + acc_key(v, h) < N ? fast_exp2(__builtin_fmaf(a[v], sc, -g[q])) : 0.f;
                z += e;
                u[v] += e;
              }
              z_run[q] += z;
            }
          }
        } else {
          own_any<QBT>(QB, whole_block);
        }
        put(fold16_over32(u, t), kbase);
      };
      if (b < nb) {
        while (true) {
          load_k_block<D>(ks, N, (b + kOwnWaves) << 5, lane, kb);
          process(ka, b);
          b += kOwnWaves;
          if (b >= nb) break;
          load_k_block<D>(ks, N, (b + kOwnWaves) << 5, lane, ka);
          process(kb, b);
          b += kOwnWaves;
          if (b >= nb) break;
        }
        // (neither buffer is of use to what follows)
        forget<D>(ka);
        forget<D>(kb);
      }
      float* const wsum = reinterpret_cast<float*>(wstats);  // [waves][RC]
#pragma unroll
      for (int q = 0; q < QBT; ++q) {
        if (q < QB) {
          const float z = z_run[q] + __shfl_xor(z_run[q], 32);
          if (h == 0) wsum[wave * RC + q * 32 + t] = z;
        }
      }
      FINCH_PHASE(1);
      if (tid == 0) est.words[16] = 0;
      __syncthreads();
      FINCH_PHASE(2);
      // every row's log-sum-exp takes the place of its guess
      if (tid < rows) {
        float l = kInf;
        if (row0 + tid < R) {
          float z = wsum[tid];
#pragma unroll
          for (int w = 1; w < kOwnWaves; ++w) z += wsum[w * RC + tid];
          const float guess = est.lse[row0 + tid], moved = fast_log2(z);
          l = guess + moved;
          if (pb.lse_extra) l = widen_lse(l, as_global<float>(pb.lse_extra)[row0 + tid]);
          const unsigned key = order_key(fabsf(moved) <= kEstReach ? l - guess : kInf);
          most = max(most, key);
          least = max(least, ~key);
        }
        est.lse[row0 + tid] = l;
      }
      most = wave_max_u32(most);
      least = wave_max_u32(least);
      if (lane == 0) {
        est.words[2 * wave] = static_cast<int>(most);
        est.words[2 * wave + 1] = static_cast<int>(least);
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kOwnWaves; ++w) {
        most = max(most, static_cast<unsigned>(est.words[2 * w]));
        least = max(least, static_cast<unsigned>(est.words[2 * w + 1]));
      }
      spread = uni(order_value(most) - order_value(~least));
      FINCH_PHASE(3);
      // (rows that are not numbers, or one whose sum is out of range: the spread is infinite or not a number)
      if (!(spread <= kEstSpread)) {
        no_use(kWayRange);
        staged_q = (n_chunks == 1) ? pb.q : nullptr;
        return false;
      }
    }

    if constexpr (ONCE != kOnceTry) {
    // ---- pass 1: running (reference, sum exp2) per prompt row, fixed block assignment
    {
      float m_run[QBT], z_run[QBT];
#pragma unroll
      for (int q = 0; q < QBT; ++q) {
        m_run[q] = -kInf;
        z_run[q] = 0.f;
      }
      // The reference of a row only has to keep exp2 in range: it is taken from the
      // wave's first key block and moved (sum rescaled) only when a block's sum shows
      // that its logits lie far above it.
      // (bit q: row block q has been through at least one visible key block)
      unsigned seeded = 0;
      // statistics of one 32 x 32 logit block
      auto tile_stats = [&](f32x16 a, int q, int kbase) {
        if (kbase + 32 > (DOC ? min(N, lim_lo(q)) : N)) {  // keys this row does not see, or past the end
          const int lim = DOC ? lim_mine(q) : N;
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (kbase + acc_key(v, h) >= lim) a[v] = -kInf;
        }
        float z = 0.f;
        const bool was_seeded = (seeded >> q) & 1u;
        bool move = !was_seeded;
        if (was_seeded) {
          const float mu = (m_run[q] == -kInf) ? 0.f : m_run[q];
#pragma unroll
          for (int v = 0; v < 16; ++v) z += fast_exp2(__builtin_fmaf(a[v], sc, -mu));
          // (A lane without a reference - every key it has seen was masked - never meets a
          // key it sees later on: masked keys are the ones past a limit, a wave's blocks come
          // in ascending key order, and inside a block a lane's keys ascend too.)
          move = __any(!(z <= 0x1p64f));
        }
        if (move) {
          float bm = fmaxf(a[0], a[1]);
#pragma unroll
          for (int v = 2; v < 16; v += 2) bm = fmaxf(fmaxf(bm, a[v]), a[v + 1]);
          const float mn = fmaxf(m_run[q], bm * sc);
          z_run[q] = (mn == -kInf) ? 0.f : z_run[q] * fast_exp2(m_run[q] - mn);
          m_run[q] = mn;
          const float mu = (mn == -kInf) ? 0.f : mn;
          z = 0.f;
#pragma unroll
          for (int v = 0; v < 16; ++v) z += fast_exp2(__builtin_fmaf(a[v], sc, -mu));
        }
        z_run[q] += z;
        seeded |= 1u << q;
      };
      // Row blocks go through in pairs, one pair behind: while the matrix pipe works
      // on the logits of pair i, the vector units take the exponentials of pair i - 1.
      // In DOC kernels a pair none of whose rows sees the key block is left out (the
      // limits grow with the row, and a wave's key blocks come in ascending order, so a
      // row block that is left out once stays out).
      // A block every row sees all of, once there are references (false: some logits lie too far
      // above them; nothing has been added).
      auto whole_block = [&](const bf16x8(&kf)[D / 16], auto qb) {
        constexpr int QBC = decltype(qb)::value;
        float z[QBC];
#pragma unroll
        for (int q = 0; q < QBC; ++q) z[q] = 0.f;
        for_block_logits<D, QBC>(kf, lds_q, lane, [&](int q, int, float a) { z[q] += fast_exp2(__builtin_fmaf(a, sc, -m_run[q])); });
        bool far = false;
#pragma unroll
        for (int q = 0; q < QBC; ++q) far |= !(z[q] <= 0x1p64f);
        if (__any(far)) return false;
#pragma unroll
        for (int q = 0; q < QBC; ++q) z_run[q] += z[q];
        return true;
      };
      auto process = [&](const bf16x8(&kf)[D / 16], int blk) {
        const int kbase = blk << 5;
        if (WHOLE && seeded && kbase + 32 <= min(N, lim0) && whole(QB, [&](auto qb) { return whole_block(kf, qb); })) return;
        auto pair_visible = [&](int q) { return !DOC || kbase < lim_hi(q + 1 < QB ? q + 1 : q); };
        f32x16 acc[QBT];
#pragma unroll
        for (int q = 0; q < QBT + 2; q += 2) {
          if (q < QBT && q < QB && pair_visible(q)) {
            if (q + 1 < QB) {
              mfma_block_pair_lds<D>(kf, lds_q, q, lane, acc[q], acc[q + 1]);
            } else {
              bf16x8 qf0[D / 16];
              load_q_frags<D>(lds_q, q, lane, qf0);
              acc[q] = mfma_block<D>(kf, qf0);
            }
          }
          if (q >= 2 && q - 2 < QB && pair_visible(q - 2)) {
            tile_stats(acc[q - 2], q - 2, kbase);
            if (q - 1 < QB) tile_stats(acc[q - 1], q - 1, kbase);
          }
        }
      };
      if (b < nbc) {
        auto next_block = [&] { return !DOC || b + kOwnWaves < nbc ? b + kOwnWaves : nbc - 1 - wave; };
        while (true) {
          load_k_block<D>(ks, N, next_block() << 5, lane, kb);
          process(ka, b);
          b += kOwnWaves;
          if (b >= nbc) {
            if (DOC) copy_block<D>(kb, ka);
            break;
          }
          load_k_block<D>(ks, N, next_block() << 5, lane, ka);
          process(kb, b);
          b += kOwnWaves;
          if (b >= nbc) break;
        }
      }
#pragma unroll
      for (int q = 0; q < QBT; ++q) {
        if (q < QB) {
          float m = m_run[q], z = z_run[q];
          const float m2 = __shfl_xor(m, 32);
          const float z2 = __shfl_xor(z, 32);
          merge_stats(m, z, m2, z2);
          if (h == 0) wstats[wave * RC + q * 32 + t] = make_float2(m, z);
        }
      }
    }

    FINCH_PHASE(1);
    // ---- pass 2 walks the keys from the end (what pass 1 read last is what the
    // caches most likely still hold); its first block is requested before the merge
    b = nbc - 1 - wave;
    if (!DOC) load_k_block<D>(ks, N, b * 32, lane, ka);
    if (tid == 0) *sh_next = kOwnWaves;
    __syncthreads();
    FINCH_PHASE(2);
    for (int i = own_thread(); i < rows; i += kOwnThreads) {
      float l = kInf;  // padding rows add exp2(-inf) = 0
      if (row0 + i < R) {
        float2 a = wstats[i];
#pragma unroll
        for (int w = 1; w < kOwnWaves; ++w) {
          const float2 c = wstats[w * RC + i];
          merge_stats(a.x, a.y, c.x, c.y);
        }
        l = a.x + fast_log2(a.y);
        if (lim_step == 0) {
          if (pb.lse_extra) l = widen_lse(l, as_global<float>(pb.lse_extra)[row0 + i]);
        } else {
          // normalisation step: the row's weights times (keys it sees) / (c + m)
          l -= fast_log2(static_cast<float>(lim0 + i) / static_cast<float>(N));
        }
      }
      lds_lse[i] = l;
      if (ONCE && row0 + i < est.cap) est.lse[row0 + i] = l;
    }
    __syncthreads();
    FINCH_PHASE(3);
    }

    // ---- pass 2, and the selection behind the last chunk of rows.  After the only pass it comes
    // first, and pass 2 is for the keys that it leaves open (`list`; null: all).
    if (LOOP) asm volatile("" ::"v"(asked));
    int n2 = N, nb2 = nbc;
    KeySource ks2 = ks;
    for (int turn = ONCE == kOnceTry ? 1 : 0; turn < 3; ++turn) {
    if (turn != 1) {
      const int tid = own_thread(), lane = tid & 63, t = lane & 31, h = lane >> 5;
      auto process = [&](const bf16x8(&kf)[D / 16], int blk) {
        const int kbase = blk << 5;
        float u[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) u[v] = 0.f;
        auto tile_sums = [&](f32x16 a, int q) {
          const float L = lds_lse[q * 32 + t];
          if (DOC && kbase + 32 > lim_lo(q)) {  // keys this row does not see add nothing
            const int lim = lim_mine(q);
#pragma unroll
            for (int v = 0; v < 16; ++v)
              if (kbase + acc_key(v, h) >= lim) a[v] = -kInf;
          }
#pragma unroll
          for (int v = 0; v < 16; ++v) u[v] += fast_exp2(__builtin_fmaf(a[v], sc, -L));
        };
        auto whole_block = [&](auto qb) {
          constexpr int QBC = decltype(qb)::value;
          float L[QBC];
#pragma unroll
          for (int q = 0; q < QBC; ++q) L[q] = lds_lse[q * 32 + t];
          for_block_logits<D, QBC>(kf, lds_q, lane, [&](int q, int v, float a) { u[v] += fast_exp2(__builtin_fmaf(a, sc, -L[q])); });
          return true;
        };
        if (!WHOLE || kbase + 32 > min(n2, lim0) || !whole(QB, whole_block)) {
          auto pair_visible = [&](int q) { return !DOC || kbase < lim_hi(q + 1 < QB ? q + 1 : q); };
          // pairs of row blocks, the vector work one pair behind the matrix work
          f32x16 acc[QBT];
#pragma unroll
          for (int q = 0; q < QBT + 2; q += 2) {
            if (q < QBT && q < QB && pair_visible(q)) {
              if (q + 1 < QB) {
                mfma_block_pair_lds<D>(kf, lds_q, q, lane, acc[q], acc[q + 1]);
              } else {
                bf16x8 qf0[D / 16];
                load_q_frags<D>(lds_q, q, lane, qf0);
                acc[q] = mfma_block<D>(kf, qf0);
              }
            }
            if (q >= 2 && q - 2 < QB && pair_visible(q - 2)) {
              tile_sums(acc[q - 2], q - 2);
              if (q - 1 < QB) tile_sums(acc[q - 1], q - 1);
            }
          }
        }
        const float tot = fold16_over32(u, t);
        int key = kbase + acc_key(t >> 1, h);
        if ((t & 1) == 0 && key < n2) {
          if (ONCE == kOnceTry) {
            if (ks2.list) key = ks2.list[key];
            lkeys[key] = order_key(tot);
            return;
          }
          float val = tot;
          if (!first_chunk) val += lkeys ? order_value(lkeys[key]) : dst[key];
          if (lkeys) lkeys[key] = order_key(val);
          if (lkeys_sum) return;
          // (scores other workgroups will read go out past this compute unit's caches)
          if (layered) __hip_atomic_store(dst + key, val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          else dst[key] = val;
        }
      };
      // the next key block, or the next chunk's rows when there is none
      auto load_next = [&](int bn, bf16x8(&kf)[D / 16]) {
        if (!DOC || bn >= 0) {
          load_k_block<D>(ks2, n2, bn * 32, lane, kf);
        } else {
          const RowChunk nx = row_chunk(min(ch + 1, n_chunks - 1));
          hold_q<D, kOwnThreads>(nx.qsrc, nx.R, nx.row0, RC, tid, kf);
        }
      };
      if (b >= 0) {
        while (true) {
          int bn = nb2 - 1 - own_next_block(sh_next, lane);
          load_next(bn, kb);
          process(ka, b);
          b = bn;
          if (b < 0) break;
          bn = nb2 - 1 - own_next_block(sh_next, lane);
          load_next(bn, ka);
          process(kb, b);
          b = bn;
          if (b < 0) {
            if (DOC) copy_block<D>(ka, kb);
            break;
          }
        }
      } else {
        load_next(b, kb);
      }
      if (DOC) {
        load_k_block<D>(ks, N, wave << 5, lane, ka);  // the next chunk's first
      } else if (LOOP) {
        // (What is still on its way is awaited here, with few stores behind it.  Left to itself the compiler
        // waits where it takes the registers again, at the next step's start, and there for all stores
        // of the step: 45 of 1020 us in the loop of 1024 problems, 32 rows, 512-token chunks.)
        forget<D>(ka);
        forget<D>(kb);
      }
    FINCH_PHASE(4);
    __syncthreads();  // scores of this row chunk are out; LDS may be restaged
    FINCH_PHASE(5);
    }
    if (!ONCE || !stages || ch + 1 < n_chunks) break;
    const int tid = own_thread(), lane = tid & 63, wave = uni(tid >> 6);
    SelBand band = {turn == 1 ? fast_exp2(spread) * 1.004f : est.room};
    chosen = own_select(prm, pb, slot, N, dst, sel, sel_bytes, lkeys, step_probs, epoch, layered, sync_words, tid, &band);
    FINCH_PHASE(6);
    if (turn == 2) {  // (some of what was learned: 3.80 ms in place of 3.86 in that loop)
      est.room = fmaxf(kEstRoom, 0.5f + 0.5f * est.room);
      break;
    }
    const int n_lo = uni(band.n_lo), open = n_lo - uni(band.n_hi);
    est.dense = !lkeys || (n_lo > pb.r && (n_chunks > 1 || 2 * open * QB + est_fixed<D>(QB) > N * QB));
    // (a step that has tried and started over keeps what it has learned)
    if (turn == 1) est.room = fmaxf(kEstRoom, uni(band.room));
    else if (est.way == 0) est.room = fmaxf(kEstRoom, 0.5f + 0.5f * est.room);
    if (turn != 1) break;
    // Keys below band.thr_lo are out and those above band.thr_hi are in whatever their exact scores are.
    // (The 0.4 % beside the spread are far more than what fp32 sums of exponentials differ by.)
    if (n_lo == pb.r && band.least >= kEstLeast) {
      est.way |= kWaySettled;
      est.longest = 3;
      break;
    }
    if (n_chunks > 1) {  // (rows that are no longer staged)
      no_use(kWayAgain);
      return false;
    }
    // ---- the others one by one
    const unsigned thr_lo = band.thr_lo, thr_hi = band.thr_hi;
    n2 = open;
    unsigned short* const list = reinterpret_cast<unsigned short*>(sel + static_cast<size_t>(RC) * (kOwnWaves * 8 + 4) + 16);
    if (!(band.least >= kEstLeast) || n2 <= 0 || reinterpret_cast<char*>(list + n2) > reinterpret_cast<char*>(lkeys)) {
      n2 = N;
      // (a list that is too long costs another selection and no pass: the next step may well have less to look at.  The
      // loop of 256 problems, 192 rows and 131072 tokens of evenly spread keys: 3.86 ms with a pause after those, 3.57 without)
      est.way |= kWayAll;
      if (!(band.least >= kEstLeast)) no_use(0);
    } else {
      est.way |= kWayList;
      est.longest = 3;
      for (int i0 = 0; i0 < N; i0 += kOwnThreads) {
        const int i = i0 + tid;
        const unsigned key = i < N ? lkeys[i] : 0u;
        const bool mine = i < N && key >= thr_lo && key <= thr_hi;
        const unsigned long long m = __ballot(mine);
        int at = 0;
        if (lane == 0 && m) at = atomicAdd(est.words + 16, __popcll(m));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
        if (mine) list[at] = static_cast<unsigned short>(i);
        else if (i < N) lkeys[i] = order_key(key > thr_hi ? 3.4028234e38f : 0.f);
      }
      ks2.list = list;
    }
    nb2 = (n2 + 31) >> 5;
    if (tid < rows) lds_lse[tid] = est.lse[tid];
    if (tid == 0) *sh_next = kOwnWaves;
    __syncthreads();
    b = nb2 - 1 - wave;
    load_k_block<D>(ks2, n2, b * 32, lane, ka);
    }
  }
  if (lkeys_sum && ONCE != kOnceTry)
    for (int i = tid; i < N; i += kOwnThreads) dst[i] = order_value(lkeys[i]);
  if (DOC && n_chunks == 0) own_no_rows(gscores, lkeys, N, tid);
  // what the prompt-row region of LDS holds now (selection scratch lies behind it)
  staged_q = (n_chunks == 1) ? pb.q : nullptr;
  staged_rows = Rp;
  est.q = Rp <= est.cap ? pb.q : nullptr;
  est.rows = Rp;
  if (!stages) return false;

  // ---- top-r and compaction (the pass-1 statistics are dead)
  if (ONCE) {
    own_compact<D / 8, 8, ROT>(prm, pb, N, chosen, dst, sel, lkeys != nullptr, tid, kept);
    return true;
  }
  own_finish_step<D / 8, 8, ROT>(prm, pb, slot, N, dst, sel, sel_bytes, lkeys, step_probs, epoch, layered, sync_words, tid, kept);
  return layered;
}

// Which slot workgroup b of n takes.  Normally b itself.  With layer groups the L
// workgroups of a run exchange their scores, so runs are kept on one of the chip's eight
// dies (workgroups go to the dies in turn: b % 8) and the exchange stays in that die's L2:
// die x takes the slots [x * (n / 8) + min(x, n % 8), ...) in the order of its workgroups.
__device__ __forceinline__ int own_slot_of(int b, int n, int L) {
  if (L <= 1) return b;
  const int x = b & 7, j = b >> 3;
  return x * (n >> 3) + min(x, n & 7) + j;
}

// Whether a step may leave the rows it keeps where they are: the next step's cache is exactly
// these rows, and the step after that writes as many at the same place.
typedef const __attribute__((address_space(4))) finch_problem* DescriptorPtr;  // (read through the scalar cache, as load_problem does)
typedef const __attribute__((address_space(4))) int* StepTablePtr;
__device__ __forceinline__ bool own_rows_may_stay(DescriptorPtr pb, DescriptorPtr next, DescriptorPtr after, int cap) {
  // (no short cuts: all of it is asked for at once)
  const int r = min(pb->r, pb->c + pb->m), r_after = min(after->r, after->c + after->m);
  const bool rows = (r > 0) & (r <= cap) & (next->c == r) & (r_after >= r);
  const bool places = (next->k_cache == pb->k_out) & (next->v_cache == pb->v_out) & (after->k_out == pb->k_out) & (after->v_out == pb->v_out);
  return rows & places;
}

// One launch = one step of every problem of a batch; workgroup b owns problem b.
// ROT: the compaction re-positions the kept keys (prm.rope_pairing, ascending slots).
template <int D, int QBT, bool ROT, bool DOC>
__global__ __launch_bounds__(kOwnThreads, own_lean(D, QBT, ROT, DOC) ? 4 : 2) void owner_step_bf16(LaunchParams prm, int stages) {
  extern __shared__ __align__(16) char smem[];
  const int p = own_slot_of(blockIdx.x, gridDim.x, stages ? prm.layer_group : 1);
  const finch_problem pb = prm.probs[p];
  const void* staged_q = nullptr;
  int staged_rows = 0;
  KeptRows kept;
  RowEstimates est;
  own_step_body<D, QBT, ROT, DOC, false, 0>(prm, pb, p, stages, smem, staged_q, staged_rows, prm.probs, 0, kept, est);
}

// One launch = the whole chunk loop (Method: Document Segmentation): workgroup b
// owns slot b and runs its steps one after the other; the descriptors of step s
// are prm.probs[step_first[s] + slot] for slot < step_first[s+1] - step_first[s].
// Slots do not depend on each other, so workgroups drift apart and the copy-bound
// and arithmetic-bound stages of different problems overlap.
// Kept rows are moved in a slot's last two steps; before that a step only notes where they lie
// (KeptRows) if own_rows_may_stay says so.  256 problems, 4096-token chunks, up to 1408 kept rows:
// the copies were 20 of 187 us a step, the loop takes 5533 us in place of 6080; 1024 problems of
// 32 rows, 512-token chunks and up to 1024 kept rows, where they were 18 of 42 us: 999 in place of 1354.
template <int D, int QBT, bool ROT, bool DOC, bool ONCE>
__global__ __launch_bounds__(kOwnThreads) void owner_loop_bf16(LaunchParams prm, const int* step_first,
                                                               int n_steps) {
  extern __shared__ __align__(16) char smem[];
  const int slot = own_slot_of(blockIdx.x, gridDim.x, prm.layer_group);
  const void* staged_q = nullptr;
  int staged_rows = 0;
  int epoch = 0;
  KeptRows kept;
  kept.at = reinterpret_cast<int*>(smem + prm.lds_bytes);
  kept.cap = prm.stay_rows;
  const DescriptorPtr probs = (DescriptorPtr)(unsigned long long)prm.probs;
  const StepTablePtr table = (StepTablePtr)(unsigned long long)step_first;
  if (prm.stay_rows > 0) {
    const DescriptorPtr p0 = probs + slot;
    kept.k0 = static_cast<const char*>(p0->m > 0 ? p0->k_chunk : p0->k_cache);
    kept.v0 = static_cast<const char*>(p0->m > 0 ? p0->v_chunk : p0->v_cache);
  }
  RowEstimates est;
  if (ONCE) {
    est.lse = reinterpret_cast<float*>(smem + prm.lds_bytes + 8u * static_cast<unsigned>(prm.stay_rows));
    est.cap = prm.est_words - kEstExtraWords;
    est.words = reinterpret_cast<int*>(est.lse) + est.cap;
  }
  // Descriptors come from memory that this launch has not touched yet, 1 to 2 us away, and a step begins with
  // what it and the two after it say.  So each step asks for the one three steps on (once its own first
  // loads are on their way), to have it in the L2 by then.
  auto descriptor_at = [&](int s) {
    const int at = table[min(s, n_steps - 1)];
    const bool there = s < n_steps && slot < table[s + 1] - at;
    return reinterpret_cast<const int*>(prm.probs + (there ? at : 0) + slot) + (threadIdx.x & 1) * (sizeof(finch_problem) / 4 - 1);
  };
  FINCH_PHASE_BEGIN();
  for (int s = 0; s < n_steps; ++s) {
#ifdef FINCH_PHASE_TIMERS
    if (s > 0) phase_last_ = wall_clock64();
#endif
    const int t0 = table[s], t1 = table[s + 1], t2 = table[min(s + 2, n_steps)], t3 = table[min(s + 3, n_steps)];
    if (slot >= t1 - t0) break;  // slots are filled from the front
    const bool more1 = slot < t2 - t1, more2 = slot < t3 - t2;  // (nobody is present past the last step)
    const DescriptorPtr next = probs + (more1 ? t1 : t0) + slot, after = probs + (more2 ? t2 : t0) + slot;
    kept.stay = own_rows_may_stay(probs + t0 + slot, next, after, prm.stay_rows);
    if (ONCE) {  // (as above)
      const DescriptorPtr here = probs + t0 + slot;
      est.hidden = (more1 & (next->scores == here->scores) & (next->c + next->m >= here->c + here->m)) | !here->scores;
    }
    const finch_problem pb = load_problem(prm.probs + t0 + slot);
    // (rows in a cache that an earlier step has moved would be overwritten while they are still wanted)
    kept.stay = kept.stay && more2 && (s == 0 || pb.c == 0 || kept.mapped);
    est.ask = descriptor_at(s + 3);
    est.way = 0;
    FINCH_PHASE(0);
    if constexpr (ONCE) {
      if (!own_step_body<D, QBT, ROT, DOC, true, kOnceTry>(prm, pb, slot, /*stages=*/1, smem, staged_q, staged_rows, prm.probs + t0,
                                                           epoch, kept, est))
        own_step_body<D, QBT, ROT, DOC, true, kOnceNote>(prm, pb, slot, /*stages=*/1, smem, staged_q, staged_rows, prm.probs + t0,
                                                         epoch, kept, est);
    } else if (own_step_body<D, QBT, ROT, DOC, true, 0>(prm, pb, slot, /*stages=*/1, smem, staged_q, staged_rows, prm.probs + t0,
                                                        epoch, kept, est)) {
      ++epoch;
    }
    if (ONCE && prm.ways && threadIdx.x == 0) prm.ways[static_cast<size_t>(s) * gridDim.x + slot] = est.way;
    // the rows this step wrote are the next step's cache: complete before it reads
    __syncthreads();
  }
}

namespace {

int own_qbt(int row_chunk) {
  const int qb = (row_chunk + 31) / 32;
  const int have[4] = {2, 4, 6, 8};
  for (int i = 0; i < 4; ++i)
    if (qb <= have[i]) return have[i];
  return 0;
}

// Calls f(kernel) for the instantiation that matches (head_dim, qbt, rot).  Returns false for a
// combination that is not built.
#define FINCH_OWN_CASES(KERNEL, ...)                                                      \
  FINCH_OWN_CASE(128, 2, KERNEL, __VA_ARGS__) FINCH_OWN_CASE(128, 4, KERNEL, __VA_ARGS__) \
  FINCH_OWN_CASE(128, 6, KERNEL, __VA_ARGS__) FINCH_OWN_CASE(128, 8, KERNEL, __VA_ARGS__) \
  FINCH_OWN_CASE(64, 2, KERNEL, __VA_ARGS__) FINCH_OWN_CASE(64, 4, KERNEL, __VA_ARGS__)   \
  FINCH_OWN_CASE(64, 6, KERNEL, __VA_ARGS__) FINCH_OWN_CASE(64, 8, KERNEL, __VA_ARGS__)
#define FINCH_OWN_CASE(DD, QQ, KERNEL, ...)         \
  if (head_dim == DD && qbt == QQ) {                \
    if (rot) f(&KERNEL<DD, QQ, true, __VA_ARGS__>); \
    else f(&KERNEL<DD, QQ, false, __VA_ARGS__>);    \
    return true;                                    \
  }
template <bool DOC, typename F>
bool with_step_kernel(int head_dim, int qbt, bool rot, F f) {
  FINCH_OWN_CASES(owner_step_bf16, DOC)
  return false;
}
template <bool DOC, bool ONCE, typename F>
bool with_loop_kernel(int head_dim, int qbt, bool rot, F f) {
  FINCH_OWN_CASES(owner_loop_bf16, DOC, ONCE)
  return false;
}
#undef FINCH_OWN_CASE
#undef FINCH_OWN_CASES

// p.row_chunk and p.lds_bytes must describe this kernel's layout (owner_lds_bytes).
template <bool DOC>
hipError_t launch_owner_impl(int head_dim, const LaunchParams& p, int stages, hipStream_t s) {
  if (p.n_problems <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(p.n_problems)), block(kOwnThreads);
  const bool ok = with_step_kernel<DOC>(head_dim, own_qbt(p.row_chunk), p.rope_pairing != FINCH_ROPE_OFF || p.rank_order,
                                        [&](auto kern) {
                                          hipLaunchKernelGGL(kern, grid, block, p.lds_bytes, s, p, stages);
                                        });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

// The whole loop: n_slots workgroups; step_first is a DEVICE array of n_steps + 1
// offsets into p.probs.
template <bool DOC, bool ONCE>
hipError_t launch_owner_loop_impl(int head_dim, const LaunchParams& p, const int* step_first, int n_steps,
                                  int n_slots, hipStream_t s) {
  if (n_slots <= 0 || n_steps <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(n_slots)), block(kOwnThreads);
  const bool ok = with_loop_kernel<DOC, ONCE>(head_dim, own_qbt(p.row_chunk), p.rope_pairing != FINCH_ROPE_OFF || p.rank_order,
                                        [&](auto kern) {
                                          hipLaunchKernelGGL(kern, grid, block, p.lds_bytes + 8u * static_cast<unsigned>(p.stay_rows) + 4u * static_cast<unsigned>(p.est_words), s,
                                                             p, step_first, n_steps);
                                        });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

// with(head_dim, qbt, rot, f): as above.
template <typename W>
hipError_t set_max_lds_kernels(size_t bytes, W with) {
  hipError_t err = hipSuccess;
  const int dims[2] = {128, 64}, qbts[4] = {2, 4, 6, 8};
  for (int d = 0; d < 2; ++d)
    for (int q = 0; q < 4; ++q)
      for (int rot = 0; rot < 2; ++rot)
        with(dims[d], qbts[q], rot != 0, [&](auto kern) {
          const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                                   static_cast<int>(bytes));
          if (e != hipSuccess) err = e;
        });
  return err;
}
template <bool DOC>
hipError_t set_max_lds_owner_impl(size_t bytes) {
  const hipError_t e = set_max_lds_kernels(bytes, [](int d, int q, bool rot, auto f) { with_step_kernel<DOC>(d, q, rot, f); });
  if (e != hipSuccess) return e;
  return set_max_lds_kernels(bytes, [](int d, int q, bool rot, auto f) { with_loop_kernel<DOC, false>(d, q, rot, f); });
}

}  // namespace

}  // namespace finch
