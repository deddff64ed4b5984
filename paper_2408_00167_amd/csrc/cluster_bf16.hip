// Several workgroups per problem for a whole prefill step in ONE launch, bf16 Q/K/V on
// gfx950: for batches with far fewer problems than the chip has compute units - the KV heads
// of one layer, which is what a model's forward pass has in hand at a time.  Such a step
// moves few bytes; what it costs is latency: launches (3.7 us each, back to back), chains of
// dependent loads, and compute units that have no workgroup.  So a problem's keys are cut
// into S slices, S * problems <= compute units, and one workgroup takes a slice through all
// stages (Method: attention of the prompt rows over cache + chunk keys, sum over heads and
// prompt rows; t = top-r(A_agg, r); Managing the Cache):
//   pass 1   (max, sum exp2) of every prompt row over the slice's keys  -> memory
//   meeting  all slices of the problem have published theirs (1-2 us; a launch would cost 4)
//   pass 2   every row's log-sum-exp from the S records, the slice's scores -> memory
//   meeting  all slices (of the problem; with layer groups, of the layer) have published
//   top-r    by every workgroup for itself on all scores (the same answer everywhere, which
//            is cheaper than a third meeting), then its S-th part of the compaction.
// One layer of 8 KV heads, 192 prompt rows, 4800 candidates: 80.9 us a step with one kernel per
// stage (16 workgroups in each of its two passes, and four launches), 26.5 us with two
// streaming passes here, 22.5 us with the tiles held in registers and the instructions counted:
// a wave issues one every four to five clocks, and 1250 of them stood before the first barrier.
//
// Meetings.  A slice's workgroup sets a flag per meeting; the others poll the flags, at most
// prm.help_ticks in all: the time spent polling counts, not the time spent working.  When it is
// up (other work keeps some of the workgroups from starting), a workgroup does what is missing
// ITSELF - the same instructions on the same
// inputs, hence the same bits, written to the same places - so every workgroup can finish
// whatever the others do, and no wait depends on all of them being on the chip at once.
// A flag is set when it holds the launch's number, generation + 1.  The generation is a
// word of memory that the last workgroup to be through with its waits advances, so a launch
// leaves the words ready for the next one on the same stream and nothing has to be cleared
// in between (a launch that clears them costs 3 us of a step's 15 to 23).  Two launches that
// overlap in time need words of their own; api.hip sees to that.
//
// Data that crosses workgroups goes through agent-scope relaxed atomics (past the caches
// that are not shared), and is complete before the flag: each thread waits for its own
// stores, then a barrier, then the flag.
#include "owner_body.h"

namespace finch {

namespace {

constexpr int kCluThreads = kOwnThreads;
constexpr int kCluWaves = kOwnWaves;

// words of the meeting area (LaunchParams::meet)
constexpr int kMeetGen = 0, kMeetExit = 16, kMeetExitOf = 32;   // (one word per 64-byte line, except:)
constexpr int kMeetFlags = kMeetExitOf + 16 * kMaxClusterGrid;  // [2][kMaxClusterGrid]
static_assert(kMeetFlags + 2 * kMaxClusterGrid == kClusterMeetWords, "size of the meeting area");

template <typename T>
__device__ __forceinline__ T agent_load(const T* p) {
  return __hip_atomic_load((const FINCH_GLOBAL T*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(T* p, T v) {
  __hip_atomic_store((FINCH_GLOBAL T*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// a / b for 0 <= a < 2^20, 0 < b: a fraction of the instructions of an integer division ((a + 1/2)
// / b is at least 1/(2 b) away from the next whole number, far more than the error).
__device__ __forceinline__ int div_small(int a, int b) {
  return static_cast<int>((static_cast<float>(a) + 0.5f) * __builtin_amdgcn_rcpf(static_cast<float>(b)));
}

// Every thread's stores are out; then one thread sets the flag.  Whole workgroup.
__device__ __forceinline__ void meet_set(int* flag, int target, int tid) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) agent_store(flag, target);
}

// Waits until the flags i < n with i % stride < used all hold `target`; -1, or the first missing
// one once `budget` ticks are used up.  What the wait took is taken from `budget` (wave 0 has
// it).  Whole workgroup; a barrier at the end.
__device__ __forceinline__ int meet_wait(const int* flags, int n, int stride, int used, int target, long long& budget,
                                         int* sh, int lane, int wave) {
  if (wave == 0) {
    constexpr int kLoads = kMaxClusterGrid / 64;
    bool want[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int i = lane + 64 * u;
      want[u] = i < n && i - div_small(i, stride) * stride < used;
    }
    const long long end = wall_clock64() + budget;
    long long now = end - budget;
    int missing;
    while (true) {
      missing = -1;
      bool there[kLoads];
#pragma unroll
      for (int u = 0; u < kLoads; ++u) there[u] = 64 * u >= n || agent_load(flags + min(lane + 64 * u, n - 1)) == target;
#pragma unroll
      for (int u = kLoads - 1; u >= 0; --u) {
        const unsigned long long m = __ballot(want[u] && !there[u]);
        if (m) missing = 64 * u + __ffsll(static_cast<long long>(m)) - 1;
      }
      if (missing < 0) break;
      now = wall_clock64();
      if (now >= end) break;
      __builtin_amdgcn_s_sleep(1);
    }
    budget = max(0ll, end - now);
    if (lane == 0) *sh = missing;
  }
  __syncthreads();
  const int r = *sh;
  __syncthreads();  // (*sh may be written again)
  return r;
}

// One 32-key block of K as MFMA A operands (see load_k_block); rows from `lim` on repeat the
// last one below it - their logits are masked, or their sums not used.
template <int D>
__device__ __forceinline__ void load_k_rows(const KeySource& ks, int lim, int kbase, int lane, bf16x8 (&kf)[D / 16]) {
  const int key = min(kbase + (lane & 31), lim - 1);
  const char* base = key < ks.c ? ks.cache : ks.chunk;
  const int row = key < ks.c ? key : key - ks.c;
  const FINCH_GLOBAL u32x4* rp = as_global<u32x4>(base + static_cast<size_t>(row) * (D * 2) + (lane >> 5) * 16);
#pragma unroll
  for (int s = 0; s < D / 16; ++s) kf[s] = __builtin_bit_cast(bf16x8, static_cast<u32x4>(rp[2 * s]));
}

// Prompt rows [row0, row0 + 32 qb) into LDS as stage_q does, rows from R on repeating row R - 1
// (what comes of them is not used).  All of a thread's loads are in flight together: TURNS,
// at least the turns the rows take; turns past the last repeat it.
template <int D, int TURNS>
__device__ __forceinline__ void stage_rows_turns(const void* q, int R, int row0, int qb, char* lds_q, int tid) {
  constexpr int kSegs = D / 8, kStride = D * 2 + 16, kRows = kCluThreads / kSegs;  // rows per turn
  const FINCH_GLOBAL u32x4* src = as_global<u32x4>(q);
  const int sub = tid / kSegs, seg = tid % kSegs;
  u32x4 val[TURNS];
#pragma unroll
  for (int u = 0; u < TURNS; ++u)
    val[u] = src[static_cast<unsigned>(min(row0 + min(u * kRows + sub, 32 * qb - 1), R - 1)) * kSegs + seg];
#pragma unroll
  for (int u = 0; u < TURNS; ++u)
    *reinterpret_cast<u32x4*>(lds_q + min(u * kRows + sub, 32 * qb - 1) * kStride + seg * 16) = val[u];
}
template <int D>
__device__ __forceinline__ void stage_rows(const void* q, int R, int row0, int qb, char* lds_q, int tid) {
  constexpr int kMost = kOwnerMaxRowChunk * (D / 8) / kCluThreads;  // turns of the largest chunk
  const int turns = (32 * qb * (D / 8) + kCluThreads - 1) / kCluThreads;
  if (turns * 4 <= kMost) stage_rows_turns<D, kMost / 4>(q, R, row0, qb, lds_q, tid);
  else stage_rows_turns<D, kMost>(q, R, row0, qb, lds_q, tid);
}

// Scores other workgroups have written.
struct AgentScoreVector {
  const float* p;
  __device__ __forceinline__ float operator()(int i) const { return agent_load(p + i); }
};

// Key blocks [b0, b1) of slice s of `per` blocks each.
struct Slice {
  int b0, b1;
};
__device__ __forceinline__ Slice slice_of(int nb, int per, int s) { return Slice{min(nb, s * per), min(nb, (s + 1) * per)}; }

// How the 8 waves share a slice of kb key blocks and qb row blocks: groups of rs = 2^lg waves
// take the same keys and different rows.  The split with the shortest longest
// wave, loading a key block counted like one tile of work; of equal ones the one that loads
// each key least often.  Slices of more than kSplitBlocks are not split by rows: their waves
// have keys enough.
constexpr int kSplitBlocks = 2 * kCluWaves;
__device__ __forceinline__ int row_split_log2(int kb, int qb) {
  int best = 0, cost = 1 << 30;
#pragma unroll
  for (int lg = 0; lg <= 3; ++lg) {
    const int blocks = ((kb << lg) + kCluWaves - 1) / kCluWaves, rows = (qb + (1 << lg) - 1) >> lg;
    if (blocks * (rows + 1) < cost && (lg == 0 || kb <= kSplitBlocks)) {
      cost = blocks * (rows + 1);
      best = lg;
    }
  }
  return best;
}

// HELD: the kb * qb tiles of 32 keys x 32 rows of a slice, key block by key block, are dealt out
// in runs of `held_run`, at most kHeldTiles, to the waves, which keep them in registers from
// pass 1 to pass 2.  A run reaches over at most two key blocks.
constexpr int kHeldTiles = 4;
__host__ __device__ inline int held_run(int kb, int qb) { return (kb * qb + kCluWaves - 1) / kCluWaves; }
inline bool can_hold(int kb, int qb) {
  const int run = held_run(kb, qb);
  return run <= kHeldTiles && run <= qb + 1 && kb <= kCluWaves;
}

// n <= W (maximum, sum) records, `stride` apart, merged: all reads first, one maximum, one sum.
template <int W>
__device__ __forceinline__ float2 merge_records(const float2* rec, int stride, int n) {
  float2 r[W];
#pragma unroll
  for (int w = 0; w < W; ++w) r[w] = rec[min(w, n - 1) * stride];
  float m = r[0].x;
#pragma unroll
  for (int w = 1; w < W; ++w) m = fmaxf(m, r[w].x);
  const float mu = (m == -kInf) ? 0.f : m;
  float z = 0.f;
#pragma unroll
  for (int w = 0; w < W; ++w) z += w < n ? r[w].y * fast_exp2(r[w].x - mu) : 0.f;
  return make_float2(m, z);
}

// 64 keys x 32 rows of raw dot products, or (not TWO) the first 32 keys only.  The prompt rows'
// operands are read once for both halves.
template <int D, bool TWO>
__device__ __forceinline__ void mfma_rows(const bf16x8 (&k0)[D / 16], const bf16x8 (&k1)[D / 16], const char* qrow, f32x16& a0,
                                          f32x16& a1) {
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x8 qf[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qrow + 32 * s);
  a0 = zero;
  a1 = zero;
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    a0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0[s], qf[s], a0, 0, 0, 0);
    if (TWO) a1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1[s], qf[s], a1, 0, 0, 0);
  }
}

// Key blocks a wave takes at a time, of a slice of kb that kl waves share: three where that is all it
// has - a third one loaded when the first two were done with stood in both passes' way, as its
// first two had to be loaded again in pass 2 - else two, which read the rows' operands once.
// (32 problems of 128 channels and 256 rows, 2944 candidates: 37.0 us a step, 41.7 by twos; 4992: 46.7
// and 50.6.  Five blocks a wave, 10192 candidates: 85.5 by threes, 82.3 by twos.)
__device__ __forceinline__ int blocks_at_a_time(int kb, int kl) { return kb <= 3 * kl ? 3 : 2; }

__device__ __forceinline__ void mask_keys(f32x16& a, int kbase, int h, int lim) {
  if (kbase + 32 > lim) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (kbase + acc_key(v, h) >= lim) a[v] = -kInf;
  }
}

}  // namespace

// stages: 0 = scores only, 1 = scores, top-r and compaction.  ROT: the compaction
// re-positions the kept keys (ascending slots).
// HELD: every problem's slices fit into the waves' registers (the host has checked it): the
// exponentials of pass 1 stay there and pass 2 only scales and adds them, so that the logits
// are formed once.
template <int D, bool ROT, bool HELD>
__global__ __launch_bounds__(kCluThreads) void cluster_step_bf16(LaunchParams prm, int stages) {
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int t = lane & 31, h = lane >> 5;
  constexpr int kStride = D * 2 + 16;
  // (what the launch was called with, in one go: left to itself the compiler fetches some of it in
  // turn before the descriptor, each time with a wait)
  asm volatile("" ::"s"(prm.probs), "s"(prm.n_problems), "s"(prm.group), "s"(prm.rpad_max), "s"(prm.row_chunk), "s"(prm.layer_group),
               "s"(prm.cluster_slices), "s"(prm.meet), "s"(prm.help_ticks), "s"(prm.stats), "s"(prm.scale_log2), "s"(stages));
  const int S = prm.cluster_slices, RC = prm.row_chunk;
  const int L = stages ? prm.layer_group : 1;
  // a problem's workgroups (and a layer's) stand together on one of the chip's dies where the
  // numbers allow it
  const int role = own_slot_of(blockIdx.x, gridDim.x, 2);
  const int my_p = uni(div_small(role, S)), my_s = role - my_p * S;
  const int cluster = uni(div_small(my_p, L)), p_first = cluster * L;  // the problems that select together
  int* const meet = prm.meet;
  int gen = agent_load(meet + kMeetGen);  // (looked at when it is needed: it comes from far away)
  int* const stat_flags = meet + kMeetFlags;
  int* const score_flags = stat_flags + kMaxClusterGrid;
  long long budget = prm.help_ticks;  // how long this workgroup still waits for others
  const finch_problem mine = load_problem(prm.probs + my_p);
  const int N = mine.c + mine.m;
  const float sc = prm.scale_log2;

  char* lds_q = smem;
  float2* wstats = reinterpret_cast<float2*>(smem + RC * kStride);                             // [waves][RC]
  float* lds_lse = reinterpret_cast<float*>(smem + RC * (kStride + kCluWaves * 8));             // [RC]
  int* sh_miss = reinterpret_cast<int*>(smem + RC * (kStride + kCluWaves * 8 + 4));
  float* ksum = reinterpret_cast<float*>(smem + RC * (kStride + kCluWaves * 8 + 4) + 16);       // [row split][keys of the slice]

  // What this workgroup is working on: a slice of its own problem, or - after a wait that has
  // run out - one that is missing.
  finch_problem pb = mine;
  int wp = my_p, ws = my_s;
  int staged_row0 = -1;  // first of the prompt rows of `pb` that are in LDS (-1: none)
  while (true) {
    const int n = pb.c + pb.m, nb = (n + 31) >> 5, R = prm.group * pb.n_que;
    const int per = max(1, uni(div_small(nb + S - 1, S)));
    const int used = uni(div_small(nb + per - 1, per));  // slices that have keys
    const KeySource ks = {static_cast<const char*>(pb.k_cache), static_cast<const char*>(pb.k_chunk), pb.c};
    unsigned long long* const stats =
        reinterpret_cast<unsigned long long*>(prm.stats) + static_cast<size_t>(wp) * S * prm.rpad_max;
    auto stage = [&](int row0, int rows) {
      if (staged_row0 == row0) return;
      int own_tid = tid;  // (opaque: the addresses are not worth keeping through the loops)
      asm volatile("" : "+v"(own_tid));
      stage_rows<D>(pb.q, R, row0, rows >> 5, lds_q, own_tid);
      staged_row0 = row0;
    };
    if (ws < used) {
      bf16x8 k0[D / 16], k1[D / 16], k2[D / 16];
      // slice whose key blocks are in k0, k1, k2 (if a wave has no more than three), or whose tiles are held
      int held = -1;
      f32x16 tile[HELD ? kHeldTiles : 1];     // exp2(logit - tile_ref), tile_ref per lane
      float tile_ref[HELD ? kHeldTiles : 1];
      bool met = false;
      // ---- pass 1, and the first meeting
      int s1 = ws;
      while (true) {
        const Slice sl = slice_of(nb, per, s1);
        const int kb = sl.b1 - sl.b0, lim = min(n, sl.b1 << 5);
        for (int row0 = 0; row0 < R; row0 += RC) {
          const int rows = min(RC, round_up32(R - row0)), QB = rows >> 5;
          const int lg = row_split_log2(kb, QB), rs = 1 << lg, kl = kCluWaves >> lg;
          const int qper = (QB + rs - 1) >> lg;
          const int q_lo = min(QB, (wave & (rs - 1)) * qper), q_hi = min(QB, q_lo + qper);
          const int kw = wave >> lg;
          float2* const out = wstats + kw * RC;
          int b = sl.b0 + kw;
          // HELD: this wave's tiles [f0, f1), the first j1 of them in key block hb, the others in
          // the next
          const int f0 = min(kb * QB, wave * held_run(kb, QB)), f1 = min(kb * QB, f0 + held_run(kb, QB));
          const int hb = uni(div_small(f0, QB)), hq = f0 - hb * QB, nt = f1 - f0, j1 = QB - hq;
          if constexpr (HELD) {
            if (nt > 0) load_k_rows<D>(ks, lim, (sl.b0 + hb) << 5, lane, k0);
            if (nt > j1) load_k_rows<D>(ks, lim, (sl.b0 + hb + 1) << 5, lane, k1);
          } else {
            if (b < sl.b1) load_k_rows<D>(ks, lim, b << 5, lane, k0);
            if (b + kl < sl.b1) load_k_rows<D>(ks, lim, (b + kl) << 5, lane, k1);
            if (kb <= 3 * kl && b + 2 * kl < sl.b1) load_k_rows<D>(ks, lim, (b + 2 * kl) << 5, lane, k2);
          }
          stage(row0, rows);
          __syncthreads();
          if constexpr (HELD) {
#pragma unroll
            for (int j = 0; j < kHeldTiles; ++j) {
              if (j < nt) {
                if (j == j1) {
#pragma unroll
                  for (int s = 0; s < D / 16; ++s) k0[s] = k1[s];
                }
                const int q = j < j1 ? hq + j : j - j1;
                bf16x8 qf[D / 16];
                load_q_frags<D>(lds_q, q, lane, qf);
                tile[j] = mfma_block<D>(k0, qf);
              }
            }
#pragma unroll
            for (int j = 0; j < kHeldTiles; ++j) {
              if (j < nt) {
                const int q = j < j1 ? hq + j : j - j1, bk = j < j1 ? hb : hb + 1;
                mask_keys(tile[j], (sl.b0 + bk) << 5, h, lim);
                float m = fmaxf(tile[j][0], tile[j][1]);
#pragma unroll
                for (int v = 2; v < 16; v += 2) m = fmaxf(fmaxf(m, tile[j][v]), tile[j][v + 1]);
                m *= sc;
                tile_ref[j] = m;
                const float mu = (m == -kInf) ? 0.f : m;
                float z = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                  tile[j][v] = fast_exp2(__builtin_fmaf(tile[j][v], sc, -mu));
                  z += tile[j][v];
                }
                const float m2 = __shfl_xor(m, 32);
                const float z2 = __shfl_xor(z, 32);
                merge_stats(m, z, m2, z2);
                // (tiles formed once more: their statistics are published, and these words are
                // pass 2's from here on - no barrier lies between)
                if (h == 0 && !met) wstats[bk * RC + q * 32 + t] = make_float2(m, z);
              }
            }
          } else {
            auto keep = [&](int q, float m, float z, bool first) {
              const float m2 = __shfl_xor(m, 32);
              const float z2 = __shfl_xor(z, 32);
              merge_stats(m, z, m2, z2);
              if (h == 0) {
                if (!first) {
                  const float2 o = out[q * 32 + t];
                  merge_stats(m, z, o.x, o.y);
                }
                out[q * 32 + t] = make_float2(m, z);
              }
            };
            // key block blk (and blk + kl) against this wave's row blocks
            auto blocks = [&](const bf16x8(&kx)[D / 16], const bf16x8(&ky)[D / 16], int blk, bool first, auto two) {
              constexpr bool TWO = decltype(two)::value;
              const bool ragged = (blk + (TWO ? kl : 0) + 1) << 5 > lim;
              for (int q = q_lo; q < q_hi; ++q) {
                f32x16 a0, a1;
                mfma_rows<D, TWO>(kx, ky, lds_q + (q * 32 + t) * kStride + 16 * h, a0, a1);
                if (ragged) {
                  mask_keys(a0, blk << 5, h, lim);
                  if (TWO) mask_keys(a1, (blk + kl) << 5, h, lim);
                }
                float bm = fmaxf(a0[0], a0[1]);
#pragma unroll
                for (int v = 2; v < 16; v += 2) bm = fmaxf(fmaxf(bm, a0[v]), a0[v + 1]);
                if (TWO) {
#pragma unroll
                  for (int v = 0; v < 16; v += 2) bm = fmaxf(fmaxf(bm, a1[v]), a1[v + 1]);
                }
                const float m = bm * sc;
                const float mu = (m == -kInf) ? 0.f : m;
                float z = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) z += fast_exp2(__builtin_fmaf(a0[v], sc, -mu));
                if (TWO) {
#pragma unroll
                  for (int v = 0; v < 16; ++v) z += fast_exp2(__builtin_fmaf(a1[v], sc, -mu));
                }
                keep(q, m, z, first);
              }
            };
            if (b >= sl.b1)
              for (int q = q_lo; q < q_hi; ++q) keep(q, -kInf, 0.f, true);
            const int turn = blocks_at_a_time(kb, kl) * kl;
            for (bool first = true; b < sl.b1; first = false) {
              if (b + kl < sl.b1) blocks(k0, k1, b, first, std::true_type{});
              else blocks(k0, k0, b, first, std::false_type{});
              if (turn == 3 * kl && b + 2 * kl < sl.b1) blocks(k2, k2, b + 2 * kl, false, std::false_type{});
              b += turn;
              if (b < sl.b1) load_k_rows<D>(ks, lim, b << 5, lane, k0);
              if (b + kl < sl.b1) load_k_rows<D>(ks, lim, (b + kl) << 5, lane, k1);
            }
          }
          held = (HELD || (kb <= 3 * kl && R <= RC)) ? s1 : -1;
          if (met) break;  // (only the tiles were wanted)
          __syncthreads();
          for (int i = tid; i < rows; i += kCluThreads) {
            const float2 a = merge_records<kCluWaves>(wstats + i, RC, HELD ? kb : kl);
            agent_store(stats + static_cast<size_t>(s1) * prm.rpad_max + row0 + i,
                        static_cast<unsigned long long>(__float_as_uint(a.x)) |
                            (static_cast<unsigned long long>(__float_as_uint(a.y)) << 32));
          }
          if (row0 + RC < R) __syncthreads();  // (the staged rows and the statistics are replaced)
        }
        if (met) break;
        asm volatile("" : "+v"(gen));
        const int target = uni(gen) + 1;
        meet_set(stat_flags + wp * S + s1, target, tid);
        s1 = meet_wait(stat_flags + wp * S, used, S, used, target, budget, sh_miss, lane, wave);
        if (s1 < 0) {
          if (!HELD || held == ws) break;
          // others' work has been done in between: this slice's tiles once more
          met = true;
          s1 = ws;
        }
      }

      // ---- pass 2: the scores of slice ws
      const Slice sl = slice_of(nb, per, ws);
      const int kb = sl.b1 - sl.b0, lim = min(n, sl.b1 << 5);
      int rs_used = 1;
      for (int row0 = 0; row0 < R; row0 += RC) {
        const int rows = min(RC, round_up32(R - row0)), QB = rows >> 5;
        // (the split of the largest chunk of rows serves all: the partial sums of the chunks meet in ksum)
        const int lg = row_split_log2(kb, min(RC, round_up32(R)) >> 5), rs = 1 << lg, kl = kCluWaves >> lg;
        rs_used = rs;
        const int qper = (QB + rs - 1) >> lg;
        const int rq = wave & (rs - 1);
        const int q_lo = min(QB, rq * qper), q_hi = min(QB, q_lo + qper);
        int b = sl.b0 + (wave >> lg);
        if (!HELD && held != ws) {
          if (b < sl.b1) load_k_rows<D>(ks, lim, b << 5, lane, k0);
          if (b + kl < sl.b1) load_k_rows<D>(ks, lim, (b + kl) << 5, lane, k1);
          if (kb <= 3 * kl && b + 2 * kl < sl.b1) load_k_rows<D>(ks, lim, (b + 2 * kl) << 5, lane, k2);
        }
        stage(row0, rows);
        // every row's log-sum-exp: parts of the S records side by side, then merged
        const int parts = min(kCluWaves, uni(div_small(kCluThreads, rows)));
        const int part = div_small(tid, rows), i = tid - part * rows;
        if (part < parts) {
          float m = -kInf, z = 0.f;
          auto merge_from = [&](int s0, auto batch) {  // records s0, s0 + parts, ...; all loads in flight
            constexpr int kBatch = decltype(batch)::value;
            float2 rec[kBatch];
            const unsigned off = static_cast<unsigned>(s0 * prm.rpad_max + row0 + i);
            const unsigned last = static_cast<unsigned>((used - 1) * prm.rpad_max + row0 + i);
            const unsigned step = static_cast<unsigned>(parts * prm.rpad_max);
            unsigned long long w[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) w[u] = agent_load(stats + min(off + u * step, last));
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
              rec[u].x = off + u * step <= last ? __uint_as_float(static_cast<unsigned>(w[u])) : -kInf;
              rec[u].y = __uint_as_float(static_cast<unsigned>(w[u] >> 32));
            }
            float mm = m;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) mm = fmaxf(mm, rec[u].x);
            if (mm != -kInf) {  // (exp2(-inf) = 0)
              z *= fast_exp2(m - mm);
#pragma unroll
              for (int u = 0; u < kBatch; ++u) z += rec[u].y * fast_exp2(rec[u].x - mm);
            }
            m = mm;
          };
          if (used <= 2 * parts) {
            merge_from(part, std::integral_constant<int, 2>{});
          } else if (used <= 4 * parts) {
            merge_from(part, std::integral_constant<int, 4>{});
          } else {
            for (int s0 = part; s0 < used; s0 += 16 * parts) merge_from(s0, std::integral_constant<int, 16>{});
          }
          wstats[part * RC + i] = make_float2(m, z);
        }
        __syncthreads();
        if (tid < rows) {
          float l = kInf;  // padding rows add exp2(-inf) = 0
          if (row0 + tid < R) {
            const float2 a = merge_records<kCluWaves>(wstats + tid, RC, parts);
            l = a.x + fast_log2(a.y);
            if (pb.lse_extra) l = widen_lse(l, as_global<float>(pb.lse_extra)[row0 + tid]);
          }
          lds_lse[tid] = l;
        }
        __syncthreads();
        if constexpr (HELD) {
          // sums of the (at most two) key blocks of this wave's tiles: ksum[wave][2][32]
          const int f0 = min(kb * QB, wave * held_run(kb, QB)), f1 = min(kb * QB, f0 + held_run(kb, QB));
          const int hq = f0 - uni(div_small(f0, QB)) * QB, nt = f1 - f0, j1 = QB - hq;
          float u[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) u[v] = 0.f;
          float* const o = ksum + wave * 64 + acc_key(t >> 1, h);
#pragma unroll
          for (int j = 0; j < kHeldTiles; ++j) {
            if (j < nt) {
              if (j == j1) {
                const float tot = fold16_over32(u, t);
                if ((t & 1) == 0) o[0] = tot;
#pragma unroll
                for (int v = 0; v < 16; ++v) u[v] = 0.f;
              }
              const float w = fast_exp2(tile_ref[j] - lds_lse[(j < j1 ? hq + j : j - j1) * 32 + t]);
#pragma unroll
              for (int v = 0; v < 16; ++v) u[v] = __builtin_fmaf(tile[j][v], w, u[v]);
            }
          }
          const float tot = fold16_over32(u, t);
          if (nt > 0 && (t & 1) == 0) o[nt > j1 ? 32 : 0] = tot;
        } else {
          auto blocks = [&](const bf16x8(&kx)[D / 16], const bf16x8(&ky)[D / 16], int blk, auto two) {
            constexpr bool TWO = decltype(two)::value;
            float u0[16], u1[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              u0[v] = 0.f;
              u1[v] = 0.f;
            }
            for (int q = q_lo; q < q_hi; ++q) {
              f32x16 a0, a1;
              mfma_rows<D, TWO>(kx, ky, lds_q + (q * 32 + t) * kStride + 16 * h, a0, a1);
              const float lse = lds_lse[q * 32 + t];
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                u0[v] += fast_exp2(__builtin_fmaf(a0[v], sc, -lse));
                if (TWO) u1[v] += fast_exp2(__builtin_fmaf(a1[v], sc, -lse));
              }
            }
            float* const o = ksum + (rq * kb + (blk - sl.b0)) * 32 + acc_key(t >> 1, h);
            const float s0 = fold16_over32(u0, t);
            if ((t & 1) == 0) *o = row0 == 0 ? s0 : *o + s0;
            if (TWO) {
              const float s2 = fold16_over32(u1, t);
              float* const o1 = o + kl * 32;
              if ((t & 1) == 0) *o1 = row0 == 0 ? s2 : *o1 + s2;
            }
          };
          const int turn = blocks_at_a_time(kb, kl) * kl;
          while (b < sl.b1) {
            if (b + kl < sl.b1) blocks(k0, k1, b, std::true_type{});
            else blocks(k0, k0, b, std::false_type{});
            if (turn == 3 * kl && b + 2 * kl < sl.b1) blocks(k2, k2, b + 2 * kl, std::false_type{});
            b += turn;
            if (b < sl.b1) load_k_rows<D>(ks, lim, b << 5, lane, k0);
            if (b + kl < sl.b1) load_k_rows<D>(ks, lim, (b + kl) << 5, lane, k1);
          }
        }
        __syncthreads();
      }
      float* const dst = pb.scores ? pb.scores : prm.ws_scores + static_cast<size_t>(wp) * prm.score_stride;
      for (int i = tid; i < kb * 32; i += kCluThreads) {
        float v = 0.f;
        if constexpr (HELD) {
          // the waves whose runs reach into key block i / 32, in order
          const int QB = round_up32(R) >> 5, run = held_run(kb, QB), bk = i >> 5;
          for (int w = div_small(bk * QB, run); w * run < (bk + 1) * QB && w < kCluWaves; ++w)
            v += ksum[w * 64 + (w * run < bk * QB ? 32 : 0) + (i & 31)];
        } else {
          for (int w = 0; w < rs_used; ++w) v += ksum[w * kb * 32 + i];
        }
        const int key = (sl.b0 << 5) + i;
        if (key < n) agent_store(dst + key, v);
      }
      meet_set(score_flags + wp * S + ws, uni(gen) + 1, tid);
    }
    // ---- the second meeting: the scores of every problem of the run
    if (!stages) break;
    // (they have the same number of candidates, hence of slices with keys)
    const int nb_mine = (N + 31) >> 5, per_mine = max(1, uni(div_small(nb_mine + S - 1, S)));
    const int used_mine = uni(div_small(nb_mine + per_mine - 1, per_mine));
    if (used_mine == 0) break;
    const int miss = meet_wait(score_flags + p_first * S, L * S, S, used_mine, uni(gen) + 1, budget, sh_miss, lane, wave);
    if (miss < 0) break;
    const int g = div_small(miss, S);
    wp = uni(p_first + g);
    ws = uni(miss - g * S);
    pb = load_problem(prm.probs + wp);
    staged_row0 = -1;  // (its rows may lie at the same place and be more or fewer)
  }

  // This workgroup waits for nobody any more.  The last one to come here advances the
  // generation (two levels of counters, so that no word sees all workgroups).  What the
  // counters answer is looked at further down, when it has arrived.
  const int members = L * S;
  // (the status word of waits that expire: here none does)
  if (L > 1 && tid == 0 && role == 0) *as_global_mut<int>(prm.layer_err) = 0;
  int left = 0;
  if (tid == 0) left = __hip_atomic_fetch_add(meet + kMeetExitOf + 16 * cluster, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  auto leave = [&]() {
    if (tid == 0 && left == members - 1) {
      agent_store(meet + kMeetExitOf + 16 * cluster, 0);
      const int clusters = div_small(prm.n_problems, L);
      if (__hip_atomic_fetch_add(meet + kMeetExit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == clusters - 1) {
        agent_store(meet + kMeetExit, 0);
        agent_store(meet + kMeetGen, gen + 1);
      }
    }
  };
  const int r = min(mine.r, N);
  if (!stages || r <= 0) {
    leave();
    return;
  }

  // ---- top-r
  FINCH_GLOBAL int* gidx = as_global_mut<int>(mine.idx);
  const bool identity = r >= N;
  SelLds* fl = reinterpret_cast<SelLds*>(smem);
  int* lidx = reinterpret_cast<int*>(smem + sizeof(SelLds));
  unsigned* lkeys = reinterpret_cast<unsigned*>(lidx + ((r + kSelIdxPad + 3) & ~3));
  __syncthreads();  // (the scratch lies over what the passes used)
  if (!identity) {
    if (L > 1) {
      if (tid < L) {
        const finch_problem* pg = prm.probs + p_first + tid;
        fl->layer_src[tid] = pg->scores ? pg->scores : prm.ws_scores + static_cast<size_t>(p_first + tid) * prm.score_stride;
      }
      __syncthreads();
      sel_stage_layer_keys<kCluThreads>(fl->layer_src, L, N, lkeys, tid);
    } else {
      const AgentScoreVector own{mine.scores ? mine.scores : prm.ws_scores + static_cast<size_t>(my_p) * prm.score_stride};
      // (more than 4096 candidates in one go rather than in two, one wait for the L2 after the other: 8 problems of 4800
      // candidates, 192 rows 22.5 -> 22.1 us; up to 4096 the idle half of the loads would cost 0.3 us of instructions)
      if (N > 8 * kCluThreads) sel_stage_keys_batch<kCluThreads, 16>(own, N, lkeys, tid);
      else sel_stage_keys<kCluThreads>(own, N, lkeys, tid);
    }
    __syncthreads();
    select_keys_any<kCluThreads, true>(lkeys, N, r, gidx, lidx, fl, tid, lane, wave);
    __syncthreads();
  }
  leave();

  // ---- this workgroup's part of the compaction
  const int t_per = uni(div_small(r + S - 1, S));
  const int t0 = min(r, t_per * my_s), t1 = min(r, t0 + t_per);
  for (int i = t0 + tid; i < t1; i += kCluThreads) gidx[i] = identity ? i : lidx[i];
  // (a part is mostly no more than one or two turns of rows: what counts then is the number of instructions)
  constexpr int kTurn = kCluThreads / (D / 8);
  if (ROT) {
    if (t_per <= 2 * kTurn)
      own_gather_rot<D / 8, kCluThreads, 8, 1>(mine, N, r, lidx, gidx, identity, prm.rope_pairing, prm.rope_log2_base, tid, nullptr, t0, t1);
    else
      own_gather_rot<D / 8, kCluThreads, 8>(mine, N, r, lidx, gidx, identity, prm.rope_pairing, prm.rope_log2_base, tid, nullptr, t0, t1);
  } else if (t_per <= kTurn) {
    own_gather<D / 8, kCluThreads, 1>(mine, N, lidx, gidx, identity, tid, t0, t1);
  } else {
    own_gather<D / 8, kCluThreads, 4>(mine, N, lidx, gidx, identity, tid, t0, t1);
  }
}

namespace {

template <typename F>
bool with_cluster_kernel(int head_dim, bool rot, bool held, F f) {
#define FINCH_CLU_CASE(DD, HH)                      \
  if (head_dim == DD && held == HH) {               \
    if (rot) f(&cluster_step_bf16<DD, true, HH>);   \
    else f(&cluster_step_bf16<DD, false, HH>);      \
    return true;                                    \
  }
  FINCH_CLU_CASE(128, true) FINCH_CLU_CASE(128, false) FINCH_CLU_CASE(64, true) FINCH_CLU_CASE(64, false)
#undef FINCH_CLU_CASE
  return false;
}

}  // namespace

// LDS of a launch: the passes' (row_chunk staged rows, slices of at most slice_blocks key
// blocks) or the selection's (n_max candidates, r_max kept), whichever is more.
size_t cluster_lds_bytes(int head_dim, int row_chunk, int slice_blocks, int n_max, int r_max) {
  // a slice of at most kSplitBlocks may be split by rows, each part with sums of its own
  const int blocks = kSplitBlocks * kCluWaves > slice_blocks ? kSplitBlocks * kCluWaves : slice_blocks;
  const size_t sums = static_cast<size_t>(blocks) * 32 * 4;
  const size_t passes = static_cast<size_t>(row_chunk) * (head_dim * 2 + 16 + kCluWaves * 8 + 4) + 16 + sums;
  const size_t select = sizeof(SelLds) + (static_cast<size_t>(r_max) + kSelIdxPad + 3 + n_max) * 4;
  return passes > select ? passes : select;
}

hipError_t launch_cluster_bf16(int head_dim, const LaunchParams& p, int n_max, int stages, hipStream_t s) {
  if (p.n_problems <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(p.n_problems) * static_cast<unsigned>(p.cluster_slices)), block(kCluThreads);
  // (what holds for every number of key and row blocks up to the largest)
  const int blocks = ((n_max + 31) / 32 + p.cluster_slices - 1) / p.cluster_slices;
  bool held = p.rpad_max <= p.row_chunk;
  for (int kb = 1; kb <= blocks && held; ++kb)
    for (int qb = 1; qb <= p.rpad_max / 32 && held; ++qb) held = can_hold(kb, qb);
  const bool ok = with_cluster_kernel(head_dim, p.rope_pairing != FINCH_ROPE_OFF, held, [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, p.lds_bytes, s, p, stages);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t set_max_lds_cluster(size_t bytes) {
  hipError_t err = hipSuccess;
  for (int d = 64; d <= 128; d += 64)
    for (int v = 0; v < 4; ++v)
      with_cluster_kernel(d, (v & 1) != 0, (v & 2) != 0, [&](auto kern) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
        if (e != hipSuccess) err = e;
      });
  return err;
}

}  // namespace finch
