// Single-launch prune: score -> Top_T -> compaction (Sec. 3.2 selection, Fig. 1 storage) with
// NOTHING before or after the one kernel -- gfx950, wave64.
//
// The three-launch form (thk_prune_fused.hip) needs a kernel in front that clears the hand-off
// state and computes the query norms, and one behind that compacts what a block left undone
// when its bounded wait ran out.  For calls of a few hundred microseconds and less those two
// launches and the gaps around them are 10-15 % of the call.  Here both jobs move inside:
//
//   * Blocks 0 .. U-1 of the grid are PROLOGUE blocks, one per unit, the U * NB row blocks of
//     k_prune_onepass follow.  A prologue block has no rows; it clears its unit's hand-off state
//     (index-list words, query-norm words, group vectors, give-up flags and tickets), waits until
//     all of that has been acknowledged, initialises the unit's arrival counters, and only then
//     computes the query norms, whose words carry a validity mark: they are wanted last, and with
//     them in front of the counters (4.5 us into the launch) every row block of a short call
//     waited for the prologue.  (A unit's prologue block directly in front of its row blocks, the
//     first layout, put NB + 1 blocks per unit into a chip that holds a whole number of NB-block
//     units: units straddled the rounds of resident blocks and long launches ran 6-12 % slower.)
//   * The arrival counters are the first shared thing a row block touches, and they are TAGGED:
//     the upper 48 bits hold the call's nonce.  A block whose atomic add returns a word with
//     another tag has arrived before the prologue's initialisation (which will overwrite what
//     it added): it waits for the tag and adds again.  A block that has arrived under the right
//     tag is thereby ordered after everything the prologue cleared.  Nothing has to be clean
//     when the kernel starts.  The block that completes a counter stores 0 into it, so that a
//     replay of the same launch from a graph, which carries the same nonce, does not mistake
//     the previous replay's count for its own.
//   * One block of every unit waits for no other row block: the FINISHER, whose arrival completes
//     the unit's sums.  (It may wait for the query norms of the prologue block, which has started
//     and itself waits for nobody.)  A block that gives up waiting raises a flag for its rows and
//     draws a ticket from the unit's give-up counter; the finisher draws the closing ticket, learns from it how
//     many blocks gave up before, and compacts their rows after its own (re-reading them).
//     A block that gives up later than that finds the closing ticket in the counter: the list is
//     there by then, so it fetches it and carries on by itself.  Every block exits whatever the
//     others do.  All sums run in a fixed order: the result does not depend on who arrives last.
//
// Waiting is safe for the same reason as in the three-launch form: a block only waits for blocks
// of its own unit, which have lower or neighbouring block numbers and were dispatched with it
// (the prologue blocks have the lowest numbers of all).
#include <algorithm>
#include <atomic>
#include <chrono>

#include "thk_prune_proto.h"

namespace thk {

// What a block knows when solo_index_list returns.
enum ListState { kGaveUp = 0, kHaveList = 1, kFinisher = 2 };
constexpr int kFinisherDone = 1 << 24;   // the finisher's closing ticket on the give-up counter
constexpr unsigned long long kNormValid = 1ull << 63;   // mark of a published query norm
constexpr int kSurePolls = 1 << 20;      // polls for what is in place or a running block is about to publish
constexpr int kAheadKB = 24;              // of the next round's rows that a waiting block fetches into the L2
constexpr int kInitPolls = 1 << 22;      // polls for the prologue's initialisation (a block that was dispatched earlier)

// ---- the prologue block --------------------------------------------------------------------
// lds: at least 5 * 128 doubles.
template <int DT, bool GRP>
__device__ __forceinline__ void solo_prologue(const PruneFusedArgs &a, int64_t u, double *lds) {
  const int tid = tid_here();
  double *hn = lds, *qn_l = lds + 4 * kD;
  // test hook (THK_PRUNE_PROLOGUE_DELAY_US): a late prologue makes the row blocks arrive on
  // counters that are not initialised yet, the path that otherwise needs an unlucky schedule
  for (int t = a.prologue_delay; t > 0; t -= 127) __builtin_amdgcn_s_sleep(127);
  if (tid < kWave) __hip_atomic_store(a.idx_pub + (size_t)u * kWave + tid, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int i = tid; i < a.NB; i += 256)
    __hip_atomic_store(a.undone + (size_t)u * a.NB + i, (unsigned char)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid == 0) {
    __hip_atomic_store(a.gaveup + u * kCtrStep<int>, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.arrived + u * kCtrStep<int>, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (tid < kD) pub_store_f64(a.qn + (size_t)u * kD + tid, 0.0);
  if constexpr (GRP)
    for (int i = tid; i < kMaxGroups * kD; i += 256) pub_store_f64(a.gpartial + (size_t)u * kMaxGroups * kD + i, 0.0);
  block_stores_done();
  // everything above has landed: the counters may now be found initialised
  if constexpr (GRP) {
    const int n_grp = (a.NB + a.GS - 1) / a.GS;
    if (tid < n_grp)
      __hip_atomic_store(a.tctr_g + ((size_t)u * kMaxGroups + tid) * kCtrStep<unsigned long long>, a.nonce << 16,
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (tid == 0) {
    __hip_atomic_store(a.tctr + u * kCtrStep<unsigned long long>, a.nonce << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // test hook (THK_PRUNE_NORM_DELAY_US): the unit's sums are complete before its norms are
  for (int t = a.norm_delay; t > 0; t -= 127) __builtin_amdgcn_s_sleep(127);
  block_query_norm<DT, 4>(a.q_obs, u, a.G, a.S_obs, qn_l, hn);
  __syncthreads();
  // the norms carry their own validity mark, the sign bit, which a sum of norms leaves free: a row
  // block may want them before they are there
  if (tid < kD)
    __hip_atomic_store((unsigned long long *)a.qn + (size_t)u * kD + tid, (unsigned long long)__double_as_longlong(qn_l[tid]) | kNormValid,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The unit's query norm of channel tid (threads < 128) from `w`, the word loaded earlier (behind a
// counter whose tag was there, i.e. after the prologue had cleared the words).  The prologue block is
// running then and waits for nobody, so the word comes; if the looks run out all the same the
// norm is NaN, and so is the score: no list is made of sums that lack their norms without a sign.
__device__ __forceinline__ double query_norm_of(const PruneFusedArgs &a, int64_t u, unsigned long long w) {
  if (tid_here() >= kD) return 0.0;
  const double *p = a.qn + (size_t)u * kD + tid_here();
  for (int n = 0; (w & kNormValid) == 0 && n < a.norm_polls; ++n) {
    __builtin_amdgcn_s_sleep(2);
    w = pub_load_bits(p);
  }
  return (w & kNormValid) != 0 ? __longlong_as_double((long long)(w & ~kNormValid)) : __builtin_nan("");
}
__device__ __forceinline__ unsigned long long query_norm_word(const PruneFusedArgs &a, int64_t u) {
  return tid_here() < kD ? pub_load_bits(a.qn + (size_t)u * kD + tid_here()) : 0ull;
}

// One arrival on a tagged counter: true in every thread of the block that makes the count `full`.
__device__ __forceinline__ bool arrive_tagged(unsigned long long *ctr, unsigned long long nonce, int full,
                                              int *s_flag) {
  if (tid_here() == 0) {
    unsigned long long old = atomicAdd(ctr, 1ull);
    if ((old >> 16) != nonce) {
      // earlier than the prologue's initialisation, whose store wipes what was just added
      for (int n = 0; n < kInitPolls; ++n) {
        if ((__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16) == nonce) break;
        __builtin_amdgcn_s_sleep(8);
      }
      old = atomicAdd(ctr, 1ull);
    }
    const bool last = (int)(old & 0xffffu) == full - 1;
    // nobody comes after the last arrival: leave a word without the tag behind
    if (last) __hip_atomic_store(ctr, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_flag = last;
  }
  __syncthreads();
  const bool last = *s_flag != 0;
  __syncthreads();   // everyone has read the flag before it is reused
  return last;
}

// One-level form: the published index list -> s_idx, polling at most `limit` times.  True in
// every thread if the whole list was there.
__device__ __forceinline__ bool read_list_words(const PruneFusedArgs &a, int64_t u, int16_t *s_idx, int *s_flag,
                                                int limit) {
  const int tid = tid_here();
  if (tid < kWave) {
    const uint32_t *p = a.idx_pub + (size_t)u * kWave + tid;
    uint32_t w = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int n = 0; __any((w & kPubValid) == 0) && n < limit; ++n) {
      for (int t = a.poll_ticks; t > 0; t -= 4) __builtin_amdgcn_s_sleep(4);
      if ((w & kPubValid) == 0) w = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const bool ok = __all((w & kPubValid) != 0);
    if (ok) {
      s_idx[2 * tid] = (int16_t)(w & 0x7fffu);
      s_idx[2 * tid + 1] = (int16_t)((w >> 16) & 0x7fffu);
    }
    if (tid == 0) *s_flag = ok;
  }
  __syncthreads();
  const bool ok = *s_flag != 0;
  __syncthreads();   // everyone has read the flag before it is reused
  return ok;
}

// Two-level form: the unit's column sums from its (at most 16) group vectors, added in group
// order (the first eight, the others, the two sums), polling at most `limit` times.  Two waves poll, thread c channel c of all groups,
// through a buffer resource that ends with the last group's vector, all loads in flight at once: a wave's loads return in order, and the
// other two may have rows ahead in flight (rows_ahead; with four waves polling behind them 96 units x 54784 rows took 417 us instead
// of 392).  True in every thread if all vectors were there; the sum is then valid in threads < 128.
__device__ __forceinline__ bool read_group_sums(const PruneFusedArgs &a, int64_t u, int *s_flag, int limit, double &kss) {
  const int tid = tid_here();
  const int n_grp = (a.NB + a.GS - 1) / a.GS;
  kss = 0.0;
  if (tid == 0) *s_flag = 1;
  __syncthreads();
  if (tid < kD) {
    constexpr int kRow = kD * (int)sizeof(double), kDeviceScope = 16;   // sc1, as pub_load_bits
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(a.gpartial + (size_t)u * kMaxGroups * kD), (short)0, n_grp * kRow, 0x00027000);
    auto look = [&](int j) {
      return __builtin_bit_cast(unsigned long long, __builtin_amdgcn_raw_buffer_load_b64(rsrc, tid * (int)sizeof(double) + j * kRow, 0, kDeviceScope));
    };
    // all groups in flight at once; a wave looks again at all of them while one is missing (registers are short: three tiles are
    // held beside these words)
    unsigned long long w[kMaxGroups];
    bool ok;
    for (int n = 0;; ++n) {
#pragma unroll
      for (int j = 0; j < kMaxGroups; ++j) w[j] = look(j);
      int there = 0;   // (what lies past the last group comes as 0)
#pragma unroll
      for (int j = 0; j < kMaxGroups; ++j) there += (int)((uint32_t)w[j] & 1u);
      ok = there == n_grp;
      if (__all(ok) || n >= limit) break;
      for (int t = a.poll_ticks; t > 0; t -= 4) __builtin_amdgcn_s_sleep(4);
      asm volatile("" ::: "memory");   // look again
    }
    double half[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < kMaxGroups; ++j) half[j / (kMaxGroups / 2)] += __longlong_as_double((long long)(w[j] & ~1ull));
    kss = half[0] + half[1];
    if (!ok) *s_flag = 0;      // any thread that ran out of polls
  }
  __syncthreads();
  const bool all_ok = *s_flag != 0;
  __syncthreads();           // the flag may be reused
  return all_ok;
}

// A row block's way from its column sums (`part`: of channel tid, threads < 128) to the unit's index
// list (s_idx).  item: u * NB + the block's number among the unit's row blocks.
// UN: partial sums of other blocks in flight per thread while they are merged.  ahead(w): called by blocks that have arrived and now wait, to
// put idle time to use with waves w .. 3.
template <int UN, bool GRP, class Ahead>
__device__ __forceinline__ int solo_index_list(const PruneFusedArgs &a, int64_t u, int64_t item, double part, double *s_part,
                                               float *s_sc, int16_t *s_idx, int *s_flag, Ahead &&ahead) {
  const int tid = tid_here();
  if (tid < kD) pub_store_f64(a.partial + (size_t)item * kD + tid, part);
  block_stores_done();

  const double *src = a.partial + (size_t)u * a.NB * kD;
  if constexpr (GRP) {
    // Two levels: the last block of a group of a.GS consecutive blocks merges the group's sums
    // into one vector and publishes it; EVERY block of the unit then reads the (at most 16)
    // group vectors, adds them in group order and makes the index list for itself -- the same
    // bits everywhere.  The block that publishes the unit's LAST vector is the finisher: every
    // publisher counts its group only after the vector has landed, so the finisher finds all of
    // them at its first look.  It also stores the caller's copy of scores and list.
    const int blk = (int)(item - u * a.NB);
    const int g = blk / a.GS;
    const int gsize = min(a.GS, a.NB - g * a.GS);
    const int n_grp = (a.NB + a.GS - 1) / a.GS;
    double *gp = a.gpartial + (size_t)u * kMaxGroups * kD;
    bool finisher = false;
    const bool group_last = arrive_tagged(a.tctr_g + ((size_t)u * kMaxGroups + g) * kCtrStep<unsigned long long>, a.nonce, gsize, s_flag);
    // from here on the prologue's work is visible: the query norms travel with whatever comes next
    const unsigned long long qn_w = query_norm_word(a, u);
    if (group_last) {
      const double gs = merge_partials_once<UN>(src + (size_t)g * a.GS * kD, gsize, s_part);
      if (tid < kD) pub_store_marked(gp + (size_t)g * kD + tid, gs);
      block_stores_done();
      finisher = arrive(a.arrived + u * kCtrStep<int>, n_grp, s_flag);
    } else {
      ahead(2);
    }
    double kss;
    if (!read_group_sums(a, u, s_flag, finisher ? kSurePolls : a.spin_limit, kss)) return kGaveUp;
    score_and_select(a, u, query_norm_of(a, u, qn_w), kss, s_sc, s_idx, finisher);
    return finisher ? kFinisher : kHaveList;
  }

  if (arrive_tagged(a.tctr + u * kCtrStep<unsigned long long>, a.nonce, a.NB, s_flag)) {
    const unsigned long long qn_w = query_norm_word(a, u);
    const double kss = merge_partials_once<UN>(src, a.NB, s_part);
    score_and_select(a, u, query_norm_of(a, u, qn_w), kss, s_sc, s_idx, true);
    if (tid < kWave) {
      const uint32_t lo = 2 * tid < a.T ? (uint16_t)s_idx[2 * tid] : 0u;
      const uint32_t hi = 2 * tid + 1 < a.T ? (uint16_t)s_idx[2 * tid + 1] : 0u;
      __hip_atomic_store(a.idx_pub + (size_t)u * kWave + tid, lo | (hi << 16) | kPubValid, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    return kFinisher;
  }
  // ---- wait (bounded) for the unit's index list; wave 0 polls
  ahead(1);
  return read_list_words(a, u, s_idx, s_flag, a.spin_limit) ? kHaveList : kGaveUp;
}

// A block whose wait ran out leaves its rows to the unit's finisher: it raises its flag, makes
// sure the flag has landed, and draws a ticket.  A ticket drawn after the finisher's closing one
// means that the finisher will not look again -- and that the list is in place: the block then
// fetches it after all (true) and goes on as usual.
template <bool GRP>
__device__ __forceinline__ bool hand_over_rows(const PruneFusedArgs &a, int64_t u, int64_t item, float *s_sc, int16_t *s_idx,
                                               int *s_flag) {
  const int tid = tid_here();
  if (tid == 0)
    __hip_atomic_store(a.undone + item, (unsigned char)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  block_stores_done();
  if (tid == 0) *s_flag = atomicAdd(a.gaveup + u * kCtrStep<int>, 1) >= kFinisherDone;
  __syncthreads();
  const bool late = *s_flag != 0;
  __syncthreads();
  if (!late) return false;
  if constexpr (GRP) {
    const unsigned long long qn_w = query_norm_word(a, u);
    double kss;
    read_group_sums(a, u, s_flag, kSurePolls, kss);
    score_and_select(a, u, query_norm_of(a, u, qn_w), kss, s_sc, s_idx, false);
  } else {
    read_list_words(a, u, s_idx, s_flag, kSurePolls);
  }
  return true;
}

// The finisher closes the unit BEFORE it compacts its own rows: it draws the closing ticket from
// the give-up counter, whose value is the number of blocks that gave up so far (their flags are
// in place: a block raises its flag, waits for the acknowledgement, and only then draws its
// ticket).  A block that gives up later finds the closing ticket, fetches the list -- published
// before the ticket was drawn; the late block polls for it all the same -- and carries on by
// itself.  (Drawing the ticket after the finisher's own rows instead, behind a wait for the
// acknowledgement of everything it had published, measured the same on every shape.)
__device__ __forceinline__ int close_unit(const PruneFusedArgs &a, int64_t u, int *s_flag) {
  if (tid_here() == 0) *s_flag = atomicAdd(a.gaveup + u * kCtrStep<int>, kFinisherDone);
  __syncthreads();
  const int n = *s_flag;
  __syncthreads();
  return n;
}

// ... and after its own rows it compacts the row blocks whose flags are raised (re-reading them
// from memory).  tab: the gather table of the unit.
template <int DT>
__device__ __forceinline__ void serve_gaveup(const PruneFusedArgs &a, int64_t u, const u32x4 *src,
                                             const FlatOut<DT> &dst, const int16_t *tab, u32x4 *tiles) {
  const unsigned char *flags = a.undone + (size_t)u * a.NB;
  for (int blk = 0; blk < a.NB; ++blk) {
    // block-uniform: every thread reads the same byte
    if (__hip_atomic_load(flags + blk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) continue;
    const int64_t s0 = (int64_t)blk * a.RB;
    const int64_t s1c = min(a.S_keep, s0 + a.RB);
    if (s0 < s1c) compact_rows<DT>(src, dst, s0, s1c, a.T, a.ld, tab, tiles);
  }
}

// The row blocks keep their rows (NTW tiles of 32 rows per wave, RB = 128 * NTW rows) on chip
// from the column sums until the index list arrives: the first NTW - NLT tiles of a wave in
// registers, the last NLT in the wave's LDS tiles -- exactly as k_prune_onepass does.
// GRP: units of more than 64 blocks, whose sums travel in two levels (kernels of their own: the registers of one form are not
// those of the other, and a short launch fetches less code).  LONG: more blocks than are resident at once.
template <int DT, int NTW, int NLT, bool GRP, bool LONG>
__global__ __launch_bounds__(256, Elem<DT>::EB == 4 ? 2 : (NTW - NLT) * 16 * Elem<DT>::EB <= 32 ? 4 : 3)
void k_prune_solo(PruneFusedArgs a) {
  using E = Elem<DT>;
  constexpr int VEC = E::VEC, CPR = kD / VEC, TR = kCompactTileRows, NLD = TR * CPR / kWave;
  constexpr int NRT = NTW - NLT;             // tiles per wave held in registers ...
  constexpr int kHeld = NRT * 16 * E::EB;    // ... and the registers they take
  extern __shared__ u32x4 smem[];
  int16_t *tab = (int16_t *)smem;            // 2 KiB
  u32x4 *tiles = smem + 128;                 // [4 waves][NLT] x [32][128] elements
  __shared__ double red[4][kD];
  __shared__ double s_part[kD];
  __shared__ float s_sc[kD];
  __shared__ int16_t s_idx[kD];
  __shared__ int s_flag;
  const int tid = tid_here(), lane = tid % kWave;
  // A launch of this kernel is over in ten to a hundred microseconds and runs most of its code
  // once, so what it executes is kept SHORT: instructions come from memory at about 45 ns per
  // 64 bytes.  The wave index is uniform (row counts and their branches are scalar), rows are
  // numbered in 32 bits (a unit held on chip has fewer than 2^19), every load takes the same
  // form and only a ragged tile pays for its raggedness.  8 units x 5003 rows: first load issued after 0.6
  // instead of 1.8 us.
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  // What the block needs in front of its first loads, asked for at once: an argument loaded where it is
  // first used is a trip of its own, and there were two.  Medians of 15 turns in alternation: 8 units
  // x 5003 rows 11.28 -> 11.13 us, 32 x 347 9.65 -> 9.50, fp32 8 x 2048 9.38 -> 9.31 (0.7 to 1.6 %, the same sign in every
  // turn; two runs of one side differ by up to 1.6 %); calls above 20 us do not change.
  asm volatile("" ::"s"(a.k), "s"(a.S), "s"(a.NB), "s"(a.U), "s"(a.stagger_blocks), "s"(a.stagger_units), "s"(a.stagger_ticks));
  if (blockIdx.x < (uint32_t)a.U) {
    solo_prologue<DT, GRP>(a, blockIdx.x, (double *)tiles);   // the tiles are free in a block without rows
    return;
  }
  const uint32_t item = blockIdx.x - (uint32_t)a.U;
  const uint32_t u = item / (uint32_t)a.NB;
  const int blk = (int)(item - u * (uint32_t)a.NB);
  const int S = (int)a.S;
  const int s0 = blk * (128 * NTW);          // a.RB == 128 * NTW
  const int s1 = min(S, s0 + 128 * NTW);
  const char *src = (const char *)a.k + (size_t)u * S * (kD * E::EB);
  u32x4 *wtile = tiles + (size_t)wave * NLT * Tile<DT>::CHUNKS;   // this wave's NLT tiles

  // tile n of this wave = rows s0 + (4 n + wave) * 32 .. + 32, nr of them inside [s0, hi)
  auto tile_row0 = [&](int n) { return s0 + (4 * n + wave) * TR; };
  auto tile_rows = [&](int n, int hi) { return max(0, min(TR, hi - tile_row0(n))); };

  // the graded start of the launch's first round (see k_prune_onepass)
  if (item < (uint32_t)a.stagger_blocks) {
    int ticks = (int)(u % (uint32_t)a.stagger_units) * a.stagger_ticks;
    for (; ticks >= 127; ticks -= 127) __builtin_amdgcn_s_sleep(127);
    for (; ticks >= 16; ticks -= 16) __builtin_amdgcn_s_sleep(16);
  }

  // ---- load: in a launch of one round every chunk of the block's rows is in flight at once ----
  // Blocks of a long launch load their tiles through buffer resources (request_tile), at most 8 KB of a wave in flight: all four tiles at
  // once only fill the queues that the blocks' exchange of sums has to pass as well (64 units x 26736 rows 150.6 -> 148.1 us,
  // 8 x 131072 83.6 -> 81.7; 16 KB no gain, 4 KB a loss).  A launch of one round wants all of it as early as it can: one
  // clamped byte offset per load, and ragged tiles are masked below (32 x 10000 rows 20.2 us, as above 20.7; 24 x 7629 19.4 / 20.0).
  constexpr bool kKeepOffsets = NTW * E::EB == 8;   // blocks of 128 KB
  u32x4 r[NTW][NLD];
  if constexpr (LONG) {
#pragma unroll
    for (int n = 0; n < NTW; ++n) request_tile<DT, 8>(r[n], src, tile_row0(n), tile_rows(n, s1), lane, n * NLD);
  } else {
    const uint32_t last = (uint32_t)S * CPR - 1;
#pragma unroll
    for (int n = 0; n < NTW; ++n)
#pragma unroll
      for (int j = 0; j < NLD; ++j) {
        const uint32_t c = (uint32_t)tile_row0(n) * CPR + (uint32_t)(j * kWave + lane);
        r[n][j] = ld_stream((const u32x4 *)(src + min(c, last) * 16u));
      }
  }
  if (a.ld != a.T)
#pragma unroll
    for (int n = 0; n < NLT; ++n) tile_clear_padding<DT>(wtile + (size_t)n * Tile<DT>::CHUNKS, lane);

  // ---- column sums of squares; the last NLT tiles then move to LDS -----------------------------
  double dacc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) dacc[v] = 0.0;
#pragma unroll
  for (int nn = 0; nn < NTW; ++nn) {
    const int n = (nn + NRT) % NTW;          // LDS-bound tiles first: their registers free up early
    if constexpr (!LONG) {
      const int nr = tile_rows(n, s1);
      if (__builtin_expect(nr < TR, 0)) {    // rows past the block's end count nothing
#pragma unroll
        for (int j = 0; j < NLD; ++j)
          if (j * kWave + lane >= nr * CPR) r[n][j] = u32x4{0u, 0u, 0u, 0u};
      }
    }
    float facc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) facc[v] = 0.f;
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
      float f[VEC];
      E::unpack(r[n][j], f);
#pragma unroll
      for (int v = 0; v < VEC; ++v) facc[v] = fmaf(f[v], f[v], facc[v]);
      if (n >= NRT) wtile[(size_t)(n - NRT) * Tile<DT>::CHUNKS + Tile<DT>::slot(j * kWave + lane)] = r[n][j];
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) dacc[v] += (double)facc[v];
  }
#pragma unroll
  for (int v = 0; v < VEC; ++v) dacc[v] = add_lane_groups<CPR>(dacc[v]);
  if (lane < CPR)
#pragma unroll
    for (int v = 0; v < VEC; ++v) red[wave][lane * VEC + v] = dacc[v];
  __syncthreads();
  const double part = tid < kD ? ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid] : 0.0;

  // What a block does between its arrival and the list is wait, 5 to 10 us, and the blocks of a round wait at about the same
  // time, while the memory idles.  In that time it fetches the first rows of the block that will take its place, one round of
  // resident blocks further on, without a hint against caching: workgroup i runs on XCD i % 8, a round is a multiple of 8, so the rows
  // are in that XCD's L2 when they are wanted.  24 KB: 96 blocks an XCD x 24 KB of 4 MB L2 (16: half of the gain, 48: less than 32, 96: a loss).  What
  // arrives is dropped into 1 KB of LDS that nobody reads.  Whole calls, without / with: 64 units x 26736 rows, T = 97, 147 -> 137 us, 80 x
  // 29502, T = 34, 146 -> 139, 56 x 15051 76.7 -> 73.5, 64 x 36965 171 -> 165, 8 x 131072 80.4 -> 77.
  [[maybe_unused]] auto rows_ahead = [&](int w0) {
    if constexpr (LONG) {
      __shared__ __attribute__((aligned(16))) u32x4 s_drop[kWave];
      const uint32_t next = item + (uint32_t)a.round_blocks;
      if (wave < w0 || next >= (uint32_t)a.U * (uint32_t)a.NB) return;
      const uint32_t un = next / (uint32_t)a.NB;
      const int per = kAheadKB / (4 - w0);
      const uint32_t last = (uint32_t)S * CPR - 1, c0 = (next - un * (uint32_t)a.NB) * (128 * NTW * CPR) + (uint32_t)((wave - w0) * per * kWave + lane);
      const char *srcn = (const char *)a.k + (size_t)un * S * (kD * E::EB);
#pragma unroll 4
      for (int i = 0; i < per; ++i)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(srcn + min(c0 + (uint32_t)(i * kWave), last) * 16u),
                                         (__attribute__((address_space(3))) void *)s_drop, 16, 0, 0);
    }
  };
  int st = solo_index_list<kHeld == 0 ? 24 : kHeld <= 32 ? 16 : 8, GRP>(a, u, item, part, s_part, s_sc, s_idx, &s_flag, rows_ahead);
  // (the rows ahead have landed before anything else happens to this block's LDS, whose end they must not outlive)
  if constexpr (LONG) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (st == kGaveUp) {
    if (!hand_over_rows<GRP>(a, u, item, s_sc, s_idx, &s_flag)) return;
    st = kHaveList;
  }
  const int n_gaveup = st == kFinisher ? close_unit(a, u, &s_flag) : 0;

  // ---- compaction: the LDS tiles first, then the register tiles through slot 0 ---------------
  const FlatOut<DT> dst((char *)a.kp + (size_t)u * a.kp_unit_rows * a.ld * E::EB);
  compact_build_tab<DT>(tab, s_idx, a.T, a.ld, dst.sh);
  __syncthreads();
  // (one or two tiles per wave: keeping the gathers' offsets costs more than it saves, 128 units x 430 rows 12.1 -> 12.3 us)
  [[maybe_unused]] Emit<DT> emit;
  if constexpr (kKeepOffsets) emit.init(tab, dst.sh, a.ld, lane);
  auto emit_tile = [&](const u32x4 *t, int r0, int nr) {
    if constexpr (kKeepOffsets) emit.tile(t, dst, r0, nr, a.ld, tab, lane);
    else compact_emit_tile<DT>(t, dst, r0, nr, a.ld, tab, lane);
  };
  const int s1c = min(s1, (int)a.S_keep);
#pragma unroll
  for (int n = NRT; n < NTW; ++n) {
    const int nr = tile_rows(n, s1c);
    if (nr > 0) emit_tile(wtile + (size_t)(n - NRT) * Tile<DT>::CHUNKS, tile_row0(n), nr);
  }
#pragma unroll
  for (int n = 0; n < NRT; ++n) {
    const int nr = tile_rows(n, s1c);
    if (nr > 0) {   // wave-uniform
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();       // the slot's previous tile has been read
#pragma unroll
      for (int j = 0; j < NLD; ++j) wtile[Tile<DT>::slot(j * kWave + lane)] = r[n][j];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      emit_tile(wtile, tile_row0(n), nr);
    }
  }
  if (n_gaveup > 0) {   // block-uniform
    __syncthreads();   // every wave is done with the tiles, which the re-read uses
    serve_gaveup<DT>(a, u, (const u32x4 *)src, dst, tab, tiles);
  }
}

// ---- host side --------------------------------------------------------------------------------
namespace {
// A 48-bit number, never 0, different for every call of the process and spread over the whole
// range, so that what an earlier call or other data left in a workspace does not look like it.
unsigned long long next_nonce48() {
  static std::atomic<unsigned long long> counter{
      (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull};
  unsigned long long z = counter.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z = (z ^ (z >> 31)) >> 16;
  return z != 0 ? z : 1;
}
int solo_group_size(int NB) { return NB > 64 ? (NB + kMaxGroups - 1) / kMaxGroups : 0; }
}  // namespace

size_t prune_solo_ws_bytes(int64_t U, int NB) {
  size_t b = (size_t)U * NB * kD * sizeof(double);                                   // partial
  if (solo_group_size(NB) > 0) {
    b += (size_t)U * kMaxGroups * kD * sizeof(double);                               // gpartial
    b += (size_t)U * kMaxGroups * kCtrBytes;                                         // tctr_g
  }
  b += (size_t)U * kD * sizeof(double);                                              // qn
  b += 3 * (size_t)U * kCtrBytes;                                                    // tctr, arrived, gaveup
  b = (b + 15) & ~(size_t)15;
  b += (size_t)U * kWave * sizeof(uint32_t);                                         // idx_pub
  b += ((size_t)U * NB + 15) & ~(size_t)15;                                          // undone
  return b;
}

hipError_t launch_prune_solo(int dtype, const void *q_obs, const void *k, float *score, int16_t *idx, void *kp,
                             void *ws, int64_t U, int64_t S, int64_t S_keep, int64_t kp_unit_rows, int G,
                             int S_obs, int T, int ld, int NB, int64_t RB, int hold, int spin_limit,
                             hipStream_t st) {
  clear_stale_hip_error();
  PruneFusedArgs a = {};
  const int eb = dtype == THK_BF16 ? 2 : 4;
  a.k = k; a.q_obs = q_obs; a.kp = kp; a.score = score; a.idx = idx;
  a.GS = solo_group_size(NB);
  char *w = (char *)ws;
  a.partial = (double *)w; w += (size_t)U * NB * kD * sizeof(double);
  if (a.GS > 0) {
    a.gpartial = (double *)w;            w += (size_t)U * kMaxGroups * kD * sizeof(double);
    a.tctr_g = (unsigned long long *)w;  w += (size_t)U * kMaxGroups * kCtrBytes;
  }
  a.qn = (double *)w;                w += (size_t)U * kD * sizeof(double);
  a.tctr = (unsigned long long *)w;  w += (size_t)U * kCtrBytes;
  a.arrived = (int *)w;              w += (size_t)U * kCtrBytes;
  a.gaveup = (int *)w;               w += (size_t)U * kCtrBytes;
  w = (char *)(((uintptr_t)w + 15) & ~(uintptr_t)15);
  a.idx_pub = (uint32_t *)w;         w += (size_t)U * kWave * sizeof(uint32_t);
  a.undone = (unsigned char *)w;
  a.nonce = next_nonce48();
  a.round_blocks = kCUs * (dtype == THK_BF16 ? 3 : 2);
  // at most 500 us, in 64-cycle ticks at about 2.4 GHz
  a.prologue_delay = (int32_t)(std::min(std::max(env_switches().prologue_delay_us, 0L), 500L) * 2400 / 64);
  a.norm_delay = (int32_t)(std::min(std::max(env_switches().norm_delay_us, 0L), 500L) * 2400 / 64);
  a.norm_polls = env_switches().norm_polls >= 0 ? (int32_t)std::min(env_switches().norm_polls, (long)kSurePolls) : kSurePolls;
  a.S = S; a.S_keep = S_keep; a.kp_unit_rows = kp_unit_rows; a.RB = RB; a.T = T; a.ld = ld; a.G = G;
  a.S_obs = S_obs; a.NB = NB; a.spin_limit = spin_limit;
  // Pause between two looks: 4 ticks while all blocks are resident at once (8 units x 5003 rows: a
  // quarter of a microsecond less from list to first store), 16 in longer launches, whose polls
  // would queue among the streams.  A look takes 0.25 us then instead of 0.53: twice as many keep the
  // time after which a block resigns (4096 looks: 2.1 ms).
  a.poll_ticks = 16;
  if (U * NB <= (int64_t)kCUs * (dtype == THK_BF16 ? 3 : 2)) {
    a.poll_ticks = 4;
    a.spin_limit = (int32_t)std::min<int64_t>(2 * (int64_t)spin_limit, 0x7fffffff);
  }
  a.stagger_blocks = 0; a.stagger_units = 1; a.stagger_ticks = 0;
  a.U = U;
  {
    // the graded start of the first round, as in the three-launch form
    const int64_t resident = (int64_t)kCUs * (dtype == THK_BF16 ? 3 : 2);
    const int64_t total = U * NB;
    const int64_t res_units = resident / NB;
    double ns = -1.0;
    if (env_switches().stagger_set) ns = env_switches().stagger_ns;
    else if (res_units >= 2 && total >= 2 * resident) ns = 0.6 * (double)S * kD * eb * 1.5 / 5.7e3;
    if (ns > 0.0 && res_units >= 2) {
      a.stagger_blocks = (int32_t)(res_units * NB);
      a.stagger_units = (int32_t)res_units;
      a.stagger_ticks = std::max((int32_t)(ns * 2.4 / 64.0), 1);   // 2.4 GHz, s_sleep counts 64-cycle ticks
    }
  }
  const bool grp = a.GS > 0, lng = U * NB > a.round_blocks;
  const void *fn = nullptr;
  auto pick = [&](const void *short1, const void *short2, const void *long1, const void *long2) {
    fn = lng ? (grp ? long2 : long1) : (grp ? short2 : short1);
  };
#define THK_SOLO(DT, NTW, GRP, LONG) (const void *)k_prune_solo<DT, NTW, 1, GRP, LONG>
  // (blocks of fewer rows than are held are taken for calls of one round only)
  if (dtype == THK_BF16) {
    switch (hold) {
      case 1: pick(THK_SOLO(THK_BF16, 1, false, false), THK_SOLO(THK_BF16, 1, true, false), THK_SOLO(THK_BF16, 1, false, false), THK_SOLO(THK_BF16, 1, true, false)); break;
      case 2: pick(THK_SOLO(THK_BF16, 2, false, false), THK_SOLO(THK_BF16, 2, true, false), THK_SOLO(THK_BF16, 2, false, false), THK_SOLO(THK_BF16, 2, true, false)); break;
      case 4: pick(THK_SOLO(THK_BF16, 4, false, false), THK_SOLO(THK_BF16, 4, true, false), THK_SOLO(THK_BF16, 4, false, true), THK_SOLO(THK_BF16, 4, true, true)); break;
    }
  } else {
    switch (hold) {
      case 1: pick(THK_SOLO(THK_F32, 1, false, false), THK_SOLO(THK_F32, 1, true, false), THK_SOLO(THK_F32, 1, false, false), THK_SOLO(THK_F32, 1, true, false)); break;
      case 2: pick(THK_SOLO(THK_F32, 2, false, false), THK_SOLO(THK_F32, 2, true, false), THK_SOLO(THK_F32, 2, false, true), THK_SOLO(THK_F32, 2, true, true)); break;
    }
  }
#undef THK_SOLO
  if (fn == nullptr || RB != 128 * hold || U * ((int64_t)NB + 1) > 2147483647LL) return hipErrorInvalidValue;
  const size_t lds = 2048 + 4 * compact_tile_bytes(eb);
  static DynLds set[2][5][2][2];
  hipError_t e = ensure_dyn_lds(fn, lds, set[dtype == THK_BF16 ? 1 : 0][hold][grp][lng]);
  if (e != hipSuccess) return e;
  void *kargs[] = {(void *)&a};
  e = launch_main_kernel(fn, dim3((unsigned)(U * (NB + 1))), dim3(256), kargs, lds, st);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace thk
