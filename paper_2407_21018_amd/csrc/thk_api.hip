// C ABI of libthk: argument checks, workspace carving, launch sizing.
// Everything here is host code; no entry point allocates or synchronises.
#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <mutex>

#include "thk_internal.h"

using namespace thk;

namespace thk {
namespace {
thread_local hipEvent_t g_prof_start = nullptr, g_prof_stop = nullptr;

std::atomic<const EnvSwitches *> g_env{nullptr};
std::mutex g_env_mu;

long env_long_raw(const char *name, long unset) {
  const char *e = getenv(name);
  return (e == nullptr || *e == 0) ? unset : atol(e);
}

// A fresh, immutable snapshot of the switches; earlier snapshots stay valid for threads that
// still hold them (reloading is a test hook: the few bytes per reload are never freed).
const EnvSwitches *read_env() {
  EnvSwitches *s = new EnvSwitches();
  const char *path = getenv("THK_PRUNE_PATH");
  s->prune_path = (path != nullptr) ? path[0] : 0;
  s->group_mib = env_long_raw("THK_PRUNE_GROUP_MIB", 0);
  s->block_rows = env_long_raw("THK_PRUNE_BLOCK_ROWS", 0);
  s->hold_rows = env_long_raw("THK_PRUNE_HOLD_ROWS", 0);
  s->max_blocks = env_long_raw("THK_PRUNE_MAX_BLOCKS", -1);
  s->spin_limit = env_long_raw("THK_PRUNE_SPIN_LIMIT", -1);
  const char *ns = getenv("THK_PRUNE_STAGGER_NS");
  s->stagger_set = ns != nullptr;
  s->stagger_ns = ns != nullptr ? atof(ns) : -1.0;
  const char *mf = getenv("THK_DECODE_MFMA");
  s->decode_mfma_off = mf != nullptr && mf[0] == '0';
  const char *pl = getenv("THK_PRUNE_LAUNCH");
  s->prune_launch = pl != nullptr ? pl[0] : 0;
  s->prologue_delay_us = env_long_raw("THK_PRUNE_PROLOGUE_DELAY_US", 0);
  s->norm_delay_us = env_long_raw("THK_PRUNE_NORM_DELAY_US", 0);
  s->norm_polls = env_long_raw("THK_PRUNE_NORM_POLLS", -1);
  const char *mk = getenv("THK_DECODE_MERGE");
  s->decode_merge = mk != nullptr ? mk[0] : 0;
  const char *vc = getenv("THK_VALUE_COMPACT");
  s->value_compact = vc != nullptr ? vc[0] : 0;
  return s;
}
}  // namespace

const EnvSwitches &env_switches() {
  const EnvSwitches *s = g_env.load(std::memory_order_acquire);
  if (s == nullptr) {
    std::lock_guard<std::mutex> lock(g_env_mu);
    s = g_env.load(std::memory_order_relaxed);
    if (s == nullptr) {
      s = read_env();
      g_env.store(s, std::memory_order_release);
    }
  }
  return *s;
}

hipError_t launch_main_kernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t st) {
  // the runtime reduces 2^32 work-items or more modulo 2^32 without an error
  if ((uint64_t)grid.x * block.x > 0xffffffffull) return hipErrorInvalidConfiguration;
  if (g_prof_start == nullptr || g_prof_stop == nullptr) return hipLaunchKernel(fn, grid, block, args, lds, st);
  const hipEvent_t e0 = g_prof_start, e1 = g_prof_stop;
  g_prof_start = g_prof_stop = nullptr;
  return hipExtLaunchKernel(fn, grid, block, args, lds, st, e0, e1, 0);
}
}  // namespace thk

namespace {

thread_local hipError_t g_last_hip = hipSuccess;   // the launch error behind the last THK_ERR_HIP
inline bool failed(hipError_t e) {
  if (e != hipSuccess) g_last_hip = e;
  return e != hipSuccess;
}

inline bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

// Compute units of the current device, looked up once per device: 256 on the MI355X the launch
// heuristics are fitted to, fewer on a partitioned one; 256 where no device answers (the planning
// functions are also called by hosts without a GPU).  Only the rule that decides whether a unit's
// row blocks can all be resident at once -- a matter of safety of the one-pass prune, whose
// blocks wait for each other -- uses it; the tuning constants stay those of the 256-unit chip.
int device_cus() {
  constexpr int kMaxDev = 64;
  static std::atomic<int> cache[kMaxDev];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) {
    (void)hipGetLastError();
    return kCUs;
  }
  int n = cache[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
      (void)hipGetLastError();
      n = kCUs;
    }
    cache[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}
inline int elem_bytes(int dtype) { return dtype == THK_BF16 ? 2 : 4; }
inline int64_t units_of(const thk_shape *s) { return (int64_t)s->L * s->B * s->N_kv; }
inline int ld_of(const thk_shape *s) { return s->ld_keep ? s->ld_keep : s->T; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// rows of the prunable segment that get compacted, and rows between units of K_pruned / V
inline int64_t keep_rows(const thk_shape *s) { return s->S - s->S_recent; }
inline int64_t cache_rows(const thk_shape *s, int64_t used) { return s->S_cap ? s->S_cap : used; }

constexpr int kMaxSplit = 4096;
constexpr int64_t kMaxGrid = 2147483647LL;

// Shape checks common to all entry points.
thk_status check_shape(const thk_shape *s, bool need_obs) {
  if (s == nullptr) return THK_ERR_NULL;
  if (s->L < 1 || s->B < 1 || s->N_q < 1 || s->N_kv < 1 || s->D < 1 || s->S < 1) return THK_ERR_SHAPE;
  if (s->N_q % s->N_kv != 0) return THK_ERR_SHAPE;
  if (s->T < 1 || s->T > s->D) return THK_ERR_SHAPE;
  // rows of K_pruned hold T kept channels and at most D elements in all (the compaction's gather
  // table and the decode kernels' staging are sized for rows of up to D elements)
  if (s->ld_keep != 0 && (s->ld_keep < s->T || s->ld_keep > s->D)) return THK_ERR_SHAPE;
  if (need_obs && (s->S_obs < 1 || (int64_t)s->S_obs > s->S)) return THK_ERR_SHAPE;
  if (s->n_split < 0 || s->n_split > kMaxSplit) return THK_ERR_SHAPE;
  if (s->S_recent < 0 || (int64_t)s->S_recent >= s->S) return THK_ERR_SHAPE;
  if (s->S_cap < 0) return THK_ERR_SHAPE;
  if (s->dtype != THK_F32 && s->dtype != THK_BF16) return THK_ERR_UNSUPPORTED;
  if (s->D != kD) return THK_ERR_UNSUPPORTED;
  if (s->S > (int64_t)1 << 40 || units_of(s) > kMaxGrid) return THK_ERR_SHAPE;
  return THK_OK;
}

// Split of the S axis for the column reduction: `rows` rows per piece.
struct Split { int n; int64_t rows; };

Split score_split(const thk_shape *s, int64_t units) {
  int n = s->n_split;
  if (n == 0) {
    // aim at ~8 blocks per compute unit over the call, pieces of >= 256 rows
    n = (int)ceil_div((int64_t)kCUs * 8, units);
    const int64_t cap = ceil_div(s->S, 256);
    if (n > cap) n = (int)cap;
    if (n > kMaxSplit) n = kMaxSplit;
    if (n < 1) n = 1;
  }
  int64_t rows = ceil_div(s->S, n);
  rows = ceil_div(rows, 16) * 16;
  return {n, rows};
}

int group_width(int G) { return G <= 2 ? G : 4; }   // head slots per block of the general decode kernel

// Query heads that share a block of the decode kernel the shape takes.
int decode_heads_per_block(const thk_shape *s) {
  DecodeArgs a = {};
  a.T = s->T; a.ldk = ld_of(s); a.N_q = s->N_q; a.N_kv = s->N_kv; a.dtype = s->dtype;
  return decode_mq_serves(a) ? decode_mq_heads(a) : group_width(s->N_q / s->N_kv);
}

// Head groups (blocks per split) of a call, and the bytes of its split records rounded up to
// the 8-byte boundary where the flag words (one per group and split) start.
int64_t decode_groups(const thk_shape *s) {
  return units_of(s) * ceil_div(s->N_q / s->N_kv, decode_heads_per_block(s));
}
size_t decode_records_bytes(const thk_shape *s, int n_split) {
  const size_t b = (size_t)s->L * s->B * s->N_q * n_split * (kD + 2) * sizeof(float);
  return (b + 7) & ~(size_t)7;
}

size_t decode_ws_bytes(const thk_shape *s, int n_split) {
  return decode_records_bytes(s, n_split) + (size_t)decode_groups(s) * n_split * sizeof(unsigned long long);
}

// A 64-bit number, never 0, different for every call of the process and spread over the whole
// range (what an earlier call or other data left in a workspace will not look like it).
unsigned long long next_nonce() {
  static std::atomic<unsigned long long> counter{
      (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull};
  unsigned long long z = counter.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z = z ^ (z >> 31);
  return z != 0 ? z : 1;
}

// The split records of a call are merged inside the launch (by the block that finishes last for
// a head group) where that saves more than it costs -- see decode_merge_in_launch below.
bool decode_merge_in_launch(const thk_shape *s, int n_split);
bool merges_in_launch(int hpb, int64_t blocks);

// The most pieces worth an estimate: more than eight blocks per compute unit never pay.
int64_t most_pieces(int64_t wgs, int64_t steps, int n0) {
  constexpr int64_t kMaxPieces = 128;
  return std::min({steps, kMaxPieces, std::max<int64_t>(n0, 8 * (int64_t)kCUs / wgs)});
}

// Blocks of the decode kernels that are resident on a compute unit.
int decode_resident(const thk_shape *s, int hpb) {
  const bool wide = ld_of(s) > 79;   // the staging class of long rows
  return s->dtype == THK_F32 ? (hpb == 4 || wide ? 2 : 3) : (hpb == 8 ? 3 : 4) - (wide ? 1 : 0);
}

// The first estimate: the number of pieces (no fewer than least, no more than top) with the least estimated time, if that
// is at least 9 % below the estimate for n0.  With k = steps of a piece (128 rows by four waves), R = resident blocks of a
// compute unit and L = blocks on the fullest one, in us:
//     sum over rounds of resident blocks of max(k t_step, l k t_stream), l = R, in the last round what is left,
//     +  t_block L  +  merge
// t_step: a step that waits for its own loads, 2.4, 2.7 where a block serves eight heads, 4.8 in fp32; t_stream: a compute
// unit's share of the memory rate, 0.036 per KB of a step's rows (full-width values); t_block: what a block costs whatever
// its length, 0.8, in fp32 3.4; merge: nothing for one piece, 3.5 up to two blocks of at most four heads per compute unit,
// else 4, 0.015 per piece and 0.2 per thousand records.
// Fitted to 570 random shapes, a third of them fp32, when calls above two blocks per compute unit merged in a launch of
// their own; with the merge of fp32 calls of one and two heads priced as it is now (merges_in_launch), 4 of 520 shapes take
// another count (0.92, 0.95, 1.00 and 1.08 of the time), so the fitted price stays.  Pieces are told apart by their
// steps: by their 64-row runs, pieces of half a step count as shorter ones (fp32, 52 units x 7 heads, 2304 rows: 9 pieces
// instead of 2, 53.1 -> 66.4 us; 40 shapes that differed took 1.06x).
int pieces_by_rounds(const thk_shape *s, int hpb, int64_t wgs, int64_t steps, int n0, int least, int64_t top) {
  const bool f32 = s->dtype == THK_F32;
  const int64_t heads = (int64_t)s->L * s->B * s->N_q;
  const int resident = decode_resident(s, hpb);
  const double t_step = f32 ? 4.8 : hpb == 8 ? 2.7 : 2.4, t_block = f32 ? 3.4 : 0.8;
  const double t_stream = 0.036 * 128 * (ld_of(s) + kD) * elem_bytes(s->dtype) / 1024.0;
  auto around = [&](int64_t n) {   // what the tiles do not pay for; grows with n
    const int64_t blocks = wgs * n;
    const bool in_launch = n <= kDecodeFuseMaxSplit && blocks <= 2 * kCUs && hpb <= 4;
    const double merge = n == 1 ? 0.0 : in_launch ? 3.5 : 4.0 + 0.015 * (double)n + 0.0002 * (double)(heads * n);
    return t_block * (double)ceil_div(blocks, kCUs) + merge;
  };
  auto cost = [&](int64_t n, int64_t k) {
    const int64_t per_cu = ceil_div(wgs * n, kCUs), rounds = ceil_div(per_cu, resident);
    auto round = [&](int64_t l) { return (double)k * std::max(t_step, (double)l * t_stream); };
    return (double)(rounds - 1) * round(resident) + round(per_cu - (rounds - 1) * resident) + around(n);
  };
  const double least_time = (double)wgs * (double)steps / kCUs * t_stream;   // all rows at the memory rate
  double best = 0.91 * cost(n0, ceil_div(ceil_div(s->S, n0), 128));
  int64_t n_best = n0, k_last = 0;
  for (int64_t i = least; i <= top; ++i) {
    const int64_t k = (steps + i - 1) / i;
    if (k == k_last) continue;   // the same pieces, some of them empty
    k_last = k;
    if (least_time + around(i) >= best) break;   // nor does any count from here on
    const double c = cost(i, k);
    if (c < best) { best = c; n_best = i; }
  }
  return (int)n_best;
}

// bf16 calls have a second estimate, and take the number of pieces with the least time by it if that is at least 6 % below
// its time for n0 and 2 % below that for the count of the first estimate, which they take otherwise: what both are wrong
// about by a few percent is left as the first has it.  (fp32 has the first one only: the second one fitted to fp32 made calls
// of over 600 MB up to 10 % slower.)  With k = steps of a piece (128 rows by
// four waves, b KB of rows each), R = blocks that are resident on a compute unit, in us:
//     sum over rounds of resident blocks  +  t_block * blocks on the fullest compute unit  +  merge  +  t0
// A round's compute units hold q blocks each and some of them one more.  They move their rows at the least of what the memory
// gives them (an equal share of 7.6 TB/s: 30 KB/us, more for the ones left over once the others are done), of what a compute
// unit takes (c1 KB/us with one block, c2 with several), and of what waiting for its own loads lets a block take (k t_step).
// t_block: what a block costs whatever its length; merge: nothing for one piece, m_in for a short one (cheap_merge), m_out + 0.01
// per piece + 0.2 per thousand records for others.  Rows whose pitch makes the kernels put words together (odd) and
// long ones that take the wide staging class (wide) slow t_step, c1 and c2 by a factor.  The width of
// the value rows is not known here (the workspace must not depend on it), so the estimate is the mean of those of 128
// and of 64 channels.
// Constants fitted per kernel to 1400 random bf16 shapes (1-8 heads per KV head, 1-1280 units, 256-131072 rows, a
// quarter with pruned values), each measured at up to 29 piece counts; over these and 330 others the count taken costs 1.7 %
// more than the best one on average (the first estimate alone: 3.7 %): 306 of 1728 bf16 shapes take 3 % and more less than with
// that, 11 more.  (Without the look at the first estimate's count 355 less and 52 more, some of them slower than they had
// been before this estimate: 8 units x 8 heads, T = 51, 71436 rows, pruned values, 94 pieces instead of 63, 39.4 -> 47.5 us; 56 x 5
// heads x 13325 rows, 12 instead of 9, 50.3 -> 55.4.)
// What it knows that a resident set of blocks (n0) misses: a few
// blocks more than a multiple of 256 cost a round of few (64 units x 32768 rows, 4 heads: 4 pieces 121 us, 5 151); pieces of one
// step that leave compute units idle (16 units x 1815 rows: 15 pieces instead of 8, 11.0 -> 9.5); that one
// block per compute unit saturates the memory and fewer, longer streams use it better.
struct DecodeCost { double t0, t_step, c1, c2, t_block, m_in, m_out, odd, wide; };
const DecodeCost &decode_cost(int hpb) {
  static constexpr DecodeCost h1 = {3.45, 1.0, 56.3, 44.7, 0.59, 2.04, 3.69, 1.05, 1.20}, h2 = {3.89, 1.12, 43.5, 44.3, 0.82, 2.33, 3.39, 1.18, 1.19},
                              h4 = {3.69, 1.17, 38.8, 39.0, 0.50, 2.35, 3.59, 1.22, 1.0}, h8 = {3.9, 1.57, 30.5, 38.3, 0.98, 3.04, 3.82, 1.15, 1.13};
  return hpb == 1 ? h1 : hpb == 2 ? h2 : hpb == 4 ? h4 : h8;
}
int decode_pieces(const thk_shape *s, int hpb, int64_t wgs, int64_t steps, int n0, int least) {
  constexpr double kRate = 7600.0;   // KB per us
  // more pieces only while the records fit the scratch array of thk_decode_attn_static, which takes
  // every call that n0 pieces fit
  const int64_t heads = (int64_t)s->L * s->B * s->N_q;
  const int64_t fit = (int64_t)THK_STATIC_SCRATCH_BYTES / ((kD + 2) * 4 + 8) / heads;
  if (n0 > 1 && n0 > fit) return n0;
  const int64_t top = std::min(most_pieces(wgs, steps, n0), std::max<int64_t>(fit, 1));
  const int n1 = pieces_by_rounds(s, hpb, wgs, steps, n0, least, top);
  if (s->dtype == THK_F32) return n1;
  if (n0 >= 8) least = std::max(least, 4);
  const bool wide = ld_of(s) > 79;
  const int resident = decode_resident(s, hpb);
  const DecodeCost &c = decode_cost(hpb);
  const bool odd = ld_of(s) % (hpb <= 2 ? 2 : 4) != 0;
  const double slow = (odd ? c.odd : 1.0) * (wide ? c.wide : 1.0);
  const double t_step = c.t_step * slow;
  // A call plans this before it can launch, over up to 113 counts: nothing is divided that can be multiplied, and the search
  // ends where all rows at the memory rate and what a count adds to them reach the best time found.  Host time of
  // thk_default_split, plain formula / so: 8 units x 8 heads x 131072 rows 1980 / 110 ns, 64 x 4 x 32768 1060 / 80, 8 x 4 x
  // 1000 170 / 155.
  // Value rows of one width.  us per step: a block at the memory rate (t_one) and one on every compute unit (t_mem), a
  // block at the rate of a compute unit that it has alone (t1) or shares (t2), a whole round (t_round).
  struct Width {
    double t_one, t_mem, t1, t2, t_round;
    int resident;
  };
  static constexpr double inv[] = {0.0, 1.0, 1.0 / 2, 1.0 / 3, 1.0 / 4, 1.0 / 5};
  auto round = [&](const Width &w, int q, int r) {   // us per step: q blocks on every compute unit, one more on r of them
    double t = 0.0;
    if (q > 0) t += std::max({q * w.t_mem, q * (q == 1 ? w.t1 : w.t2), t_step});
    if (r > 0) t += std::max({r * w.t_one, q == 0 ? w.t1 : w.t2, t_step * inv[q + 1]});
    return std::max(t, t_step);
  };
  auto width = [&](int channels, int resident) {
    const double b = 128.0 * 2 * (ld_of(s) + channels) / 1024.0;
    Width w{b / kRate, b * (kCUs / kRate), b * slow / c.c1, b * slow / c.c2, 0.0, resident};
    w.t_round = round(w, resident, 0);
    return w;
  };
  const Width w_full = width(kD, resident), w_half = width(kD / 2, resident);
  // A merge of up to 16 pieces costs m_in, inside the launch or, for eight heads, in a launch whose blocks are one wave each; with
  // two blocks per compute unit and more the launch is priced.  (With eight heads priced at m_out, as it is or at 2.6 or 3.0, 4 % of 3000
  // random shapes take another count and those 118 to 127 are 1.2 to 1.3 % longer on average, 67 to 69 of them by 2 % and more, up to
  // 16; 32 to 39 are shorter: 256 units x 8 heads x 1071 rows 1 piece 21.0 us, 2 23.9; 24 x 8 heads x 6975 10 16.2, 19 17.1.)
  auto cheap_merge = [&](int64_t n, int64_t blocks) { return n <= kDecodeFuseMaxSplit && (merges_in_launch(hpb, blocks) || (hpb == 8 && blocks < 2 * (int64_t)kCUs)); };
  auto around = [&](int64_t n) {   // what the tiles do not pay for; grows with n
    const int64_t blocks = wgs * n;
    const double t = c.t0 + c.t_block * (double)ceil_div(blocks, kCUs);
    if (n == 1) return t;
    return t + (cheap_merge(n, blocks) ? c.m_in : c.m_out + 0.01 * (double)n + 0.0002 * (double)(heads * n));
  };
  // (for rows of unknown value width)
  auto estimate = [&](int64_t i, const Width &wide_rows, const Width &narrow_rows) {
    const int64_t rows = (ceil_div(s->S, i) + 63) & ~(int64_t)63, n = ceil_div(s->S, rows), blocks = wgs * n, per_cu = blocks / kCUs;
    const int r = (int)(blocks % kCUs);
    const double fixed = around(n);
    auto time = [&](const Width &w) {
      const int64_t full = per_cu / w.resident;
      const int q = (int)(per_cu - full * w.resident);
      double t = (double)full * w.t_round;
      if (q + r > 0) t += round(w, q, r);
      return fixed + (double)((rows + 127) / 128) * t;
    };
    return time(wide_rows) * time(narrow_rows);
  };
  const double least_full = (double)wgs * (double)steps * w_full.t_one, least_half = (double)wgs * (double)steps * w_half.t_one;
  double best = 0.94 * 0.94 * estimate(n0, w_full, w_half);
  int64_t n_best = n0, k_last = 0;
  for (int64_t i = least; i <= top; ++i) {
    const int64_t k = (steps + i - 1) / i;
    if (k == k_last) continue;   // the same pieces, some of them empty
    k_last = k;
    const int64_t n = ceil_div(steps, k);   // pieces of k steps: at least this many
    const double fixed = around(n);
    if ((least_full + fixed) * (least_half + fixed) >= best) break;
    const double e = estimate(i, w_full, w_half);
    if (e < best) { best = e; n_best = i; }
  }
  if (n_best == n1) return n1;
  // (between the two counts, blocks of eight heads count as two to a compute unit with pruned value rows, whose wide staging
  // class has two, and with key rows of odd pitch, where a third one does not help)
  const Width c_full = hpb == 8 && odd ? width(kD, 2) : w_full, c_half = hpb == 8 ? width(kD / 2, 2) : w_half;
  return estimate(n_best, c_full, c_half) < 0.98 * 0.98 * estimate(n1, c_full, c_half) ? (int)n_best : n1;
}

// Calls so short that a block per 64 rows leaves no compute unit with two take such pieces (0: another call).  Two of
// a block's waves have a tile of pruned rows each and the other two are free for the tail's, which a wave with rows of its own
// takes 1 to 2 us after those.  us per call without a tail, with 38 rows, with the append in front, pieces of whole steps / these:
// 8 units x 4 heads x 743 rows 7.5 8.3 10.2 / 7.4 7.4 9.0, 16 x 7 heads x 1020 9.0 10.3 12.2 / 8.1 8.2 10.1, fp32 8 x 2 heads x
// 614 9.1 10.9 12.6 / 8.7 8.8 10.5, 8 x 2 heads x 1581 9.2 10.8 12.6 / 8.5 8.7 10.7, 40 x 4 heads x 227 9.9 13.0 14.6 / 9.3 9.6 11.5.
// With a tail, blocks of eight heads and fp32 ones of the narrow staging class go on up to 1.75 blocks per compute unit (24 x 8 heads x
// 779 10.5 / 9.3, 8 x 7 heads x 2989 11.1 / 9.4, fp32 16 x 4 heads x 1227 12.5 / 11.6, 8 x 2779 12.3 / 9.7); bf16 blocks of four heads do not gain
// (32 x 785 8.7 / 9.1, 24 x 694 8.3 / 8.1), wide fp32 ones lose (24 x 4 heads x 936, T = 100 15.2 / 20.8), nor does a call without a
// tail gain (8 x 4 heads x 2910 7.5 / 8.2). In bf16
//   * not up to 256 rows, below which one block without a merge is shorter (16 x 4 heads x 182 6.2 7.4 9.0 / 7.1 7.1 8.8);
//   * blocks of one or two heads not above 16 pieces, whose merge is a second launch: with an append in front the host
//     takes longer to issue the three than the GPU to run them (8 units x 2 heads x 1191 rows 7.5 8.1 9.9 / 7.2 6.9 10.2).  Blocks of four heads
//     do go on: their calls of 1025 to 2048 rows of eight units, 4096 of four and fewer, merged in the launch with whole steps and gain more
//     (8 x 4 heads x 1188 7.8 8.5 / 7.3 7.3, x 2048 7.4 8.3 / 6.9 7.2, 4 x 4 x 3000 8.1 8.4 / 6.9 7.2), so the host decides with the append in
//     front: it issues the three in 9.0 us in most processes and in 10.9 in others (three and two of five, medians), which is what they
//     take then: 8 x 4 heads x 1188 9.7 / 9.1 or 10.9, 4 x 4 x 3000 9.9 / 9.1 or 10.9, 1 x 4 x 1188 9.4 / 9.0 or 10.7, 1 x 4 x 1500 8.8 / 9.0 or
//     10.7, fp32 1 x 1 head x 1300 10.2 / 8.9 or 10.8;
//   * calls of at most 16 pieces that have no tail, and blocks of at most four heads: their merge, inside the launch, grows by what the
//     shorter pieces save (8 x 4 heads x 947 7.2 / 7.6, 16 x 391 6.3 / 6.5).  A count is planned and reported as if there was a tail.
// One case is kept for what it reports and not for its time: up to 512 rows of eight units, and in bf16 blocks of one head of eight units, have the
// counts that thk_default_split gave before there were these pieces (4 of 512 rows, 8 of 1024), which its tests state.  They would gain as their
// neighbours do (with the append in front, as it is / these: 8 units x 4 heads x 450 rows 9.9 / 8.7, x 2 heads 12.7 / 9.0, 8 heads 11.8 / 11.5,
// one head x 512 9.6 / 8.1, x 743 11.5 / 8.3, fp32 8 x 1 head x 384 13.6 / 9.6; without a tail 7.1 / 7.0, 9.8 / 7.3, 8.2 / 8.0, 6.6 / 5.8, 8.8 / 6.6,
// 10.1 / 7.7).
int pieces_of_half_steps(const thk_shape *s, int hpb, int64_t wgs, bool tail) {
  const int64_t n = ceil_div(s->S, 64), heads = (int64_t)s->L * s->B * s->N_q;
  const bool eight = units_of(s) <= 8;
  const bool more = tail && (s->dtype == THK_F32 ? ld_of(s) <= 79 : hpb == 8);
  const int64_t most = more ? kCUs * 7 / 4 : kCUs;
  if (wgs * n > most || s->S <= (eight ? 512 : s->dtype == THK_BF16 ? 256 : 128)) return 0;
  if (s->dtype == THK_BF16) {
    if (hpb <= 2 && (n > kDecodeFuseMaxSplit || (hpb == 1 && eight))) return 0;
    if (hpb <= 4 && n <= kDecodeFuseMaxSplit && !tail) return 0;
  }
  return n * heads <= (int64_t)THK_STATIC_SCRATCH_BYTES / ((kD + 2) * 4 + 8) ? (int)n : 0;
}

// ws_bytes: what the caller's workspace holds.  The estimate's count goes up and down with S, so a
// workspace asked for at a sequence's final length can hold fewer pieces than a shorter length
// would take; a call then takes the pieces that fit, down to an eighth of the count n0 that the estimate
// starts from, and to two.  n0 never falls with S, the estimate takes a quarter of it or more in pieces of at least 127 rows, of
// which cutting into whole 64-row runs leaves more than half; pieces of 64 rows only raise a count and lose none to the cut:
// the workspace of the final length serves every shorter one.  Less than that is refused.  One piece,
// which needs no workspace, is taken only where n0 is 1 and by calls of at least 128 blocks per piece
// under 4096 rows (beyond, the estimate wants it of calls of over 500 blocks, to save 2-4 %): those
// are served with any workspace.
Split decode_split(const thk_shape *s, size_t ws_bytes = SIZE_MAX, bool tail = true) {
  int n = s->n_split;
  const int G = s->N_q / s->N_kv;
  const int64_t wgs = units_of(s) * ceil_div(G, decode_heads_per_block(s));
  if (n == 0) {
    // About one resident set of blocks over the call (4 per compute unit, 3 where a block
    // serves eight heads), a power of two pieces per unit.  The four waves of a block take 128 rows
    // per step; a piece has at least two steps, or one while the launch stays within one block per
    // compute unit (a started step counts: 8 units x 1000 rows take 8 pieces, not the 4 of at least
    // 128 whole rows: 11.4 -> 9.0 us; 64 units x 2000 rows 8 instead of 4: 18.0 -> 16.0 us); more than
    // 64 pieces (the merge grows with n) only where even that leaves compute units idle.  Short sequences
    // take one block per unit: below these lengths the second launch (the merge) costs more
    // than the split saves.  Big calls still get two pieces per unit so that the last blocks
    // to finish are short.
    const int hpb = decode_heads_per_block(s);
    const int per_cu = hpb == 8 ? 3 : 4;
    const int64_t one_block_rows = (hpb >= 4 ? 320 : 768) * 2 / elem_bytes(s->dtype);   // bf16 rows; half as many fp32 rows
    const int64_t steps = ceil_div(s->S, 128);
    n = 1;
    while (s->S > one_block_rows && n < 128) {
      const int64_t blocks = (int64_t)n * 2 * wgs;
      if (blocks > (int64_t)kCUs * per_cu || (n >= 64 && blocks > kCUs)) break;
      if ((int64_t)n * 2 * (blocks <= kCUs ? 1 : 2) > steps) break;
      n *= 2;
    }
    if (n == 1 && s->S >= 2048) n = 2;
    const int n0 = n;
    const bool one = n0 == 1 || (wgs >= kCUs / 2 && s->S < 4096);
    if (s->S > one_block_rows || units_of(s) > 8) n = decode_pieces(s, hpb, wgs, steps, n0, one ? 1 : std::max(2, n0 / 4));
    n = std::max(n, pieces_of_half_steps(s, hpb, wgs, tail));
    const int64_t fit = (int64_t)std::min<size_t>(ws_bytes / decode_ws_bytes(s, 1), (size_t)n);
    if (fit < n && fit >= (one ? 0 : std::max(2, n0 / 8))) n = std::max((int)fit, 1);
  }
  int64_t rows = ceil_div(s->S, n);
  rows = ceil_div(rows, 64) * 64;
  if (s->n_split == 0) n = (int)ceil_div(s->S, rows);   // drop empty pieces
  return {n, rows};
}

// Calls of at most 16 pieces merge their split records inside the launch: the block that finishes last for a
// head group does it, and the second launch goes away.  The hand-off is three memory round trips
// at the end of the kernel; a second launch costs the GPU as much and its dispatch and the host 2.5 us, which is what counts where
// a call takes the GPU about as long as the host.  Merged by the kernel / inside, us per call, and with the append in front:
// one head, 8 units x 571 rows 5.9 8.5 / 6.3 7.9, 40 x 1226 8.9 10.5 / 8.6 10.3; two, 24 x 6140 16.7 17.9 / 16.2 17.9; four,
// 8 x 881 7.1 10.9 / 7.5 8.9, 40 x 2629 (440 blocks) 13.8 15.4 / 13.9 15.6, before the kernel was made shorter 96 x 5971 (768) 38.5 / 39.8,
// 128 x 12777 (1024) 108.1 / 110.4.  A block of eight heads exchanges eight records and is better off with the kernel:
// 16 x 1929 9.9 11.7 / 10.3 12.3, 16 x 3207 11.8 13.6 / 12.3 14.2, 40 x 433 10.1 11.8 / 10.6 12.4, 40 x 5340 21.3 22.6 / 21.4 23.0.
// Hence: up to two heads per block always, four up to two blocks per compute unit, eight never.
// THK_DECODE_MERGE = kernel | fused overrides (fused only within the 16 pieces and the four heads).
bool merges_in_launch(int hpb, int64_t blocks) {
  return hpb <= 2 || (hpb == 4 && blocks <= 2 * (int64_t)kCUs);
}
bool decode_merge_in_launch(const thk_shape *s, int n_split) {
  if (n_split < 2 || n_split > kDecodeFuseMaxSplit) return false;
  const int hpb = decode_heads_per_block(s);
  const char sw = env_switches().decode_merge;
  if (hpb > 4 || sw == 'k') return false;
  return sw == 'f' || merges_in_launch(hpb, decode_groups(s) * n_split);
}

// Units per group in the staged form of thk_prune (three launches per group).
// Small groups would let the compaction re-read K from the memory-side cache,
// but measured launch overheads outweigh that; the default keeps groups large.
int64_t prune_group_units(const thk_shape *s) {
  size_t budget = (size_t)1024 << 20;
  if (env_switches().group_mib > 0) budget = (size_t)env_switches().group_mib << 20;
  const size_t per_unit = (size_t)s->S * kD * elem_bytes(s->dtype);
  int64_t g = (int64_t)(budget / per_unit);
  if (g < 1) g = 1;
  const int64_t U = units_of(s);
  return g > U ? U : g;
}

// ---- one-launch prune: eligibility and blocking -------------------------------
struct FusedPlan;
bool value_compact_in_bursts(const thk_shape *s, const FusedPlan &fp);

struct FusedPlan { bool ok; int NB; int64_t RB; int hold; };

// The one-launch forms of thk_prune.  Blocks take 512 bf16 / 256 fp32 rows each (measured best on
// MI355X; fewer for small calls) and the blocks of a unit wait for each other; a unit may have
// as many as are resident at once (768 bf16 / 512 fp32; above 64 their sums travel in two
// levels), longer sequences go through the staged path instead.
FusedPlan fused_plan(const thk_shape *s) {
  FusedPlan p{false, 0, 0, 0};
  const EnvSwitches &env = env_switches();
  const char path = env.prune_path;
  if (path == 's') return p;   // "staged": the three-kernel path
  if (s->S_cap != 0 && s->S_cap < keep_rows(s)) return p;
  int64_t rb = env.block_rows;
  if (rb <= 0) {
    // the default block size: 128 KB of rows, the most a block can hold on chip (512 bf16 rows,
    // 256 fp32 rows); small calls take the smallest held size (down to 128 rows) that keeps the
    // launch within two blocks per compute unit, i.e. within one round of resident blocks:
    // a launch that spills into a second round pays the whole load -> list -> store chain twice
    // (32 units of 4096 bf16 rows: 23 us with 512 blocks of 256 rows, 36 us with 1024 of 128)
    const int64_t rb_max = env.hold_rows > 0 ? env.hold_rows : (s->dtype == THK_BF16 ? 512 : 256);
    auto blocks = [&](int64_t r) { return units_of(s) * ceil_div(s->S, r); };
    rb = rb_max;
    while (rb > 128 && (blocks(rb / 2) <= (int64_t)kCUs * 2 || blocks(rb / 2) == blocks(rb))) rb /= 2;
  }
  if (rb < 32) rb = 32;
  rb = ceil_div(rb, 32) * 32;
  // blocks of 128, 256 or 512 rows (fp32: 128 or 256) keep their rows on chip between the
  // column sums and the compaction; other sizes, or THK_PRUNE_PATH=reread, read them twice
  const bool reread = path == 'r';
  if (!reread && (rb == 128 || rb == 256 || (rb == 512 && s->dtype == THK_BF16))) p.hold = (int)(rb / 128);
  const int64_t nb = ceil_div(s->S, rb);
  // the blocks of a unit wait for each other, so all of them must be resident at once; 256 where
  // the rows are read twice (the second read wants the unit's rows still in the memory-side cache)
  // (LDS decides: 2 KB + four tiles + 7 KB per block, i.e. three bf16 blocks or two fp32 blocks
  // per compute unit)
  const long fit = p.hold == 0 ? 256L : (s->dtype == THK_BF16 ? 3L : 2L) * std::min(device_cus(), kCUs);
  const bool forced = path == 'f' || path == 'r';   // regardless of the env limit
  if (nb > (forced || env.max_blocks < 0 ? fit : std::min(fit, env.max_blocks))) return p;
  p.RB = rb;
  p.NB = (int)nb;
  p.ok = units_of(s) * p.NB <= kMaxGrid;
  return p;
}

// Calls whose rows are held on chip and whose blocks make at most two rounds of resident blocks
// (three for units of more than 64 blocks) run as ONE launch (thk_prune_solo.hip): the two extra
// launches of the other form and the gaps around them are 7-30 % of such a call (fp32, 8 units
// x 2048 rows: 17.8 -> 12.8 us; 128 units x 4096 bf16 rows: 58.1 -> 51.8 us; 8 units x 131072
// rows: 97 -> 88-90 us).  From about four rounds on the single launch is no better (4 x 128
// units x 4096 rows: 161 against 161 us) and then worse (32 x 128 units: 1151-1282 against
// 1141-1154 us; 1280 units x 16384 rows: 1379-1497 against 1287-1306 us), so longer launches keep
// the three-launch form.  THK_PRUNE_LAUNCH = solo | classic overrides.
bool prune_single_launch(const thk_shape *s, const FusedPlan &fp) {
  if (!fp.ok || fp.hold == 0) return false;
  if (units_of(s) * ((int64_t)fp.NB + 1) > kMaxGrid) return false;
  const char sw = env_switches().prune_launch;
  if (sw == 'c') return false;
  if (sw == 's') return true;
  const int64_t resident = (int64_t)kCUs * (s->dtype == THK_BF16 ? 3 : 2);
  return units_of(s) * fp.NB <= (fp.NB > 64 ? 3 : 2) * resident;
}

// thk_prune_value compacts V through the one-pass prune kernels (index list given) where a call
// is long enough for the grouping of stores to pay: rows held on chip and at least 16 rounds of
// resident blocks.  Measured against the plain compaction kernel, whole thk_prune_value calls:
// units of 4096 bf16 rows +5 % at 2.7 rounds, +1 % at 5, -2 % at 11, -2.5 % at 16, -4.4 % at 32,
// -5 % at 43; units of 32768 rows +2 % at 5, +1 % at 11, -1.6 % at 21.
// With the values that the score leaves in the memory-side cache (prunes of two query tiles and more) the line lies where
// it did: 50 calls, one and two tiles +2 to +3 % at 4 to 6 rounds, 0 at 10 to 13, -2 to -3.4 % at 16 to 20, -4.5 % from 22 on;
// four and eight tiles 0 to +6 % below 8, +-1 % at 15 to 19, -2 to +1 % at 22 to 28.
// THK_VALUE_COMPACT = flat | burst overrides (burst only where the rows can be held).
bool value_compact_in_bursts(const thk_shape *s, const FusedPlan &fp) {
  if (!fp.ok || fp.hold == 0) return false;
  const char sw = env_switches().value_compact;
  if (sw == 'f') return false;
  if (sw == 'b') return true;
  const int64_t resident = (int64_t)kCUs * (s->dtype == THK_BF16 ? 3 : 2);
  return units_of(s) * (int64_t)fp.NB >= 16 * resident;
}

// Split of the S axis for the value score: pieces are whole 128-row chunks, few enough that the merge kernel's weight table (at
// most 256 pieces) fits.  The count starts from one resident set of blocks (two per compute unit: 74 KB of LDS each) in pieces of at
// least 512 rows (fp32: 128) and is the estimate's where that is surely better (value_pieces).
Split value_cut(const thk_shape *s, int n) {
  int64_t rows = ceil_div(s->S, n);
  rows = ceil_div(rows, 128) * 128;
  return {(int)ceil_div(s->S, rows), rows};   // empty pieces dropped
}
// The number of pieces (no fewer than least) with the least estimated time of a value prune, if that is at least 4 % below the
// estimate for n0.  In us, chunk = 128 rows, R = blocks resident on a compute unit, l of them on the fullest one:
//     launches and copy  +  the longer of  all rows at the memory rate  and  the sum over rounds of R blocks of
//     t0 + chunks of a piece * max(t_own, l t_shared)  +  records (t_rec each, 1.4 where the merge has more than eight)
// t_own: a chunk of a block by itself; t_shared: what each resident block adds.  Fitted per kernel (32-row query tiles a block
// carries; fp32 blocks of two are left out) to 160 random bf16 and 110 fp32 shapes at up to ten piece counts each, within 4.4 %; the count taken costs 0.9 and
// 1.0 % more than the best one on average, n0 5.9 and 7.6 %.  The margin is no larger than the fit's error, so what decides is the trial: 110
// random value prunes of other shapes, with all that changed beside the counts, bf16 of one, two, more query tiles 1.15, 1.13, 1.10 times as
// fast, fp32 of one or four tiles a block 1.43, of two (not planned here) 1.05; the least 0.995 and 0.998.  Host time of a plan
// (thk_prune_value makes two) 0.0-0.2 us before, 0.1-0.3 and up to 0.7 (131072 rows) with it.  What it knows that n0 does not: short calls are as long as a piece, and
// 128-row pieces use idle compute units (16 units x 311 rows 18.8 -> 16.0 us, 8 x 8 heads x 897 29.8 -> 26.8); the records of
// many query tiles (16 units x 8 heads x 7007 rows 14 pieces 64.0, 8 53.6); fp32 blocks of one wave are four to a compute
// unit (24 units x 17810 rows 20 pieces 214, 70 178).
int value_pieces(const thk_shape *s, int nqt, int QT, int n0, int least) {
  struct Cost { double base, copy, t0, t_own, t_shared, rate, t_rec, t_piece; int resident; };
  static constexpr Cost b1 = {12.7, 4.52, 2.27, 1.59, 1.59, 7.46, 0.0039, 0.164, 2}, b2 = {12.7, 4.52, 3.50, 2.03, 1.48, 6.85, 0.0039, 0.164, 2},
                        b4 = {12.7, 4.52, 6.02, 2.43, 2.43, 5.90, 0.0039, 0.164, 1}, f1 = {14.5, 5.38, 0.57, 17.2, 5.14, 5.48, 0.0003, 0.149, 4},
                        f4 = {14.5, 5.38, 5.72, 15.5, 15.8, 6.0, 0.0003, 0.149, 2};
  const bool f32 = s->dtype == THK_F32;
  const Cost &c = f32 ? (QT == 1 ? f1 : f4) : (QT == 1 ? b1 : QT == 2 ? b2 : b4);
  const int64_t U = units_of(s);
  const double mb = (double)U * (double)s->S * 2.0 * kD * elem_bytes(s->dtype) / 1e6;   // keys and values
  const double base = c.base + 0.75 * mb / c.copy, stream = mb / c.rate;
  const int wide = !f32 && QT == 4 ? value_wide_tiles(s->N_q / s->N_kv, s->S_obs) : 0;
  auto cost = [&](int64_t n, int64_t chunks) {
    int tiles = QT;
    if (wide == 8 && U * n * ceil_div(nqt, 8) >= kCUs) tiles = 8;   // (as the launch chooses)
    const double twice = tiles == 8 ? 2.0 : 1.0;
    const int64_t blocks = U * n * ceil_div(nqt, tiles), per_cu = ceil_div(blocks, kCUs), full = per_cu / c.resident, rest = per_cu % c.resident;
    auto round = [&](int64_t l) { return c.t0 + (double)chunks * twice * std::max(c.t_own, (double)l * c.t_shared); };
    const double t = (double)full * round(c.resident) + (rest > 0 ? round(rest) : 0.0);
    return base + std::max(t, stream) + (double)(U * n * ceil_div(nqt, tiles) * tiles) * c.t_rec + (n > 8 ? 1.4 : 0.0) + (double)n * c.t_piece;
  };
  // a last piece of less than 48 rows is not worth a block
  const int64_t top = std::min<int64_t>({256, std::max<int64_t>((s->S + 80) / 128, 1), 6 * (int64_t)n0});
  double best = 0.96 * cost(n0, ceil_div(ceil_div(s->S, n0), 128));
  int64_t n_best = n0, k_last = 0;
  for (int64_t i = least; i <= top; ++i) {
    const int64_t k = ceil_div(ceil_div(s->S, i), 128);
    if (k == k_last) continue;   // the same pieces, some of them empty
    k_last = k;
    const int64_t n = ceil_div(s->S, 128 * k);   // what i whole-chunk pieces leave
    if (n < least) continue;
    const double t = cost(n, k);
    if (t < best) { best = t; n_best = i; }
  }
  return (int)n_best;
}

// least (may be null): the fewest pieces a call with a smaller workspace is cut into
// instead, never more for a shorter S than what any longer one reports (as in decode_split; half of
// the count that is independent of rounds, for the runs are whole 128-row chunks).
Split value_split(const thk_shape *s, int *least = nullptr) {
  const int G = s->N_q / s->N_kv;
  const int QT = value_attn_qt(G, s->S_obs);
  const int nqt = (G * s->S_obs + 31) / 32;
  const int64_t blocks1 = units_of(s) * ceil_div(nqt, QT);
  int n = s->n_split, floor_n = kMaxSplit;
  if (n == 0) {
    n = (int)ceil_div((int64_t)kCUs * 2, blocks1);
    // fp32: pieces down to one 128-row chunk (a block is one to four wavefronts bound by the
    // fp32 matrix rate: 8 units x 2048 rows 110 -> 47 us, 64 x 1024 rows 112 -> 48 us); bf16
    // blocks take four chunks side by side and lose 10-15 % with smaller pieces
    const int64_t cap = ceil_div(s->S, s->dtype == THK_F32 ? 128 : 512);
    if (n > cap) n = (int)cap;
    if (n < 1) n = 1;
    floor_n = n;
    if (s->dtype == THK_BF16 && QT == 4) {
      // The 8-wave kernel for grouped heads, one block per compute unit: the pieces that give the
      // shortest sum of rounds x (rows of a piece + 256 for its start, end and share of the merge).
      // 64 units x 32768 rows: 4 pieces instead of 8, 278 -> 268 us; 96 units: 5 instead of 3
      // (288 blocks would be a round of 256 and one of 32).
      const int64_t tiles = value_wide_tiles(G, s->S_obs);
      const int64_t b1 = units_of(s) * ceil_div(nqt, tiles);
      int64_t best = INT64_MAX;
      for (int64_t c = 1; c <= std::min<int64_t>(cap, std::max<int64_t>(ceil_div((int64_t)kCUs * 2, b1), 1)); ++c) {
        const int64_t piece = ceil_div(ceil_div(s->S, c), 128) * 128;
        const int64_t cost = ceil_div(b1 * c, kCUs) * (piece + 256);
        if (cost < best) { best = cost; n = (int)c; }
      }
      floor_n = (int)std::min<int64_t>(cap, std::max<int64_t>(kCUs / b1, 1));   // the most that one round holds
    }
    floor_n = std::max(std::min(floor_n, 256) / 2, 1);
    // (not fp32 blocks of two query tiles, whose times the estimate does not know well: 24 units x 7 heads x 7674 rows, S_obs = 8
    // 126 us with the count there is, 150 with the estimate's)
    if (s->dtype == THK_BF16 || QT != 2) n = value_pieces(s, nqt, QT, std::min(n, 256), floor_n);
  }
  if (n > 256) n = 256;
  if (least != nullptr) *least = floor_n;
  return value_cut(s, n);
}

// The value score's pieces in a workspace of ws_bytes, of which a call of n pieces takes bytes(s, n).
Split value_split_in(const thk_shape *s, size_t ws_bytes, size_t (*bytes)(const thk_shape *, int)) {
  int least = 1;
  const Split want = value_split(s, &least);
  for (int n = want.n; n >= least; --n) {
    const Split sp = value_cut(s, n);
    if (bytes(s, sp.n) <= ws_bytes) return sp;
  }
  return want;
}

size_t value_ws_bytes(const thk_shape *s, int n) {
  return value_part_bytes(units_of(s), s->N_q / s->N_kv, s->S_obs, n);
}
size_t prune_value_ws_bytes(const thk_shape *s, int n) {
  size_t a = value_ws_bytes(s, n);
  const FusedPlan fp = fused_plan(s);
  if (value_compact_in_bursts(s, fp)) a = std::max(a, prune_fused_ws_bytes(units_of(s), fp.NB));
  return ((a + 15) & ~(size_t)15) + (size_t)units_of(s) * kD * sizeof(float);
}

size_t score_ws_bytes(const thk_shape *s, int64_t units) {
  return (size_t)units * score_split(s, units).n * kD * sizeof(double);
}

}  // namespace

extern "C" {

int32_t thk_version(void) { return 200; }

void thk_reload_env(void) {
  std::lock_guard<std::mutex> lock(g_env_mu);
  g_env.store(read_env(), std::memory_order_release);
}

void thk_profile_next(void *ev_start, void *ev_stop) {
  g_prof_start = (ev_start != nullptr && ev_stop != nullptr) ? (hipEvent_t)ev_start : nullptr;
  g_prof_stop = (ev_start != nullptr && ev_stop != nullptr) ? (hipEvent_t)ev_stop : nullptr;
}

thk_status thk_bench_stream(int32_t mode, const void *src, void *dst, int64_t n_blocks, int32_t w, void *stream) {
  if (mode < THK_STREAM_READ || mode > THK_STREAM_WRITE) return THK_ERR_SHAPE;
  if (n_blocks < 1 || n_blocks > 2147483647LL || w < 0 || w > 32) return THK_ERR_SHAPE;
  if (mode != THK_STREAM_READ && w < 1) return THK_ERR_SHAPE;
  if (mode != THK_STREAM_WRITE && src == nullptr) return THK_ERR_NULL;
  if (mode != THK_STREAM_READ && dst == nullptr) return THK_ERR_NULL;
  if (!aligned16(src) || !aligned16(dst)) return THK_ERR_ALIGN;
  clear_stale_hip_error();
  return failed(launch_bench_stream(mode, src, dst, n_blocks, w, (hipStream_t)stream)) ? THK_ERR_HIP : THK_OK;
}

const char *thk_last_hip_error(void) { return hipGetErrorString(g_last_hip); }

const char *thk_status_string(thk_status st) {
  switch (st) {
    case THK_OK: return "ok";
    case THK_ERR_NULL: return "null pointer";
    case THK_ERR_SHAPE: return "invalid shape";
    case THK_ERR_UNSUPPORTED: return "unsupported configuration";
    case THK_ERR_ALIGN: return "pointer not 16-byte aligned";
    case THK_ERR_WORKSPACE: return "workspace missing or too small";
    case THK_ERR_HIP: return "HIP launch failed";
    case THK_ERR_SCRATCH: return "the call needs more scratch than the library's static buffer holds";
  }
  return "unknown status";
}

int32_t thk_keep_count(int32_t D, double lambda) {
  if (D < 1 || !(lambda >= 0.0) || !(lambda < 1.0)) return -1;
  return (int32_t)floor((1.0 - lambda) * (double)D + 1e-9);
}

int32_t thk_default_split(const thk_shape *s, int32_t op) {
  if (check_shape(s, false) != THK_OK) return 0;
  thk_shape t = *s;
  t.n_split = 0;
  if (op == THK_OP_DECODE) return decode_split(&t).n;
  if (op == THK_OP_SCORE) return score_split(&t, units_of(&t)).n;
  if (op == THK_OP_PRUNE) return score_split(&t, prune_group_units(&t)).n;
  if (op == THK_OP_SCORE_VALUE || op == THK_OP_PRUNE_VALUE) return (t.S_obs >= 1 && t.S_obs <= t.S) ? value_split(&t).n : 0;
  return 0;
}

int32_t thk_prune_is_fused(const thk_shape *s) {
  if (check_shape(s, true) != THK_OK) return 0;
  const FusedPlan fp = fused_plan(s);
  return !fp.ok ? 0 : fp.hold != 0 ? 2 : 1;
}

int32_t thk_prune_launches(const thk_shape *s) {
  if (check_shape(s, true) != THK_OK) return 0;
  const FusedPlan fp = fused_plan(s);
  if (!fp.ok) return 3 * (int32_t)ceil_div(units_of(s), prune_group_units(s));
  return prune_single_launch(s, fp) ? 1 : 3;
}

int32_t thk_decode_on_matrix_cores(const thk_shape *s, int32_t T_v, int32_t ld_v) {
  if (check_shape(s, false) != THK_OK) return 0;
  if (T_v < 0 || T_v > kD || (T_v > 0 && (ld_v < T_v || ld_v > kD))) return 0;
  DecodeArgs a = {};
  a.T = s->T; a.ldk = ld_of(s); a.N_q = s->N_q; a.N_kv = s->N_kv; a.dtype = s->dtype;
  a.T_v = T_v; a.ld_v = T_v > 0 ? ld_v : 0;
  return decode_mq_serves(a) ? 1 : 0;
}

size_t thk_workspace_bytes(const thk_shape *s, int32_t op) {
  if (check_shape(s, false) != THK_OK) return 0;
  switch (op) {
    case THK_OP_SCORE:
      return score_ws_bytes(s, units_of(s));
    case THK_OP_DECODE: {
      const Split sp = decode_split(s);
      return sp.n == 1 ? 16 : decode_ws_bytes(s, sp.n);
    }
    case THK_OP_SCORE_VALUE:
      if (s->S_obs < 1 || (int64_t)s->S_obs > s->S) return 0;
      return value_ws_bytes(s, value_split(s).n);
    case THK_OP_PRUNE_VALUE:
      if (s->S_obs < 1 || (int64_t)s->S_obs > s->S) return 0;
      return prune_value_ws_bytes(s, value_split(s).n);
    case THK_OP_PRUNE: {
      // a score array for the whole call + the larger of the two paths' scratch
      const FusedPlan fp = fused_plan(s);
      size_t a = score_ws_bytes(s, prune_group_units(s));
      if (fp.ok) {
        const size_t b = std::max(prune_fused_ws_bytes(units_of(s), fp.NB), prune_solo_ws_bytes(units_of(s), fp.NB));
        if (b > a) a = b;
      }
      return ((a + 15) & ~(size_t)15) + (size_t)units_of(s) * kD * sizeof(float);
    }
  }
  return 0;
}

static thk_status score_common(const thk_shape *s, int mode, const void *q_obs, const void *k,
                               float *score, void *ws, size_t ws_bytes, void *stream) {
  thk_status st = check_shape(s, mode == 0);
  if (st != THK_OK) return st;
  if (k == nullptr || score == nullptr || (mode == 0 && q_obs == nullptr)) return THK_ERR_NULL;
  if (!aligned16(k) || !aligned16(score) || (mode == 0 && !aligned16(q_obs))) return THK_ERR_ALIGN;
  const int64_t U = units_of(s);
  const Split sp = score_split(s, U);
  if (U * sp.n > kMaxGrid) return THK_ERR_SHAPE;
  if (ws == nullptr || !aligned16(ws) || ws_bytes < score_ws_bytes(s, U)) return THK_ERR_WORKSPACE;
  hipStream_t hs = (hipStream_t)stream;
  if (failed(launch_colsum(s->dtype, k, (double *)ws, U, s->S, sp.n, sp.rows, mode == 1 ? 1 : 2, hs)))
    return THK_ERR_HIP;
  if (failed(launch_finalize(s->dtype, mode, (const double *)ws, q_obs, score, nullptr, U, s->N_q / s->N_kv,
                      s->S_obs, sp.n, s->T, hs)))
    return THK_ERR_HIP;
  return THK_OK;
}

thk_status thk_score(const thk_shape *s, const void *q_obs, const void *k, float *score, void *ws,
                     size_t ws_bytes, void *stream) {
  return score_common(s, 0, q_obs, k, score, ws, ws_bytes, stream);
}

thk_status thk_score_magnitude(const thk_shape *s, const void *k, int32_t p, float *score,
                               void *ws, size_t ws_bytes, void *stream) {
  if (p != 1 && p != 2) return s == nullptr ? THK_ERR_NULL : THK_ERR_SHAPE;
  return score_common(s, p == 1 ? 1 : 2, nullptr, k, score, ws, ws_bytes, stream);
}

thk_status thk_select_topk(const thk_shape *s, const float *score, int16_t *idx, void *stream) {
  thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  if (score == nullptr || idx == nullptr) return THK_ERR_NULL;
  if (!aligned16(score) || !aligned16(idx)) return THK_ERR_ALIGN;
  if (failed(launch_select(score, idx, units_of(s), s->T, (hipStream_t)stream))) return THK_ERR_HIP;
  return THK_OK;
}

thk_status thk_compact_keys(const thk_shape *s, const void *k, const int16_t *idx, void *k_pruned,
                            void *stream) {
  thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  if (k == nullptr || idx == nullptr || k_pruned == nullptr) return THK_ERR_NULL;
  if (!aligned16(k) || !aligned16(idx) || !aligned16(k_pruned)) return THK_ERR_ALIGN;
  if (units_of(s) * ceil_div(s->S, 512) > kMaxGrid) return THK_ERR_SHAPE;
  if (s->S_cap != 0 && s->S_cap < keep_rows(s)) return THK_ERR_SHAPE;
  if (failed(launch_compact(s->dtype, k, s->S, 0, idx, k_pruned, cache_rows(s, keep_rows(s)), 0, units_of(s),
                            keep_rows(s), s->T, ld_of(s), (hipStream_t)stream)))
    return THK_ERR_HIP;
  return THK_OK;
}

thk_status thk_compact_rows(const thk_shape *s, const void *src, int64_t src_unit_rows, int64_t src_row0,
                            const int16_t *idx, void *k_pruned, int64_t dst_row0, int64_t n_rows,
                            void *stream) {
  thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  if (src == nullptr || idx == nullptr || k_pruned == nullptr) return THK_ERR_NULL;
  const int64_t dst_unit_rows = cache_rows(s, s->S);
  if (n_rows < 0 || src_row0 < 0 || dst_row0 < 0 || src_row0 + n_rows > src_unit_rows ||
      dst_row0 + n_rows > dst_unit_rows)
    return THK_ERR_SHAPE;
  if (!aligned16(src) || !aligned16(idx) || !aligned16(k_pruned)) return THK_ERR_ALIGN;
  if (units_of(s) * ceil_div(n_rows > 0 ? n_rows : 1, 512) > kMaxGrid) return THK_ERR_SHAPE;
  if (failed(launch_compact(s->dtype, src, src_unit_rows, src_row0, idx, k_pruned, dst_unit_rows, dst_row0,
                     units_of(s), n_rows, s->T, ld_of(s), (hipStream_t)stream)))
    return THK_ERR_HIP;
  return THK_OK;
}

thk_status thk_copy_rows(const thk_shape *s, const void *src, int64_t src_unit_rows, int64_t src_row0,
                         void *dst, int64_t dst_unit_rows, int64_t dst_row0, int64_t n_rows,
                         void *stream) {
  thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  if (src == nullptr || dst == nullptr) return THK_ERR_NULL;
  if (n_rows < 0 || src_row0 < 0 || dst_row0 < 0 || src_row0 + n_rows > src_unit_rows ||
      dst_row0 + n_rows > dst_unit_rows)
    return THK_ERR_SHAPE;
  if (src == dst && (dst_unit_rows != src_unit_rows || dst_row0 > src_row0)) return THK_ERR_SHAPE;
  if (!aligned16(src) || !aligned16(dst)) return THK_ERR_ALIGN;
  if (failed(launch_copy_rows(s->dtype, src, src_unit_rows, src_row0, dst, dst_unit_rows, dst_row0, units_of(s),
                       n_rows, (hipStream_t)stream)))
    return THK_ERR_HIP;
  return THK_OK;
}

thk_status thk_cache_append(const thk_shape *s, const void *k_new, const void *v_new, void *k_tail,
                            void *v, int32_t s_tail, int32_t s_tail_cap, void *stream) {
  thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  if (k_new == nullptr || v_new == nullptr || k_tail == nullptr || v == nullptr) return THK_ERR_NULL;
  if (s_tail < 0 || s_tail >= s_tail_cap) return THK_ERR_SHAPE;
  if (s->S + s_tail >= cache_rows(s, s->S)) return THK_ERR_SHAPE;   // the value cache is full
  if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_tail) || !aligned16(v)) return THK_ERR_ALIGN;
  if (failed(launch_tail_append(s->dtype, k_new, v_new, k_tail, v, units_of(s), s_tail_cap, s_tail,
                         cache_rows(s, s->S), s->S + s_tail, (hipStream_t)stream)))
    return THK_ERR_HIP;
  return THK_OK;
}

thk_status thk_tail_flush(const thk_shape *s, const int16_t *idx, void *k_pruned, void *k_tail, void *v,
                          void *v_tail, int32_t s_tail, int32_t s_tail_cap, int32_t n_flush,
                          void *stream) {
  thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  if (idx == nullptr || k_pruned == nullptr || k_tail == nullptr) return THK_ERR_NULL;
  if ((v == nullptr) != (v_tail == nullptr)) return THK_ERR_NULL;
  if (s_tail < 0 || s_tail > s_tail_cap || n_flush < 0 || n_flush > s_tail) return THK_ERR_SHAPE;
  const int64_t unit_rows = cache_rows(s, s->S);
  if (s->S + n_flush > unit_rows) return THK_ERR_SHAPE;   // no room left in the pruned cache
  if (!aligned16(idx) || !aligned16(k_pruned) || !aligned16(k_tail) ||
      (v != nullptr && (!aligned16(v) || !aligned16(v_tail))))
    return THK_ERR_ALIGN;
  hipStream_t hs = (hipStream_t)stream;
  const int64_t U = units_of(s);
  if (v != nullptr && n_flush == s_tail) {   // nothing stays behind to be shifted
    hipError_t e = hipSuccess;
    if (launch_flush(s->dtype, k_tail, v_tail, s_tail_cap, idx, k_pruned, v, unit_rows, s->S, U, n_flush, s->T,
                     ld_of(s), hs, &e))
      return failed(e) ? THK_ERR_HIP : THK_OK;
  }
  if (failed(launch_compact(s->dtype, k_tail, s_tail_cap, 0, idx, k_pruned, unit_rows, s->S, U, n_flush, s->T,
                     ld_of(s), hs)))
    return THK_ERR_HIP;
  if (failed(launch_copy_rows(s->dtype, k_tail, s_tail_cap, n_flush, k_tail, s_tail_cap, 0, U, s_tail - n_flush,
                       hs)))
    return THK_ERR_HIP;
  if (v != nullptr) {
    if (failed(launch_copy_rows(s->dtype, v_tail, s_tail_cap, 0, v, unit_rows, s->S, U, n_flush, hs)))
      return THK_ERR_HIP;
    if (failed(launch_copy_rows(s->dtype, v_tail, s_tail_cap, n_flush, v_tail, s_tail_cap, 0, U, s_tail - n_flush,
                         hs)))
      return THK_ERR_HIP;
  }
  return THK_OK;
}

thk_status thk_prune(const thk_shape *s, const void *q_obs, const void *k, float *score,
                     int16_t *idx, void *k_pruned, void *ws, size_t ws_bytes, void *stream) {
  thk_status st = check_shape(s, true);
  if (st != THK_OK) return st;
  if (q_obs == nullptr || k == nullptr || idx == nullptr || k_pruned == nullptr) return THK_ERR_NULL;
  if (!aligned16(q_obs) || !aligned16(k) || !aligned16(idx) || !aligned16(k_pruned) ||
      (score != nullptr && !aligned16(score)))
    return THK_ERR_ALIGN;
  if (ws == nullptr || !aligned16(ws) || ws_bytes < thk_workspace_bytes(s, THK_OP_PRUNE)) return THK_ERR_WORKSPACE;
  const int64_t U = units_of(s);
  const int G = s->N_q / s->N_kv;
  hipStream_t hs = (hipStream_t)stream;
  const size_t score_off = thk_workspace_bytes(s, THK_OP_PRUNE) - (size_t)U * kD * sizeof(float);
  float *sc = score != nullptr ? score : (float *)((char *)ws + score_off);
  const FusedPlan fp = fused_plan(s);
  if (fp.ok) {
    const int spin = env_switches().spin_limit >= 0 ? (int)env_switches().spin_limit : 4096;
    if (prune_single_launch(s, fp)) {
      if (failed(launch_prune_solo(s->dtype, q_obs, k, sc, idx, k_pruned, ws, U, s->S, keep_rows(s),
                                   cache_rows(s, keep_rows(s)), G, s->S_obs, s->T, ld_of(s), fp.NB, fp.RB, fp.hold,
                                   spin, hs)))
        return THK_ERR_HIP;
      return THK_OK;
    }
    if (failed(launch_prune_fused(s->dtype, q_obs, k, sc, idx, k_pruned, ws, U, s->S, keep_rows(s),
                                  cache_rows(s, keep_rows(s)), G, s->S_obs, s->T, ld_of(s), fp.NB, fp.RB, fp.hold,
                                  spin < 0 ? 0 : spin, 0, hs)))
      return THK_ERR_HIP;
    return THK_OK;
  }
  // staged path: score -> select -> compact per group of units
  if (s->S_cap != 0 && s->S_cap < keep_rows(s)) return THK_ERR_SHAPE;
  const int64_t kp_rows = cache_rows(s, keep_rows(s));
  const int64_t gu = prune_group_units(s);
  const Split sp = score_split(s, gu);
  if (gu * sp.n > kMaxGrid || gu * ceil_div(s->S, 512) > kMaxGrid) return THK_ERR_SHAPE;
  double *partial = (double *)ws;
  const int eb = elem_bytes(s->dtype);
  const int ld = ld_of(s);
  for (int64_t u0 = 0; u0 < U; u0 += gu) {
    const int64_t nu = (U - u0 < gu) ? U - u0 : gu;
    const char *kg = (const char *)k + (size_t)u0 * s->S * kD * eb;
    if (failed(launch_colsum(s->dtype, kg, partial, nu, s->S, sp.n, sp.rows, 2, hs))) return THK_ERR_HIP;
    // unit u reads query heads u * G .. u * G + G - 1, so a group starting at u0 starts u0 * G heads in
    const char *qg = (const char *)q_obs + (size_t)u0 * G * s->S_obs * kD * eb;
    if (failed(launch_finalize(s->dtype, 0, partial, qg, sc + (size_t)u0 * kD, idx + (size_t)u0 * s->T, nu, G,
                        s->S_obs, sp.n, s->T, hs)))
      return THK_ERR_HIP;
    const hipError_t ce = launch_compact(s->dtype, kg, s->S, 0, idx + (size_t)u0 * s->T,
                                         (char *)k_pruned + (size_t)u0 * kp_rows * ld * eb, kp_rows, 0, nu,
                                         keep_rows(s), s->T, ld, hs);
    if (failed(ce)) return THK_ERR_HIP;
  }
  return THK_OK;
}

// thk_score_value for a checked shape; with idx the selection too (the kernel that finishes a unit's score selects)
static thk_status score_value_common(const thk_shape *s, const void *q_obs, const void *k, const void *v,
                                     int32_t causal, float *score_v, int16_t *idx, void *ws, size_t ws_bytes,
                                     size_t (*bytes)(const thk_shape *, int), void *stream) {
  if (q_obs == nullptr || k == nullptr || v == nullptr || score_v == nullptr) return THK_ERR_NULL;
  if (!aligned16(q_obs) || !aligned16(k) || !aligned16(v) || !aligned16(score_v)) return THK_ERR_ALIGN;
  if (causal != 0 && causal != 1) return THK_ERR_SHAPE;
  const int G = s->N_q / s->N_kv;
  if ((int64_t)G * s->S_obs > 32 * 1024) return THK_ERR_SHAPE;
  const Split sp = value_split_in(s, ws_bytes, bytes);
  const int QT = value_attn_qt(G, s->S_obs);
  // (the launch rounds the pieces up to a multiple of 8 where a unit has several query blocks)
  const int64_t grid = (units_of(s) * sp.n + 7) * ceil_div((G * s->S_obs + 31) / 32, QT);
  if (grid > kMaxGrid) return THK_ERR_SHAPE;
  if (ws == nullptr || !aligned16(ws) || ws_bytes < bytes(s, sp.n)) return THK_ERR_WORKSPACE;
  if (failed(launch_value_score(s->dtype, q_obs, k, v, (float *)ws, score_v, idx, s->T, units_of(s), s->S, G, s->S_obs,
                         causal, sp.n, sp.rows, next_nonce(), (hipStream_t)stream)))
    return THK_ERR_HIP;
  return THK_OK;
}

thk_status thk_score_value(const thk_shape *s, const void *q_obs, const void *k, const void *v,
                           int32_t causal, float *score_v, void *ws, size_t ws_bytes, void *stream) {
  const thk_status st = check_shape(s, true);
  if (st != THK_OK) return st;
  return score_value_common(s, q_obs, k, v, causal, score_v, nullptr, ws, ws_bytes, value_ws_bytes, stream);
}

thk_status thk_prune_value(const thk_shape *s, const void *q_obs, const void *k, const void *v,
                           int32_t causal, float *score_v, int16_t *idx_v, void *v_pruned, void *ws,
                           size_t ws_bytes, void *stream) {
  thk_status st = check_shape(s, true);
  if (st != THK_OK) return st;
  if (idx_v == nullptr || v_pruned == nullptr) return THK_ERR_NULL;
  if (!aligned16(idx_v) || !aligned16(v_pruned) || (score_v != nullptr && !aligned16(score_v)))
    return THK_ERR_ALIGN;
  const size_t need = prune_value_ws_bytes(s, value_split_in(s, ws_bytes, prune_value_ws_bytes).n);
  if (ws == nullptr || !aligned16(ws) || ws_bytes < need) return THK_ERR_WORKSPACE;
  // the score array sits behind the value score's own scratch unless the caller wants it
  float *sc = score_v != nullptr ? score_v : (float *)((char *)ws + need - (size_t)units_of(s) * kD * sizeof(float));
  st = score_value_common(s, q_obs, k, v, causal, sc, idx_v, ws, need, prune_value_ws_bytes, stream);
  if (st != THK_OK) return st;
  // Long calls compact through the one-pass prune kernels with the list given: their hand-off
  // makes the blocks of a unit store together, and the memory takes a unit's rows in one burst
  // better than the same rows interleaved with other units' loads (32 layers of 128 units x
  // 4096 rows: 1225 -> 1100 us).  The value score's scratch is free again by then.
  const FusedPlan fp = fused_plan(s);
  if (value_compact_in_bursts(s, fp)) {
    const int spin = env_switches().spin_limit >= 0 ? (int)env_switches().spin_limit : 4096;
    if (failed(launch_prune_fused(s->dtype, v, v, nullptr, idx_v, v_pruned, ws, units_of(s), s->S, keep_rows(s),
                                  cache_rows(s, keep_rows(s)), 1, 0, s->T, ld_of(s), fp.NB, fp.RB, fp.hold, spin, 1,
                                  (hipStream_t)stream)))
      return THK_ERR_HIP;
    return THK_OK;
  }
  return thk_compact_keys(s, v, idx_v, v_pruned, stream);
}

static thk_status decode_common(const thk_shape *s, const void *q, const void *k_pruned,
                                const int16_t *idx, const void *v, const int16_t *idx_v, int32_t T_v,
                                int32_t ld_v, const void *k_tail, const void *v_tail, int32_t s_tail,
                                int32_t s_tail_cap, void *out, void *ws, size_t ws_bytes, void *stream,
                                const Split *split = nullptr) {
  const thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  if (q == nullptr || k_pruned == nullptr || idx == nullptr || v == nullptr || out == nullptr) return THK_ERR_NULL;
  if (s_tail < 0 || s_tail_cap < 0 || s_tail > s_tail_cap) return THK_ERR_SHAPE;
  if (s_tail > 0 && k_tail == nullptr) return THK_ERR_NULL;
  const bool pruned_v = T_v > 0;
  if (pruned_v) {
    if (idx_v == nullptr || (s_tail > 0 && v_tail == nullptr)) return THK_ERR_NULL;
    if (T_v > s->D || ld_v < T_v || ld_v > s->D) return THK_ERR_SHAPE;
    if (ld_v % 4 != 0) return THK_ERR_UNSUPPORTED;
    if (!aligned16(idx_v)) return THK_ERR_ALIGN;
  }
  const bool unified_v = s_tail > 0 && v_tail == nullptr;   // tail values follow row S in v
  const int64_t unit_rows = cache_rows(s, s->S);
  if (unit_rows < s->S + (unified_v ? s_tail : 0)) return THK_ERR_SHAPE;
  if (!aligned16(q) || !aligned16(k_pruned) || !aligned16(idx) || !aligned16(v) || !aligned16(out) ||
      (s_tail > 0 && (!aligned16(k_tail) || (v_tail != nullptr && !aligned16(v_tail)))))
    return THK_ERR_ALIGN;
  const bool ws_usable = ws != nullptr && aligned16(ws);
  const Split sp = split != nullptr ? *split : decode_split(s, ws_usable ? ws_bytes : 0, s_tail > 0);
  const int G = s->N_q / s->N_kv;
  if (units_of(s) * ceil_div(G, decode_heads_per_block(s)) * sp.n > kMaxGrid) return THK_ERR_SHAPE;
  if (sp.n > 1 && (!ws_usable || ws_bytes < decode_ws_bytes(s, sp.n))) return THK_ERR_WORKSPACE;
  DecodeArgs a;
  a.q = q; a.kp = k_pruned; a.v = v; a.kt = k_tail; a.vt = v_tail; a.idx = idx; a.out = out;
  a.ws = (float *)ws;
  a.S = s->S; a.rows_per_split = sp.rows;
  a.T = s->T; a.ldk = ld_of(s); a.N_q = s->N_q; a.N_kv = s->N_kv;
  a.s_tail = s_tail; a.s_tail_cap = s_tail_cap; a.n_split = sp.n; a.dtype = s->dtype;
  a.units = units_of(s);
  a.G = G;
  a.split_inv = ((uint64_t)1 << kSplitShift) / (uint32_t)sp.n + 1;
  a.unit_rows = unit_rows;
  a.unified_v = unified_v ? 1 : 0;
  a.scale_log2_d = 1.4426950408889634 / sqrt((double)s->D);
  a.scale_log2 = (float)a.scale_log2_d;
  a.idx_v = idx_v; a.T_v = pruned_v ? T_v : 0; a.ld_v = pruned_v ? ld_v : 0;
  // up to kDecodeFuseMaxSplit pieces per unit are merged inside the launch by the block that
  // finishes last; more pieces go to the merge kernel
  a.arrive = nullptr;
  a.nonce = 0;
  if (decode_merge_in_launch(s, sp.n)) {
    a.arrive = (unsigned long long *)((char *)ws + decode_records_bytes(s, sp.n));
    a.nonce = next_nonce();
  }
  if (failed(launch_decode(a, (hipStream_t)stream))) return THK_ERR_HIP;
  return THK_OK;
}

thk_status thk_decode_attn(const thk_shape *s, const void *q, const void *k_pruned,
                           const int16_t *idx, const void *v, const void *k_tail,
                           const void *v_tail, int32_t s_tail, int32_t s_tail_cap, void *out,
                           void *ws, size_t ws_bytes, void *stream) {
  return decode_common(s, q, k_pruned, idx, v, nullptr, 0, 0, k_tail, v_tail, s_tail, s_tail_cap, out, ws,
                       ws_bytes, stream);
}

thk_status thk_decode_attn_kv(const thk_shape *s, const void *q, const void *k_pruned,
                              const int16_t *idx, const void *v_pruned, const int16_t *idx_v,
                              int32_t T_v, int32_t ld_v, const void *k_tail, const void *v_tail,
                              int32_t s_tail, int32_t s_tail_cap, void *out, void *ws,
                              size_t ws_bytes, void *stream) {
  if (T_v < 1) return s == nullptr ? THK_ERR_NULL : THK_ERR_SHAPE;
  return decode_common(s, q, k_pruned, idx, v_pruned, idx_v, T_v, ld_v, k_tail, v_tail, s_tail, s_tail_cap, out,
                       ws, ws_bytes, stream);
}

// ---- the entry point that allocates nothing ---------------------------------------------
// Split partials of thk_decode_attn_static live in this file-scope device array instead of a
// caller workspace.  Every GPU the library runs on holds its own copy, at its own address,
// until the process ends.  In host code the array's NAME is only a stand-in for the symbol:
// the memory is reached through the per-device address hipGetSymbolAddress returns, looked up
// once per device on the entry point's first call there, and nowhere through the name.
static __device__ __align__(256) unsigned char scratch[THK_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void *> g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mu;

// Device address of `scratch` on the current device (set-up on first use, no allocation).
thk_status static_scratch(void **out) {
  int dev = -1;
  if (failed(hipGetDevice(&dev))) return THK_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return THK_ERR_UNSUPPORTED;
  void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (p == nullptr) {
      if (failed(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) || p == nullptr) return THK_ERR_HIP;
      g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
  }
  *out = p;
  return THK_OK;
}
}  // namespace

thk_status thk_decode_attn_static(const thk_shape *s, const void *q, const void *k_pruned,
                                  const int16_t *idx, const void *v, const void *k_tail,
                                  const void *v_tail, int32_t s_tail, int32_t s_tail_cap, void *out,
                                  void *stream) {
  thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  // the size check comes before anything touches the device
  const Split sp = decode_split(s, SIZE_MAX, s_tail > 0);
  if (sp.n > 1 && decode_ws_bytes(s, sp.n) > (size_t)THK_STATIC_SCRATCH_BYTES) return THK_ERR_SCRATCH;
  void *ws = nullptr;
  st = static_scratch(&ws);
  if (st != THK_OK) return st;
  return decode_common(s, q, k_pruned, idx, v, nullptr, 0, 0, k_tail, v_tail, s_tail, s_tail_cap, out, ws,
                       (size_t)THK_STATIC_SCRATCH_BYTES, stream, &sp);
}

thk_status thk_tail_append(const thk_shape *s, const void *k_new, const void *v_new, void *k_tail,
                           void *v_tail, int32_t s_tail, int32_t s_tail_cap, void *stream) {
  thk_status st = check_shape(s, false);
  if (st != THK_OK) return st;
  if (k_new == nullptr || v_new == nullptr || k_tail == nullptr || v_tail == nullptr) return THK_ERR_NULL;
  if (s_tail < 0 || s_tail >= s_tail_cap) return THK_ERR_SHAPE;
  if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_tail) || !aligned16(v_tail)) return THK_ERR_ALIGN;
  if (failed(launch_tail_append(s->dtype, k_new, v_new, k_tail, v_tail, units_of(s), s_tail_cap, s_tail, s_tail_cap,
                         s_tail, (hipStream_t)stream)))
    return THK_ERR_HIP;
  return THK_OK;
}

}  // extern "C"
