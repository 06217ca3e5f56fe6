// Value-channel score (Appendix "Value Cache Pruning"):
//   Score_v[j] = sum over the G query heads of a KV head of
//                || softmax(Q_obs K^T / sqrt(D)) V[:, j] ||_2 .
// The S_obs x S attention matrix times V is the one dense contraction of the method, so this
// file uses the matrix cores: a streaming attention over K and V (each read once) with the
// running-maximum softmax, followed by a small kernel that merges the pieces and takes the
// column norms.
//
// k_value_attn (bf16): 4 waves per block.  The G * S_obs query rows of one KV head are cut into
// tiles of 32 rows; a block carries QT of them (1 or 2; units with four or more go to
// k_value_attn_wide below) and streams the keys in chunks of
// 128 rows; wave w works on query tile w % QT and on the QT consecutive 32-key sub-tiles
// number w / QT of every chunk.  Per 32-key sub-tile a wave computes
//   S^T = K_sub Q^T        8 x v_mfma_f32_32x32x16_bf16 (A = keys from LDS, B = queries in VGPRs)
//   P^T = exp2(S^T - m)    in the accumulator layout, which already is the B-operand layout
//   O^T += V_sub^T P^T     16 x MFMA (P^T as two bf16 terms, hi + lo); the A operand (values
//                          transposed) comes from row-major LDS through ds_read_b64_tr_b16
// so neither the softmax maximum (a query is a lane column: 16 registers and one cross-half
// exchange) nor the probabilities ever move between lanes.
#include "thk_prune_device.h"

namespace thk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int kRec = 32 * kD + 64;   // floats per partial record: O^T [128][32], m [32], l [32]
constexpr float kNegBig = -1.0e30f;  // finite stand-in for "no key seen yet"

// One 32-key sub-tile of the running softmax in the MFMA accumulator layout: lane (n, h) holds, for
// query column n, the 16 keys kb + (r / 4) * 8 + h * 4 + r % 4.  Hides keys past `lim`, moves the
// reference m (rescaling the row sum and the output accumulators) and leaves the weights
// exp2(s * scale_log2 - m) in s.  m is not the running maximum itself: when some query's maximum
// passes its m, every query's m is set to kSlack above its maximum, and until one is passed again
// nothing moves (among 32 queries SOME maximum moves in most sub-tiles of a piece, 60 % of the 128
// of an 8192-row piece, 65 multiplications each time).  m above the maximum, not below it: weights
// stay at most 1, and sums that fit with the maximum itself still fit.  One octave: the rounding of
// the exponent grows with its distance from m, and the heaviest weights are within kSlack of it.
// Error of the score against 64 bits over some 50 random bf16 calls, relative to m = the maximum: 1.00 with
// 1, 1.01 with 2, 1.4 with 8.  64 units x 32768 rows, G = 4: 0 281 us, 1 277, 2 279, 8 271.
constexpr float kSlack = 1.f;
__device__ __forceinline__ void softmax_max(f32x16 &s, int64_t kb, int h, int64_t lim, int64_t lim_min,
                                            float scale_log2, float &m_run, float &l_run, f32x16 (&o)[4]) {
  if (kb + 31 > lim_min) {   // wave-uniform: only the sub-tiles that reach the window or the end
    const int64_t left = lim - kb;   // the last key of the sub-tile that counts, as a 32-bit offset (register pairs for 16 keys are too many)
    const int last = (int)(left < -1 ? -1 : left > 31 ? 31 : left) - h * 4;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if ((r >> 2) * 8 + (r & 3) > last) s[r] = -INFINITY;
    }
  }
  float mt = s[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) mt = fmaxf(mt, s[r]);
  const LanePair pr = pair32(mt);
  // the reference lives in the log2 domain (scale_log2 > 0 keeps the order)
  const float mx = fmaxf(pr.a, pr.b) * scale_log2;
  if (__any(mx > m_run)) {
    const float m_new = fmaxf(m_run, mx + kSlack);
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    l_run *= alpha;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
    m_run = m_new;
  }
}
__device__ __forceinline__ void softmax_exp(f32x16 &s, float scale_log2, float m_run) {
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2, -m_run));
}
// The probabilities of a sub-tile as two bf16 terms each, a pair per conversion instruction (one by one they take twice as
// many: value prunes of 64 units x 4 heads x 32768 rows 367.6 / 360.9 us, 32 x 8 heads x 13696 216.4 / 211.4), and their sum.
__device__ __forceinline__ void split_weights(const f32x16 &s, bf16x8 (&ph)[2], bf16x8 (&pl)[2], float &l_run) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < 16; r += 2) {
    const f32x2 p = {s[r], s[r + 1]};
    const bf16x2 hi = __builtin_convertvector(p, bf16x2);
    const uint32_t b = __builtin_bit_cast(uint32_t, hi);
    const f32x2 rest = {p[0] - __uint_as_float(b << 16), p[1] - __uint_as_float(b & 0xffff0000u)};
    const bf16x2 lo = __builtin_convertvector(rest, bf16x2);
    ph[r >> 3][r & 7] = hi[0];
    ph[r >> 3][(r & 7) + 1] = hi[1];
    pl[r >> 3][r & 7] = lo[0];
    pl[r >> 3][(r & 7) + 1] = lo[1];
    sum[r / 4] += p[0] + p[1];
  }
  l_run += (sum[0] + sum[1]) + (sum[2] + sum[3]);
}
__device__ __forceinline__ void softmax_step(f32x16 &s, int64_t kb, int h, int64_t lim, int64_t lim_min,
                                             float scale_log2, float &m_run, float &l_run, f32x16 (&o)[4]) {
  softmax_max(s, kb, h, lim, lim_min, scale_log2, m_run, l_run, o);
  softmax_exp(s, scale_log2, m_run);
}

// Which (query block, S piece, unit) a workgroup takes.  With one query block per unit the
// order is plain.  With several (more than 128 query rows per KV head) the blocks that stream
// the SAME keys and values are placed 8 workgroup numbers apart: same XCD, dispatched one after
// the other, so the second finds the rows in that XCD's L2 instead of fetching them again.
// False: a surplus workgroup of the rounded-up grid.
__device__ __forceinline__ bool value_block_work(const ValueAttnArgs &a, int &qb, int &sp, int64_t &u) {
  const int64_t bid = blockIdx.x;
  int64_t piece;   // (unit, S piece)
  if (a.n_qblk == 1) {
    qb = 0;
    piece = bid;
  } else {
    const int x = (int)(bid % kXcds);
    const int64_t slot = bid / kXcds;
    qb = (int)(slot % a.n_qblk);
    piece = (slot / a.n_qblk) * kXcds + x;
  }
  sp = (int)(piece % a.n_split);
  u = piece / a.n_split;
  return u < a.U;
}

// Partial record of one (unit, split, query tile): O^T [128][32], then m [32] and l [32].
__device__ __forceinline__ void write_record(float *rec, const f32x16 (&o)[4], float m_run, float l_tot, int n,
                                             int h) {
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int d = dt * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
      rec[d * 32 + n] = o[dt][r];
    }
  if (h == 0) {
    rec[32 * kD + n] = m_run;
    rec[32 * kD + 32 + n] = l_tot;
  }
}

// ---------------------------------------------------------------- bf16 ----
constexpr int kKst = 272;  // LDS bytes per key row: 16-lane b128 reads of 16 rows hit 64 distinct banks
constexpr int kVst = 320;  // LDS bytes per value row: the 4-row x 32-byte transposing reads of a
                           // half-wave cover all 64 banks once

// KEEP: values without the non-temporal hint (see fetch_part).
template <int QT, bool KEEP>
__global__ __launch_bounds__(256, 2) void k_value_attn_bf16(ValueAttnArgs a) {
  constexpr int KW = 4 / QT;     // waves that share a query tile, each on its own key sub-tiles
  constexpr int KT = QT;         // 32-key sub-tiles per wave and chunk
  constexpr int CR = 128;        // rows per chunk = KW * KT * 32
  constexpr int NP = 8;          // 16-row staging passes per chunk
  __shared__ __attribute__((aligned(16))) unsigned char smem[CR * (kKst + kVst)];
  unsigned char *Ks = smem, *Vs = smem + CR * kKst;

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int qt = w % QT, ksub = w / QT;
  const int n = lane & 31, h = lane >> 5;

  int qb, sp;
  int64_t u;
  if (!value_block_work(a, qb, sp, u)) return;

  const int rows_q = a.G * a.S_obs;
  const int qtile = qb * QT + qt;
  const int row = qtile * 32 + n;      // this lane's query row in the unit's (head, window row) list
  const int64_t S = a.S;

  // Query operand: 8 k-steps of 8 channels for this lane's (row, half).
  bf16x8 qreg[8];
  {
    const uint16_t *qp = (const uint16_t *)a.q_obs + ((size_t)u * rows_q + (row < rows_q ? row : 0)) * kD + h * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      u32x4 r = *(const u32x4 *)(qp + ks * 16);
      if (row >= rows_q) r = u32x4{0u, 0u, 0u, 0u};
      qreg[ks] = __builtin_bit_cast(bf16x8, r);
    }
  }
  // Last key this lane's query may see, and the smallest such limit in the call.
  const int64_t lim = a.causal ? S - a.S_obs + (row % a.S_obs) : S - 1;
  const int64_t lim_min = a.causal ? S - a.S_obs : S - 1;

  const int64_t k0 = (int64_t)sp * a.rows_per_split;
  const int64_t k1 = (k0 + a.rows_per_split < S) ? k0 + a.rows_per_split : S;
  const int nchunks = (int)((k1 - k0 + CR - 1) / CR);

  const unsigned char *kg = (const unsigned char *)a.k + (size_t)u * S * (kD * 2);
  const unsigned char *vg = (const unsigned char *)a.v + (size_t)u * S * (kD * 2);
  const int srow = tid >> 4, scol = (tid & 15) * 16;

  u32x4 pk[NP], pv[NP];
  // quarter q of the next chunk's loads: q = 0, 1 the two halves of the key rows, q = 2, 3 of
  // the value rows.  Keys are not needed again, nor are the values of a score call.  A value prune reads the values
  // once more, for the copy, and those loaded without the non-temporal hint are still in the memory-side cache then, the last
  // 256 MB of them.  The score loses by it where it is bound by memory.  Whole prunes, with the hint / without: four query tiles
  // and more (k_value_attn_wide) 64 units x 32768 rows 388 / 370 us, 184 x 15264 552 / 522, 24 x 2202, 8 heads 44.9 / 41.0, all of
  // 14 calls 1 to 9 % shorter; two tiles, MB of values: 46 57.1 / 53.4, 220 185 / 174, 300 238 / 229, 380 300 / 295, 420 299 /
  // 298, 460 305 / 310, 700 498 / 510, 850 518 / 539; one tile 24 units x 21938 rows 119.1 / 122.6, 32 x 4662 52.3 / 51.4.  Score calls
  // of two tiles 32 units x 53870 rows 168 / 185, 40 x 12645 70 / 75.  Hence KEEP in prunes of four tiles and more, and
  // of two up to 384 MiB of values.
  auto fetch_part = [&](int c, int q) {
    const unsigned char *g = q < 2 ? kg : vg;
#pragma unroll
    for (int pp = 0; pp < NP / 2; ++pp) {
      const int p = (q & 1) * (NP / 2) + pp;
      int64_t gr = k0 + (int64_t)c * CR + p * 16 + srow;
      gr = gr < S ? gr : S - 1;   // rows past the end repeat the last one; their weights are zero
      const u32x4 *src = (const u32x4 *)(g + gr * (kD * 2) + scol);
      if (q < 2) pk[p] = ld_stream(src);
      else pv[p] = KEEP ? *src : ld_stream(src);
    }
  };
  auto stash = [&]() {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      *(u32x4 *)(Ks + (p * 16 + srow) * kKst + scol) = pk[p];
      *(u32x4 *)(Vs + (p * 16 + srow) * kVst + scol) = pv[p];
    }
  };

  f32x16 o[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  float m_run = kNegBig, l_run = 0.f;

  // LDS addresses of this lane's operands inside a sub-tile
  const unsigned char *ka_p = Ks + (ksub * KT * 32 + n) * kKst + h * 16;
  const int j = lane & 15, gsub = (lane >> 4) & 1;
  const unsigned char *va_p = Vs + (ksub * KT * 32 + h * 4 + (j >> 2)) * kVst + (gsub * 16 + 4 * (j & 3)) * 2;

  if (nchunks > 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) fetch_part(0, q);
    stash();
  }
  __syncthreads();
  for (int c = 0; c < nchunks; ++c) {
    // the next chunk's loads are issued in four parts spread over this chunk's work, so that the
    // memory system has requests in flight throughout the compute phase
    const bool more = c + 1 < nchunks;
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      if (more) {
#pragma unroll
        for (int q = t * (4 / KT); q < (t + 1) * (4 / KT); ++q) fetch_part(c + 1, q);
      }
      const int64_t kb = k0 + (int64_t)c * CR + (ksub * KT + t) * 32;   // first key of the sub-tile
      if (kb >= k1) continue;
      const unsigned char *ka_t = ka_p + t * 32 * kKst, *va_t = va_p + t * 32 * kVst;
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const bf16x8 ka = *(const bf16x8 *)(ka_t + ks * 32);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qreg[ks], s, 0, 0, 0);
      }
      softmax_step(s, kb, h, lim, lim_min, a.scale_log2, m_run, l_run, o);
      // The probabilities enter the second product as TWO bf16 terms, p = hi + lo with hi the
      // nearest bf16 to p and lo the nearest bf16 to p - hi (that difference is exact in fp32):
      // |p - hi - lo| <= 2^-18 p, so the matrix product loses nothing that fp32 arithmetic keeps.
      // The row sum takes the fp32 values.
      bf16x8 ph[2], pl[2];
      split_weights(s, ph, pl, l_run);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {
          const unsigned char *vp = va_t + (k2 * 16) * kVst + dt * 64;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) s16x4 *)(vp));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) s16x4 *)(vp + 8 * kVst));
          const bf16x8 va = __builtin_bit_cast(
              bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, ph[k2], o[dt], 0, 0, 0);
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pl[k2], o[dt], 0, 0, 0);
        }
      }
    }
    __syncthreads();
    if (c + 1 < nchunks) stash();
    __syncthreads();
  }

  // The waves that carried the same query tile over different key sub-tiles meet in LDS (the
  // staging buffers are free after the loop's last barrier): common maximum, rescale, and the
  // wave of sub-tile 0 adds the others up.
  float l_tot = l_run + __shfl_xor(l_run, 32);
  if constexpr (KW > 1) {
    float *mx = (float *)smem;                 // [KW][QT][32] maxima, then [KW][QT][32] sums
    float *ox = mx + 2 * KW * QT * 32;         // [KW - 1][QT][64 registers][64 lanes]
    if (h == 0) mx[(ksub * QT + qt) * 32 + n] = m_run;
    __syncthreads();
    float M = m_run;
#pragma unroll
    for (int k = 0; k < KW; ++k) M = fmaxf(M, mx[(k * QT + qt) * 32 + n]);
    const float alpha = __builtin_amdgcn_exp2f(m_run - M);
    l_tot *= alpha;
    m_run = M;
    if (ksub > 0) {
      float *dst = ox + (size_t)((ksub - 1) * QT + qt) * 64 * 64 + lane;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[(dt * 16 + r) * 64] = o[dt][r] * alpha;
      if (h == 0) mx[(KW + ksub) * QT * 32 + qt * 32 + n] = l_tot;
    }
    __syncthreads();
    if (ksub > 0) return;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
#pragma unroll
    for (int k = 1; k < KW; ++k) {
      const float *src = ox + (size_t)((k - 1) * QT + qt) * 64 * 64 + lane;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] += src[(dt * 16 + r) * 64];
      l_tot += mx[(KW + k) * QT * 32 + qt * 32 + n];
    }
  }
  // partial record of (unit, split, query tile)
  const int nqt = a.n_qblk * QT;
  write_record(a.part + (((size_t)u * a.n_split + sp) * nqt + qtile) * kRec, o, m_run, l_tot, n, h);
}

// Units with four or more query tiles (G * S_obs > 96 rows: grouped heads): 8 waves, one block per
// compute unit, QT = 4 or 8 query tiles, so that a key / value row is fetched for 128 or 256 query rows
// at once.  Against the kernel above:
//   * rows go from memory to LDS without passing through registers (global_load_lds, 16 bytes per
//     lane): the 64 staging registers and the copy through them are gone, the next chunk is in
//     flight during all of a chunk's work, and there is one barrier per chunk;
//   * that transfer writes LDS in lane order, so bank conflicts are avoided by permuting the SOURCE:
//     16-byte chunk c of key row r lies at chunk c ^ (r & 15) (a b128 read takes one chunk of 16
//     rows), of value row r at c ^ ((r & 3) << 2) (a transposing read takes 64 bytes of 4 rows);
//   * the next sub-tile's logits are computed in front of this one's softmax, in straight-line code,
//     so that matrix and vector instructions of one wave run side by side.
// Two thirds of its time are instructions: of the 417000 cycles a compute unit is busy with 64 units x 32768 rows x 128 query rows a SIMD
// multiplies for 197000 (6144 products) and issues 40500 vector instructions, 6.6 a product.  A loop of such a mix, two waves a SIMD
// (a product of 32 cycles, six multiply-adds of 2.7, an exponential of 9.8), takes 44.6 cycles a product, for about 14 cycles of vector
// instructions run beside one: 274000.  The other third is waiting, for operands from LDS and at a chunk's barriers; the LDS
// is in use for 16 %, without conflicts.  206 GFLOP issued at 0.91 PFLOP/s, where a large product sustains 1.2 on this card; the clock
// is 1.7 to 2.0 GHz (2.4 in the copy kernel of the same run).  Operands read a sub-tile ahead measured 2-3 %
// longer, a higher priority for one of a SIMD's two waves, or waves 4 .. 7 half a step behind, the same.
// 64 units x 32768 rows, G = 4, S_obs = 32: 300 -> 277 us; 8 units x 131072 rows, S_obs = 64: 279 -> 237;
// 32 units x 16384 rows, G = 8: 150 -> 131 us (score calls, before: the kernel above with QT = 4).
constexpr int kWideRows = 128;                    // rows per chunk
constexpr int kWideBytes = kWideRows * kD * 2;    // one tensor's chunk in LDS

// One chunk of one tensor, 4 rows (1024 bytes) per instruction, KEYS: the key permutation; KEEP: without the
// non-temporal hint (see fetch_part above).
template <bool KEYS, bool KEEP>
__device__ __forceinline__ void wide_fetch(const unsigned char *g, int64_t last, unsigned char *lds, int wave,
                                           int lane) {
  constexpr int NI = kWideRows / 4 / 8;           // instructions per wave
  const int rsub = lane >> 4, slot = lane & 15;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int inst = wave * NI + i;
    const int row = inst * 4 + rsub;
    const int chunk = KEYS ? slot ^ ((inst & 3) * 4 + rsub) : slot ^ (rsub << 2);
    // rows past the end repeat the last one; their weights are zero
    const uint32_t off = (uint32_t)(row < last ? row : (int)last) * (kD * 2) + chunk * 16;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(g + off),
                                     (__attribute__((address_space(3))) void *)(lds + inst * 1024), 16, 0, KEEP ? 0 : 2 /* nt */);
  }
}

template <int QT, bool KEEP>
__global__ __launch_bounds__(512, 2) void k_value_attn_wide(ValueAttnArgs a) {
  constexpr int KW = 8 / QT;                      // waves that share a query tile, each on its own keys
  constexpr int KT = kWideRows / 32 / KW;         // sub-tiles per wave and chunk
  // a variable per buffer: reads of one are then known not to depend on transfers into another
  __shared__ __attribute__((aligned(1024))) unsigned char kb0[kWideBytes], vb0[kWideBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char kb1[kWideBytes], vb1[kWideBytes];

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qt = w % QT, ksub = w / QT;
  const int n = lane & 31, h = lane >> 5;

  int qb, sp;
  int64_t u;
  if (!value_block_work(a, qb, sp, u)) return;

  const int rows_q = a.G * a.S_obs;
  const int qtile = qb * QT + qt;
  const int row = qtile * 32 + n;      // this lane's query row in the unit's (head, window row) list
  const int64_t S = a.S;
  const int64_t k0 = (int64_t)sp * a.rows_per_split;
  const int64_t k1 = (k0 + a.rows_per_split < S) ? k0 + a.rows_per_split : S;
  const int nchunks = (int)((k1 - k0 + kWideRows - 1) / kWideRows);
  const unsigned char *kg = (const unsigned char *)a.k + ((size_t)u * S + k0) * (kD * 2);
  const unsigned char *vg = (const unsigned char *)a.v + ((size_t)u * S + k0) * (kD * 2);

  auto fetch = [&](int c, unsigned char *kb, unsigned char *vb) {
    const int64_t r0 = (int64_t)c * kWideRows;
    const int64_t last = S - 1 - k0 - r0;          // the unit's last row, seen from the chunk's first
    const int64_t lc = last < kWideRows - 1 ? last : kWideRows - 1;
    wide_fetch<true, false>(kg + r0 * (kD * 2), lc, kb, w, lane);
    wide_fetch<false, KEEP>(vg + r0 * (kD * 2), lc, vb, w, lane);
  };
  if (nchunks > 0) fetch(0, kb0, vb0);

  // Query operand: 8 k-steps of 8 channels for this lane's (row, half).
  bf16x8 qreg[8];
  {
    const uint16_t *qp = (const uint16_t *)a.q_obs + ((size_t)u * rows_q + (row < rows_q ? row : 0)) * kD + h * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      u32x4 r = *(const u32x4 *)(qp + ks * 16);
      if (row >= rows_q) r = u32x4{0u, 0u, 0u, 0u};
      qreg[ks] = __builtin_bit_cast(bf16x8, r);
    }
  }
  // Last key this lane's query may see, and the smallest such limit in the call.
  const int64_t lim = a.causal ? S - a.S_obs + (row % a.S_obs) : S - 1;
  const int64_t lim_min = a.causal ? S - a.S_obs : S - 1;

  f32x16 o[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  float m_run = kNegBig, l_run = 0.f;

  // this lane's operand offsets inside a sub-tile
  const int j = lane & 15, gsub = (lane >> 4) & 1;
  const int ka_off = (ksub * KT * 32 + n) * 256 + ((h ^ (n & 15)) << 4);       // chunk 2 ks + h: ^ ks * 32
  const int va_row = (ksub * KT * 32 + h * 4 + (j >> 2)) * 256 + gsub * 32 + (j & 3) * 8;
  int va_off[4];                                                               // 64-byte block dt
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) va_off[dt] = va_row + ((dt ^ (j >> 2)) << 6);

  auto logits = [&](const unsigned char *kb, int t) {
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const bf16x8 ka = *(const bf16x8 *)(kb + (ka_off ^ (ks * 32)) + t * 32 * 256);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qreg[ks], s, 0, 0, 0);
    }
    return s;
  };
  auto values = [&](f32x16 &s, const unsigned char *vb, int t) {
    // two bf16 terms per probability (see k_value_attn_bf16)
    bf16x8 ph[2], pl[2];
    split_weights(s, ph, pl, l_run);
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const unsigned char *vp = vb + va_off[dt] + (t * 32 + k2 * 16) * 256;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(vp));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(vp + 8 * 256));
        const bf16x8 va = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, ph[k2], o[dt], 0, 0, 0);
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pl[k2], o[dt], 0, 0, 0);
      }
  };
  const bool active = qtile * 32 < rows_q;   // a unit's last block may have tiles without rows: they only help to load
  auto chunk = [&](int c, const unsigned char *kb, const unsigned char *vb, unsigned char *kb_next, unsigned char *vb_next) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of chunk c has landed
    __syncthreads();                                   // ... everybody's, and chunk c - 1 is no longer read
    if (c + 1 < nchunks) fetch(c + 1, kb_next, vb_next);
    if (!active) return;
    const int64_t kb0_row = k0 + (int64_t)c * kWideRows + ksub * KT * 32;
    f32x16 s = logits(kb, 0);
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      softmax_max(s, kb0_row + t * 32, h, lim, lim_min, a.scale_log2, m_run, l_run, o);
      f32x16 s_next;
      if (t + 1 < KT) s_next = logits(kb, t + 1);
      softmax_exp(s, a.scale_log2, m_run);
      values(s, vb, t);
      if (t + 1 < KT) s = s_next;
    }
  };
  for (int c = 0; c < nchunks; c += 2) {
    chunk(c, kb0, vb0, kb1, vb1);
    if (c + 1 < nchunks) chunk(c + 1, kb1, vb1, kb0, vb0);
  }

  // The waves that carried the same query tile meet in LDS (as in k_value_attn_bf16).
  float l_tot = l_run + __shfl_xor(l_run, 32);
  if constexpr (KW == 2) {
    __syncthreads();                           // the last chunk is no longer read
    float *mx = (float *)kb1;                  // [2][QT][32] maxima, then the second group's sums
    float *ox0 = (float *)kb0, *ox1 = (float *)vb0;   // two query tiles' [64 registers][64 lanes] in each
    if (h == 0) mx[(ksub * QT + qt) * 32 + n] = m_run;
    __syncthreads();
    const float M = fmaxf(mx[qt * 32 + n], mx[(QT + qt) * 32 + n]);
    const float alpha = __builtin_amdgcn_exp2f(m_run - M);
    l_tot *= alpha;
    m_run = M;
    float *xch = (qt < 2 ? ox0 : ox1) + (size_t)(qt & 1) * 64 * 64 + lane;
    if (ksub > 0) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) xch[(dt * 16 + r) * 64] = o[dt][r] * alpha;
      if (h == 0) mx[2 * QT * 32 + qt * 32 + n] = l_tot;
    }
    __syncthreads();
    if (ksub > 0) return;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = o[dt][r] * alpha + xch[(dt * 16 + r) * 64];
    l_tot += mx[2 * QT * 32 + qt * 32 + n];
  }
  const int nqt = a.n_qblk * QT;
  write_record(a.part + (((size_t)u * a.n_split + sp) * nqt + qtile) * kRec, o, m_run, l_tot, n, h);
}

// ---------------------------------------------------------------- fp32 ----
// The same streaming attention in full fp32 on v_mfma_f32_32x32x2_f32 (one 32-key tile per
// step, one wave per query tile, QT waves per block).  The contraction index of an MFMA step is
// the lane half h: step j of the logits multiplies channel 8 * (j / 4) + 4 * h + j % 4, so a
// lane reads its four channels of four consecutive steps as one 16-byte LDS word; step j of
// O^T += V^T P^T multiplies key (j / 4) * 8 + 4 * h + j % 4, which is accumulator register j of
// P^T.  Probabilities stay fp32.
constexpr int kKstF = 528;  // LDS bytes per key row (b128 reads of 16 rows: 64 distinct banks)
constexpr int kVstF = 544;  // LDS bytes per value row (the two halves read rows 4 apart: 32 banks apart)

template <int QT>
__global__ __launch_bounds__(64 * QT, QT == 4 ? 2 : 1) void k_value_attn_f32(ValueAttnArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char Ks[32 * kKstF];
  __shared__ __attribute__((aligned(16))) unsigned char Vs[32 * kVstF];
  constexpr int NT = 64 * QT;
  const int tid = threadIdx.x, lane = tid & 63, qt = tid >> 6;
  const int n = lane & 31, h = lane >> 5;

  int qb, sp;
  int64_t u;
  if (!value_block_work(a, qb, sp, u)) return;

  const int rows_q = a.G * a.S_obs;
  const int qtile = qb * QT + qt;
  const int row = qtile * 32 + n;
  const int64_t S = a.S;

  float4 qreg[16];   // channels 8 * jj + 4 * h .. + 3 of this lane's query row
  {
    const float *qp = (const float *)a.q_obs + ((size_t)u * rows_q + (row < rows_q ? row : 0)) * kD + h * 4;
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      qreg[jj] = *(const float4 *)(qp + jj * 8);
      if (row >= rows_q) qreg[jj] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  const int64_t lim = a.causal ? S - a.S_obs + (row % a.S_obs) : S - 1;
  const int64_t lim_min = a.causal ? S - a.S_obs : S - 1;
  const int64_t k0 = (int64_t)sp * a.rows_per_split;
  const int64_t k1 = (k0 + a.rows_per_split < S) ? k0 + a.rows_per_split : S;

  const unsigned char *kg = (const unsigned char *)a.k + (size_t)u * S * (kD * 4);
  const unsigned char *vg = (const unsigned char *)a.v + (size_t)u * S * (kD * 4);

  f32x16 o[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  float m_run = kNegBig, l_run = 0.f;

  const unsigned char *ka_p = Ks + n * kKstF + h * 16;
  const unsigned char *va_p = Vs + (h * 4) * kVstF + n * 4;

  // 32 rows of 512 bytes each: 1024 16-byte pieces per tensor, NP of each per thread.  A tile's values are on their way during its
  // logits, the next tile's keys during its second product: a block is one to four wavefronts, and waiting for each tile in turn
  // took it as long again as its products (3.4 us).  A staging buffer is written where the barrier in front has
  // shown that everybody has read it.  us per value prune, before / so: 256 units x 867 rows 157 / 116, 48 x 2 heads x
  // 3062, S_obs = 64 193 / 136, 16 x 28441 275 / 205, 8 x 477 35.5 / 32.9
  constexpr int NP = 1024 / NT;
  u32x4 pk[NP], pv[NP];
  // Blocks of two waves load a tile when they need it: ahead they measured longer wherever several share a compute unit (16 units x
  // 12364 rows, S_obs = 64 147 / 172, 16 x 2 heads x 26432 249 / 299).
  constexpr bool AHEAD = QT != 2;
  auto fetch = [&](u32x4 (&to)[NP], const unsigned char *g, int64_t kb) {
    // (a tile is a flat run of bytes that ends with the unit: rows past the end read 0, and their weights are 0)
    const int bytes = __builtin_amdgcn_readfirstlane((int)(S - kb < 32 ? S - kb : 32) * (kD * 4));
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(g + kb * (kD * 4)), (short)0, bytes, 0x00027000);
#pragma unroll
    for (int i = 0; i < NP; ++i)
      to[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, tid * 16 + i * (NT * 16), 0, 0));
  };
  auto commit = [&](unsigned char *lds, int pitch, const u32x4 (&from)[NP]) {
#pragma unroll
    for (int i = 0; i < NP; ++i) *(u32x4 *)(lds + ((i * NT + tid) >> 5) * pitch + ((i * NT + tid) & 31) * 16) = from[i];
  };
  auto stage = [&](int64_t kb) {   // both tensors' tile, a few pieces at a time
#pragma unroll 4
    for (int i = tid; i < 1024; i += NT) {
      const int r = i >> 5, c = (i & 31) * 16;
      int64_t gr = kb + r;
      gr = gr < S ? gr : S - 1;   // rows past the end repeat the last one; their weights are zero
      *(u32x4 *)(Ks + r * kKstF + c) = *(const u32x4 *)(kg + gr * (kD * 4) + c);
      *(u32x4 *)(Vs + r * kVstF + c) = *(const u32x4 *)(vg + gr * (kD * 4) + c);
    }
  };
  if (AHEAD && k0 < k1) fetch(pk, kg, k0);
  for (int64_t kb = k0; kb < k1; kb += 32) {
    if constexpr (AHEAD) {
      commit(Ks, kKstF, pk);
      fetch(pv, vg, kb);
    } else {
      __syncthreads();   // the last tile is no longer read
      stage(kb);
    }
    __syncthreads();   // the keys are there, and the last tile's values are no longer read
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      const float4 ka = *(const float4 *)(ka_p + jj * 32);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka.x, qreg[jj].x, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka.y, qreg[jj].y, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka.z, qreg[jj].z, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka.w, qreg[jj].w, s, 0, 0, 0);
    }
    softmax_step(s, kb, h, lim, lim_min, a.scale_log2, m_run, l_run, o);
    if constexpr (AHEAD) {
      commit(Vs, kVstF, pv);
      if (kb + 32 < k1) fetch(pk, kg, kb + 32);
      __syncthreads();   // the values are there, and the keys are no longer read
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) l_run += s[r];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const unsigned char *vp = va_p + ((j >> 2) * 8 + (j & 3)) * kVstF;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const float va = *(const float *)(vp + dt * 128);
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(va, s[j], o[dt], 0, 0, 0);
      }
    }
  }
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const int nqt = a.n_qblk * QT;
  write_record(a.part + (((size_t)u * a.n_split + sp) * nqt + qtile) * kRec, o, m_run, l_tot, n, h);
}

// Merge the partial records of one 32-row query tile of one unit and normalise.  A block of
// 256 threads covers DQ = 256 / PG value channels: thread (d, pg) sums the records p = pg,
// pg + PG, ... for channel d; the PG groups meet in LDS and are added in group order.  PG = 2 for few records, 8 for many.
// A unit with a single tile gets its score here (each thread holds all of its rows).  With several, a thread has the squares
// of its tile's part of every head: it stores the sum over the heads that lie inside the tile and the parts of the head that
// began before the tile and of the one that goes on behind it (kTileSums doubles a channel), and the block of the unit that
// finishes last adds the tiles up, in their order, and takes the roots.  (Squares used to go to a launch of their own: 64 units x 4
// tiles merge 8.2 and norms 7.4 us and the gap between them.)  Hand-off as in the decode kernels: sums and flags go to the
// device's coherence point, a flag is a word per block that holds the call's nonce, each is acknowledged before the next
// is issued, so the block whose flag comes last finds all of them set; blocks within a round trip of each other may both, and
// store the same bits.  The finishing block clears the flags for a replay of the launch.
// With idx the block that has a unit's whole score (a single tile and PG = 2, or several tiles) selects its Top_T, too: 40
// units x 384 rows 25.0 -> 23.2 us.
constexpr int kTileSums = 3;   // inside, began before, goes on behind
struct ValueMergeArgs {
  const float *part;
  double *sums;                  // [U][nt][kTileSums][kD]
  unsigned long long *flags;     // [U][blocks of a unit]
  unsigned long long nonce;
  float *score;
  int16_t *idx;
  int32_t T, G, S_obs, n_part, nqt, nt;
};
__device__ __forceinline__ double load_device(const double *p) {
  return __longlong_as_double((long long)__hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void store_device(double *p, double v) {
  __hip_atomic_store((unsigned long long *)p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int PG>
__global__ __launch_bounds__(256, 2) void k_value_merge(ValueMergeArgs a) {
  constexpr int DQ = 256 / PG, NDB = kD / DQ;   // channels per block, blocks per (unit, tile)
  extern __shared__ __attribute__((aligned(16))) float wts[];   // [n_part][32] merge weights, then [PG - 1][DQ][33] for the groups
  const int nqt = a.nqt, nt = a.nt, n_part = a.n_part, S_obs = a.S_obs;
  int64_t bid = blockIdx.x;
  const int db = (int)(bid % NDB);
  bid /= NDB;
  const int64_t u = bid / nt;
  const int t = (int)(bid % nt);
  const int dl = threadIdx.x % DQ, pg = threadIdx.x / DQ;
  const int d = db * DQ + dl;
  const int rows_q = a.G * S_obs;
  const float *pu = a.part + (size_t)u * n_part * nqt * kRec;
  // the first record's outputs are asked for in front of the weights; PG = 2: each further one's in front of the sums of the one before
  float4 x[8];
  auto fetch = [&](float4 (&to)[8], int p) {
    const float4 *src = (const float4 *)(pu + ((size_t)min(p, n_part - 1) * nqt + t) * kRec + d * 32);
#pragma unroll
    for (int q4 = 0; q4 < 8; ++q4) to[q4] = src[q4];
  };
  fetch(x, pg);
  // weights of the records, row q = tid % 32, records tid / 32, + 8, ... per thread (one thread per row
  // walked all of them before: 128 records took 60 us); PG = 2: at most eight records, one per thread
  __shared__ float red_m[8][32], red_l[8][32], s_sc[kD];
  {
    const int q = threadIdx.x & 31, rg = threadIdx.x >> 5;
    const float *rec = pu + (size_t)t * kRec + 32 * kD + q;
    const size_t step = (size_t)nqt * kRec;
    const float m0 = rec[min(rg, n_part - 1) * step], l0 = rec[min(rg, n_part - 1) * step + 32];   // a repeated record is no larger
    float M = m0;
    if constexpr (PG > 2)
      for (int p = rg + 8; p < n_part; p += 8) M = fmaxf(M, rec[p * step]);
    red_m[rg][q] = M;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) M = fmaxf(M, red_m[i][q]);
    float w0 = rg < n_part ? __builtin_amdgcn_exp2f(m0 - M) : 0.f, L = rg < n_part ? w0 * l0 : 0.f;
    if constexpr (PG > 2)
      for (int p = rg + 8; p < n_part; p += 8) {
        const float wv = __builtin_amdgcn_exp2f(rec[p * step] - M);
        wts[p * 32 + q] = wv;
        L += wv * rec[p * step + 32];
      }
    red_l[rg][q] = L;
    __syncthreads();
    L = red_l[0][q];
#pragma unroll
    for (int i = 1; i < 8; ++i) L += red_l[i][q];
    const float inv = L > 0.f ? 1.f / L : 0.f;
    // normalised before the records are added: a single record's sums may be near the end of the range
    if (rg < n_part) wts[rg * 32 + q] = w0 * inv;
    if constexpr (PG > 2)
      for (int p = rg + 8; p < n_part; p += 8) wts[p * 32 + q] *= inv;
  }
  __syncthreads();
  float acc[32];
#pragma unroll
  for (int q = 0; q < 32; ++q) acc[q] = 0.f;
  auto add = [&](const float4 (&from)[8], int p) {
    const float *wp = wts + p * 32;
#pragma unroll
    for (int q4 = 0; q4 < 8; ++q4) {
      const float4 w4 = *(const float4 *)(wp + q4 * 4);
      acc[q4 * 4 + 0] += w4.x * from[q4].x;
      acc[q4 * 4 + 1] += w4.y * from[q4].y;
      acc[q4 * 4 + 2] += w4.z * from[q4].z;
      acc[q4 * 4 + 3] += w4.w * from[q4].w;
    }
  };
  if constexpr (PG > 2) {
#pragma unroll 1
    for (int p = pg; p < n_part; p += PG) {
      if (p != pg) fetch(x, p);
      add(x, p);
    }
  } else {
    float4 y[8];
#pragma unroll 1
    for (int p = pg; p < n_part; p += 2 * PG) {
      if (p + PG < n_part) fetch(y, p + PG);
      add(x, p);
      if (p + PG < n_part) {
        if (p + 2 * PG < n_part) fetch(x, p + 2 * PG);
        add(y, p + PG);
      }
    }
  }
  __syncthreads();               // the weights are no longer read
  float *xch = wts;              // [PG - 1][DQ][33]
  if (pg > 0) {
#pragma unroll
    for (int q = 0; q < 32; ++q) xch[((pg - 1) * DQ + dl) * 33 + q] = acc[q];
  }
  __syncthreads();
  if (pg == 0) {
#pragma unroll 1
    for (int g2 = 1; g2 < PG; ++g2)
#pragma unroll
      for (int q = 0; q < 32; ++q) acc[q] += xch[((g2 - 1) * DQ + dl) * 33 + q];
    // squares in fp64, head by head: pos = rows of the head that came before this one
    double ss = 0.0, inside = 0.0, before = 0.0;
    int pos = (t * 32) % S_obs;
    bool mid = pos != 0;   // the head began before the tile
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      if (t * 32 + q < rows_q) {
        ss += (double)acc[q] * (double)acc[q];
        if (++pos == S_obs) {   // last window row of a head
          if (mid) before = ss;
          else inside += sqrt(ss);
          mid = false;
          ss = 0.0;
          pos = 0;
        }
      }
    }
    if (nt == 1) {
      a.score[(size_t)u * kD + d] = (float)inside;
      s_sc[d] = (float)inside;
    } else {
      double *dst = a.sums + ((size_t)u * nt + t) * (kTileSums * kD) + d;
      store_device(dst, inside);
      store_device(dst + kD, mid ? ss : before);   // (a head that fills the tile and goes on has all of it here)
      store_device(dst + 2 * kD, mid ? 0.0 : ss);
    }
  }
  if (nt > 1) {
    __shared__ int s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's sums are acknowledged
    __syncthreads();                                   // ... and every wave's
    const int nf = nt * NDB;
    unsigned long long *flags = a.flags + (size_t)u * nf;
    if (threadIdx.x < kWave) {
      if (threadIdx.x == 0) __hip_atomic_store(flags + t * NDB + db, a.nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the flag is out before the flags are read
      bool all = true;
      for (int i = threadIdx.x; i < nf; i += kWave)
        all = all && __hip_atomic_load(flags + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.nonce;
      all = __all(all);
      if (threadIdx.x == 0) s_last = all ? 1 : 0;
    }
    __syncthreads();
    if (s_last == 0) return;
    if (threadIdx.x < kD) {
      const double *src = a.sums + (size_t)u * nt * (kTileSums * kD) + threadIdx.x;
      double total = 0.0, open = 0.0;   // open: squares so far of a head that goes on
      int pos = 0;                      // its rows so far
      // sums that cannot be there are not asked for; those of eight tiles are in flight together
      constexpr int NB = 8;
      for (int t0 = 0; t0 < nt; t0 += NB) {
        double v[NB][kTileSums];
        int at = pos;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const double *tile = src + (size_t)(t0 + i) * (kTileSums * kD);
          const int end = at + 32;
          const bool here = t0 + i < nt;
          v[i][0] = here && end >= S_obs ? load_device(tile) : 0.0;
          v[i][1] = here && at != 0 ? load_device(tile + kD) : 0.0;
          at = end % S_obs;
          v[i][2] = here && at != 0 && (at < 32 || end == 32) ? load_device(tile + 2 * kD) : 0.0;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          open += v[i][1];
          const bool ends = pos + 32 >= S_obs;   // the open head, if there is one, ends here
          if (ends && pos != 0) total += sqrt(open);
          total += v[i][0];
          open = ends || pos == 0 ? v[i][2] : open;
          pos = (pos + 32) % S_obs;
        }
      }
      s_sc[threadIdx.x] = (float)total;
      a.score[(size_t)u * kD + threadIdx.x] = (float)total;
    }
    for (int i = threadIdx.x; i < nf; i += 256) __hip_atomic_store(flags + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (a.idx == nullptr) return;
  __shared__ int16_t s_list[kD];
  __syncthreads();
  select_block(s_sc, a.T, s_list);   // (not select_wave, whose 28 unrolled steps take such a launch longer to fetch than to run)
  if ((int)threadIdx.x < a.T) a.idx[(size_t)u * a.T + threadIdx.x] = s_list[threadIdx.x];
}

}  // namespace

int value_attn_qt(int G, int S_obs) {
  const int nqt = (G * S_obs + 31) / 32;
  return nqt >= 4 ? 4 : nqt >= 2 ? 2 : 1;
}

// Eight where the records, which are laid out in fours, come out even.
int value_wide_tiles(int G, int S_obs) {
  const int nqt = (G * S_obs + 31) / 32;
  return (nqt + 3) / 4 % 2 == 0 ? 8 : 4;
}

size_t value_part_bytes(int64_t U, int G, int S_obs, int n_split) {
  const int QT = value_attn_qt(G, S_obs);
  const int nqt = (G * S_obs + 31) / 32;
  const int n_qblk = (nqt + QT - 1) / QT;
  // several tiles: room for a tile's squared outputs, of which the merge uses what its sums and flags take
  const size_t sums = nqt > 1 ? (size_t)U * nqt * 32 * kD * sizeof(float) : 0;
  static_assert(32 * kD * sizeof(float) >= kTileSums * kD * sizeof(double) + 4 * sizeof(unsigned long long), "sums and flags of a tile");
  return (size_t)U * n_split * n_qblk * QT * kRec * sizeof(float) + sums;
}

hipError_t launch_value_score(int dtype, const void *q_obs, const void *k, const void *v, float *part,
                              float *score, int16_t *idx, int T, int64_t U, int64_t S, int G, int S_obs, int causal,
                              int n_split, int64_t rows_per_split, unsigned long long nonce, hipStream_t st) {
  clear_stale_hip_error();
  const int QT = value_attn_qt(G, S_obs);
  const int nqt_real = (G * S_obs + 31) / 32;
  ValueAttnArgs a;
  a.q_obs = q_obs; a.k = k; a.v = v; a.part = part;
  a.S = S; a.rows_per_split = rows_per_split;
  a.G = G; a.S_obs = S_obs; a.n_split = n_split; a.causal = causal;
  // bf16 with four or more query tiles: the 8-wave kernel, with eight tiles per block where that
  // leaves a block for every compute unit, else with four and twice the blocks
  const bool wide = dtype == THK_BF16 && QT == 4;
  int QB = wide ? value_wide_tiles(G, S_obs) : QT;
  if (QB == 8 && U * n_split * ((nqt_real + 7) / 8) < kCUs) QB = 4;
  a.n_qblk = (nqt_real + QB - 1) / QB;
  a.scale_log2 = (float)(1.4426950408889634 / sqrt((double)kD));
  a.U = U;
  // several query blocks per (unit, piece): pieces rounded up to a multiple of the XCD count
  // (value_block_work; the surplus workgroups return at once)
  const int64_t pieces = a.n_qblk == 1 ? U * n_split : (U * n_split + kXcds - 1) / kXcds * kXcds;
  const unsigned grid = (unsigned)(pieces * a.n_qblk);
  const void *fn;
  int threads = 256;
  if (dtype == THK_BF16) {
    // a copy of the values follows, and finds enough of them in the memory-side cache (fetch_part)
    const bool keep = idx != nullptr && (wide || (size_t)U * S * (kD * 2) <= (size_t)384 << 20);
    if (wide)
      fn = keep ? (QB == 8 ? (const void *)k_value_attn_wide<8, true> : (const void *)k_value_attn_wide<4, true>)
                : (QB == 8 ? (const void *)k_value_attn_wide<8, false> : (const void *)k_value_attn_wide<4, false>);
    else if (QT == 2)
      fn = keep ? (const void *)k_value_attn_bf16<2, true> : (const void *)k_value_attn_bf16<2, false>;
    else
      fn = (const void *)k_value_attn_bf16<1, false>;
  } else {
    fn = QT == 4 ? (const void *)k_value_attn_f32<4> : QT == 2 ? (const void *)k_value_attn_f32<2> : (const void *)k_value_attn_f32<1>;
    threads = QT == 4 ? 256 : QT == 2 ? 128 : 64;
  }
  if (wide) threads = 512;
  void *kargs[] = {(void *)&a};
  hipError_t e = launch_main_kernel(fn, dim3(grid), dim3(threads), kargs, 0, st);
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int n_part = n_split;
  const int nqt = a.n_qblk * QB;
  // few records: 2 groups x 128 channels per block; many: 8 groups x 32 channels, 4 blocks
  const int PG = n_part > 8 ? 8 : 2;
  const int DQ = 256 / PG;
  size_t lds = (size_t)n_part * 32 * sizeof(float);
  const size_t xch = (size_t)(PG - 1) * DQ * 33 * sizeof(float);
  if (lds < xch) lds = xch;
  const dim3 mg((unsigned)(U * nqt_real * (kD / DQ)));
  const bool select_here = idx != nullptr && (PG == 2 || nqt_real > 1);
  ValueMergeArgs m;
  m.part = part; m.score = score; m.idx = select_here ? idx : nullptr; m.nonce = nonce;
  m.T = T; m.G = G; m.S_obs = S_obs; m.n_part = n_part; m.nqt = nqt; m.nt = nqt_real;
  m.sums = (double *)(part + (size_t)U * n_part * nqt * kRec);   // behind the partial records, then the flags
  m.flags = (unsigned long long *)(m.sums + (size_t)U * nqt_real * kTileSums * kD);
  if (PG == 8) hipLaunchKernelGGL(k_value_merge<8>, mg, dim3(256), lds, st, m);
  else hipLaunchKernelGGL(k_value_merge<2>, mg, dim3(256), lds, st, m);
  e = hipGetLastError();
  if (e != hipSuccess || select_here || idx == nullptr) return e;
  return launch_select(score, idx, U, T, st);
}

}  // namespace thk
