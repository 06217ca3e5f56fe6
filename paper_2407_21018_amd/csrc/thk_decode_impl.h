// Decode attention over the pruned key cache plus the unpruned tail
// (Sec. 3.3, Fig. 2; attention formula of Sec. 3.2) -- gfx950, wave64.
// Template body shared by the per-(dtype, group width) translation units.
//
// Work split.  A 256-thread block serves one (unit, query-head group, S-split):
// GT query heads that read the same KV head share every K and V byte the block
// streams.  Its four wavefronts work independently on tiles of TR rows, each
// with its own running softmax state (max, sum, acc[128]); the states are merged
// once at the end through LDS.  With n_split > 1 the block writes its state to
// the workspace and k_decode_merge combines the splits in index order.
//
// One tile, one wavefront.
//   K_pruned rows are T elements long and in general not 16-byte multiples, but
//   a run of whole rows is a flat byte range.  The range, widened to 16-byte
//   boundaries, is fetched with coalesced 16-byte loads into registers (the
//   next tile's range is in flight while the current tile is computed) and
//   mirrored into the wave's LDS slab.  LPK = 64 / TR lanes then walk one row
//   out of LDS, each taking a contiguous share of its channels, so the q.K dot
//   product needs at most one neighbour exchange.  V rows are 128 elements:
//   they go straight into registers, 16 bytes per lane, each lane accumulating
//   its VEC output channels over the rows it sees.  The tile's probabilities
//   travel from the row layout to the V layout through a TR-float LDS line per
//   query head.
#pragma once
#include <math.h>

#include "thk_internal.h"

namespace thk {

constexpr int kTailRows = 16;   // rows per tile in the full-width tail segment
constexpr int kQS = kD + 8;     // floats per query vector in LDS: 128 channels + 8 zeros
constexpr int kBufferWord3 = 0x00027000, kNonTemporal = 2;   // raw buffer of bytes; the hint of ld_stream

__device__ inline void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Cross-lane reductions over the 64 lanes with DPP row shifts and row
// broadcasts: after the four row_shr steps lane 15 of every 16-lane row holds
// the row's result, row_bcast:15 folds rows 0->1 and 2->3, row_bcast:31 folds
// the lower half into rows 2 and 3, and lane 63 holds the total.  A lane whose
// DPP source does not exist receives `old`; passing the lane's own value as
// `old` makes the step a no-op there (max(x, x); x + 0 needs the identity 0)
// and lets the compiler fold the move into the arithmetic instruction.
template <int CTRL, int ROW_MASK>
__device__ inline float dpp_move(float old, float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), CTRL,
                                                    ROW_MASK, 0xf, false));
}
// Wave-wide maximum with the DPP step folded into v_max_f32 (one instruction per
// step, written out because the compiler keeps a separate v_mov_dpp).  In-place
// form: a lane whose DPP source does not exist, or whose row is masked off, is
// not written and keeps its value.  The s_nop covers the two wait states a DPP
// read needs after the VALU write of the same register.
#define THK_DPP_MAX(x, ctrl) \
  asm volatile("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 " ctrl : "+v"(x))
__device__ inline float wave_max(float x) {
  THK_DPP_MAX(x, "row_shr:1 row_mask:0xf bank_mask:0xf");
  THK_DPP_MAX(x, "row_shr:2 row_mask:0xf bank_mask:0xf");
  THK_DPP_MAX(x, "row_shr:4 row_mask:0xf bank_mask:0xf");
  THK_DPP_MAX(x, "row_shr:8 row_mask:0xf bank_mask:0xf");
  THK_DPP_MAX(x, "row_bcast:15 row_mask:0xa bank_mask:0xf");
  THK_DPP_MAX(x, "row_bcast:31 row_mask:0xc bank_mask:0xf");
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ inline float max_nn(float a, float b) { return a > b ? a : b; }   // inputs are never NaN
__device__ inline float wave_sum(float x) {
  x += dpp_move<0x111, 0xf>(0.f, x);
  x += dpp_move<0x112, 0xf>(0.f, x);
  x += dpp_move<0x114, 0xf>(0.f, x);
  x += dpp_move<0x118, 0xf>(0.f, x);
  x += dpp_move<0x142, 0xa>(0.f, x);
  x += dpp_move<0x143, 0xc>(0.f, x);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
// value of the neighbouring lane (lane ^ 1): quad_perm [1,0,3,2]
__device__ inline float lane_swap1(float x) { return dpp_move<0xB1, 0xf>(0.f, x); }
__device__ inline double lane_swap1(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0xB1, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0xB1, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// RA bytes of an fp32 row in LDS.
template <int RA>
__device__ inline void lds_floats(const char *p, float *f) {
  if constexpr (RA == 16) {
    const float4 r = *(const float4 *)p; f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w;
  } else if constexpr (RA == 8) {
    const float2 r = *(const float2 *)p; f[0] = r.x; f[1] = r.y;
  } else {
    f[0] = *(const float *)p;
  }
}

// DW consecutive 32-bit words from LDS (address aligned to DW * 4 bytes).
template <int DW>
__device__ inline void lds_words(const char *p, uint32_t (&w)[DW]) {
  if constexpr (DW == 4) {
    const u32x4 r = *(const u32x4 *)p; w[0] = r.x; w[1] = r.y; w[2] = r.z; w[3] = r.w;
  } else if constexpr (DW == 2) {
    const uint2 r = *(const uint2 *)p; w[0] = r.x; w[1] = r.y;
  } else {
    w[0] = *(const uint32_t *)p;
  }
}

// DW words of a bf16 row in LDS whose rows start at multiples of RA bytes.  RA = 2 (dense rows of an odd T: 51 is
// lambda = 0.6): p is the word below the row's place, of which a lane takes the upper or the lower halves -- its
// row starts on a word or in the middle of one (shift_bytes 0, 2), the same for the whole row.
template <int RA, int DW>
__device__ __forceinline__ void bf16_words(const char *p, uint32_t shift_bytes, uint32_t (&w)[DW]) {
  if constexpr (RA >= 4 * DW) {
    lds_words<DW>(p, w);
  } else {
    const uint32_t *q = (const uint32_t *)p;
#pragma unroll
    for (int d = 0; d < DW; ++d) w[d] = RA == 2 ? __builtin_amdgcn_alignbyte(q[d + 1], q[d], shift_bytes) : q[d];
  }
}

// a.lo * b.lo + a.hi * b.hi + c with a, b pairs of bf16 (v_dot2c_f32_bf16)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ inline float dot2_bf16(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}

template <int DT> struct LogitType { using type = float; };
template <> struct LogitType<THK_F32> { using type = double; };
__device__ inline float fma_z(float a, float b, float c) { return fmaf(a, b, c); }
__device__ inline double fma_z(double a, double b, double c) { return fma(a, b, c); }

template <int DT, int GT>
struct TileState {
  float m[GT];                       // running max (log2 domain)
  float l[GT];                       // per-lane partial sum of probabilities
  float acc[GT][Elem<DT>::VEC];      // per-lane partial output channels
  float accp[GT][4];                 // channel-pruned values only: partial sums of 4 kept channels
};

// A lane's view of a tile of channel-pruned value rows staged in its wave's LDS slab: rows are
// ld elements apart, groups of 4 kept channels go to lanes (col), and rpw rows are handled per
// step (rsub = this lane's row within a step).
constexpr int kPsPad = 32;   // zero rows behind a wave's probabilities (channel-pruned values only)

struct VPruned {
  char *vbuf;
  int shift;        // bytes from the slab start to the tile's first row
  int ld;
  int rpw, rsub, col;
  bool active;
};

// ---- a tile's bytes through a buffer resource ------------------------------------------------
// `bytes` (a multiple of 16, 0: no tile) from a 16-byte boundary on, chunk j * 64 + lane per lane and load.
// The resource ends with the tile: chunks past it return 0 and move nothing, so no load is clamped and none
// sits behind a branch.  A branch around loads is what costs here: where its paths meet the compiler no
// longer knows how many loads are out and waits for ALL of them -- the first keys of a block were asked
// for only after its query had arrived (1 us of a 9 us call), the query was packed only when the first tile
// was there, and a tile's values waited for the next tile's keys.  Against clamped loads behind branches, whole
// calls: bf16, 8 units x 314 rows x 2 heads 9.5 -> 7.6 us, 8 x 4439 rows 13.1 -> 10.5, 32 x 1536 rows x 8 heads 14.6
// -> 11.5, 24 x 12801 rows 28.5 -> 26.6; fp32, 8 x 5160 rows x 7 heads 26.7 -> 22.2, 128 x 6080 rows x 5 heads 160
// -> 145; pruned values, 128 x 2096 rows 44.0 -> 39.3.  Calls of several hundred MB: 0 to 4 %.
struct ByteRange {   // wave-uniform
  const char *base;
  int bytes, shift;  // shift: from base to the first row
};
// nrows rows of W elements, ld apart, from byte beg of tensor t (16-byte aligned), widened to 16-byte
// boundaries, so up to 15 bytes before the first row and after the last are read as well: before is
// always inside the tensor; after can pass the tensor's last element by less than 16 bytes, inside the 16-byte
// granule that holds it (the API requires that granule to be readable).
template <int EB>
__device__ __forceinline__ ByteRange flat_rows(const void *t, size_t beg, int nrows, int W, int ld) {
  ByteRange r;
  r.shift = (int)(beg & 15);
  r.base = (const char *)t + (beg - r.shift);
  r.bytes = (r.shift + ((nrows - 1) * ld + W) * EB + 15) & ~15;
  return r;
}
// (stated for the compiler: a resource that it takes for divergent becomes a loop around every load)
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ const char *uniform_ptr(const char *p) {
  const uint64_t b = (uint64_t)p;
  return (const char *)((uint64_t)(uint32_t)uniform((int)(uint32_t)b) | (uint64_t)(uint32_t)uniform((int)(b >> 32)) << 32);
}
template <int N, int M>
__device__ __forceinline__ void tile_issue(u32x4 (&r)[M], const char *base, int bytes, int lane) {
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr(base), (short)0, uniform(bytes), kBufferWord3);
#pragma unroll
  for (int j = 0; j < N; ++j)
    r[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16 + j * (kWave * 16), 0, kNonTemporal));
}

template <int N, int M>
__device__ __forceinline__ void k_commit(const u32x4 (&kr)[M], char *kbuf, int lane) {
#pragma unroll
  for (int j = 0; j < N; ++j) ((u32x4 *)kbuf)[j * kWave + lane] = kr[j];   // kbuf holds M * 64 chunks
}

// The block's query rows and the unit's list of kept channels on their way to LDS: ONE trip to
// memory, 16 bytes of a row (threads 0 .. 127) and one list entry (threads 128 .. 255 keep it) per
// thread, issued before anything else and without a branch, so that waiting for them waits for nothing
// behind them.
// (Gathering q[idx[c]] from memory instead is two dependent trips, and four where the packed and
// the plain copy were made by two loops: 3-4 us at the start of every launch.)
template <int DT, int GT>
struct QueryStage {
  using B = typename Elem<DT>::Bits;
  static constexpr int LPR = kD / Elem<DT>::VEC;             // 16-byte chunks per row
  static_assert(GT * LPR <= 128, "one chunk per thread of the first two waves");
  u32x4 row;
  int16_t ch;
  __device__ __forceinline__ void issue(const void *q, size_t bn0, int heads, const int16_t *uidx, int T) {
    const int tid = threadIdx.x;
    // head slots that are not in use are past the resource's end: a zero query
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)q + bn0 * (LPR * 16)), (short)0,
                                                        heads * (LPR * 16), kBufferWord3);
    row = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, tid * 16, 0, 0));
    ch = uidx[min(tid & 127, T - 1)];
  }
  __device__ __forceinline__ void commit(char *lds) const {
    const int tid = threadIdx.x;
    if (tid < GT * LPR) ((u32x4 *)lds)[tid] = row;
    if (tid >= 128) ((int16_t *)(lds + GT * LPR * 16))[tid - 128] = ch;   // rows, then the list
  }
  // The staged rows for the logits: full [GT][kQS] and gathered kept channels (zero beyond T), both zero beyond
  // channel 128: fp32 inputs as floats (qf, qk), bf16 inputs as packed pairs (qfp, qkp, [GT][kQS / 2] words).
  static __device__ __forceinline__ void pack(const char *lds, int T, float *qf, float *qk, uint32_t *qfp, uint32_t *qkp) {
    const B *raw = (const B *)lds;
    const int16_t *list = (const int16_t *)(lds + GT * LPR * 16);
    const int w = threadIdx.x & 127, gh = threadIdx.x >> 7;
    if (w >= kQS / 2) return;
    const int c = min(2 * w, kD - 2);   // the zeros behind a vector: channels past T and past 128
    const int i0 = list[c], i1 = list[c + 1];
    const B m0 = 2 * w < T ? (B)~(B)0 : (B)0, m1 = 2 * w + 1 < T ? (B)~(B)0 : (B)0, mf = 2 * w < kD ? (B)~(B)0 : (B)0;
#pragma unroll
    for (int g0 = 0; g0 < GT; g0 += 2) {
      const int g = g0 + gh;
      if (GT % 2 != 0 && g >= GT) break;
      const B *rg = raw + g * kD;
      const uint32_t f0 = rg[c] & mf, f1 = rg[c + 1] & mf, k0 = rg[i0] & m0, k1 = rg[i1] & m1;
      if constexpr (DT == THK_BF16) {
        qfp[g * (kQS / 2) + w] = f0 | (f1 << 16);
        qkp[g * (kQS / 2) + w] = k0 | (k1 << 16);
      }
      if constexpr (DT == THK_F32) {
        *(uint2 *)(qf + g * kQS + 2 * w) = uint2{f0, f1};
        *(uint2 *)(qk + g * kQS + 2 * w) = uint2{k0, k1};
      }
    }
  }
};

// Shape of the value loads of a tile of TR full-width rows: NL chunks per lane, chunk i of row i * RPL + lane / LPR.
template <int DT, int TR>
struct VShape {
  static constexpr int LPR = kD / Elem<DT>::VEC;     // lanes (16-byte chunks) per V row
  static constexpr int RPL = kWave / LPR;            // V rows per wave-wide load
  static constexpr int NL = TR / RPL;                // loads per lane per tile
};

// One tile whose K bytes are already in LDS (kbuf): logits, running softmax,
// acc += p.V.  vr: the tile's value rows, chunk i of a lane as VShape says (rows past a ragged tile's end
// hold zeros, as do their probabilities); vr_free is called when they have been used.
// qs: [GT][kQS] floats, entries 128..135 of every vector are zero; qp: the same
// vectors as packed bf16 pairs, [GT][kQS / 2] words (bf16 inputs only).
// TV: rows of the tile that may hold values (a tail tile has 16).
// PV = 0: value rows are full width.  PV = 1: value rows are channel-pruned; their
// bytes are in vr as they lie in memory and are walked out of LDS as described by vp.
// PV = 2: a full-width tile (the tail) of a kernel that also carries pruned-value sums, which
// follow every change of the running maximum.
// Precision of a logit.  bf16 inputs: products are exact in fp32 and the sum runs in fp32.  fp32
// inputs: the dot product and the scaling run in fp64 and the running maximum is subtracted
// before the result is rounded to fp32, so the error of exp2(z - m) does not grow with |z| (an
// fp32 logit of a few thousand -- channel scales of sigma = 2 on query and keys -- is only
// accurate to 1e-4 in absolute terms, which is the whole error budget of fp32 outputs).
template <int DT, int GT, int RA, int TR, int TV, int PV, int NV, class VrFree>
__device__ __forceinline__ void tile_compute(int shift, int nrows, int W, int ld,
                                             const float *__restrict__ qs,
                                             const uint32_t *__restrict__ qp,
                                             u32x4 (&vr)[NV], const char *kbuf,
                                             float *ps, TileState<DT, GT> &st, double scale_d, int lane,
                                             const VPruned *vp, VrFree vr_free) {
  using E = Elem<DT>;
  using ZT = typename LogitType<DT>::type;   // accumulator of a logit: float (bf16 inputs), double (fp32 inputs)
  const ZT scale = (ZT)scale_d;
  using VS = VShape<DT, TR>;
  constexpr int VEC = E::VEC, EB = E::EB;
  constexpr int LPK = kWave / TR;            // lanes that share one K row (1 or 2)
  const int vrow = lane / VS::LPR;
  const int r = lane / LPK, h = lane % LPK;

  // ---- logits: two lanes per row, each a contiguous run of granules -----------
  static_assert(LPK == 2, "two lanes share a row");
  const int rr = min(r, nrows - 1);
  int row_off = shift + rr * ld * EB;
  ZT z[GT];
#pragma unroll
  for (int g = 0; g < GT; ++g) z[g] = (ZT)0;
  if constexpr (DT == THK_BF16) {
    // bf16 pairs straight from LDS into v_dot2c_f32_bf16: products are exact, sums in fp32.
    // Keys and packed query share their byte offsets (two bytes per channel), so one offset
    // walks both, in granules of DW words.  The steps that both lanes have run without a test; what is left is one
    // masked step: lane 0 of a row takes its odd granule, lane 1 the row's last, partial one, whose elements past W
    // (row padding, or whatever follows the tile) count as zero; a lane with nothing left takes zeros.
    // (Rows of odd pitch used to be read channel by channel, four times the instructions: T = 51, 80 units x 4719
    // rows 28.9 -> 25.2 us, 152 x 93039 807 -> 746; 40 x 39096 with pruned values 90.3 -> 73.8; T = 75, 2 heads, 96 x
    // 53760 345 -> 309.)
    constexpr int DW = RA == 16 ? 4 : 2, GB = 4 * DW, EPG = 2 * DW;
    const int n_gran = W / EPG, rem = W % EPG;
    const int gran0 = (n_gran + 1) / 2, common = n_gran - gran0;
    const uint32_t sb = RA == 2 ? (uint32_t)row_off & 2u : 0u;
    if constexpr (RA == 2) row_off &= ~3;
    const char *rowp = kbuf + row_off, *qb = (const char *)qp;
    const int first = h * gran0 * GB;
    constexpr int UNR = GT == 1 ? 4 : (GT == 4 && DW == 2) ? 1 : 2;   // the widest reading ahead that registers allow
#pragma unroll UNR
    for (int i = 0; i < common; ++i) {
      uint32_t kw[DW];
      bf16_words<RA, DW>(rowp + first + i * GB, sb, kw);
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        uint32_t qw[DW];
        lds_words<DW>(qb + first + g * (kQS * 2) + i * GB, qw);
#pragma unroll
        for (int d = 0; d < DW; ++d) z[g] = dot2_bf16(kw[d], qw[d], z[g]);
      }
    }
    if (common < gran0 || rem != 0) {
      const bool any = h == 0 ? common < gran0 : rem != 0;
      const int ne = !any ? 0 : h == 0 ? EPG : rem;                 // elements that count
      const int off = any ? (h == 0 ? common : n_gran) * GB : 0;
      uint32_t kw[DW];
      bf16_words<RA, DW>(rowp + off, sb, kw);
#pragma unroll
      for (int d = 0; d < DW; ++d) kw[d] &= ne >= 2 * d + 2 ? 0xffffffffu : ne == 2 * d + 1 ? 0x0000ffffu : 0u;
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        uint32_t qw[DW];
        lds_words<DW>(qb + off + g * (kQS * 2), qw);
#pragma unroll
        for (int d = 0; d < DW; ++d) z[g] = dot2_bf16(kw[d], qw[d], z[g]);
      }
    }
  } else {
    constexpr int EPR = RA / EB;               // elements per LDS row read (one granule)
    const char *rowp = kbuf + row_off;
    const int n_gran = W / EPR;
    const int gran0 = (n_gran + 1) / 2;                      // granules of lane share 0 = trip count
    const int my_first = h * gran0;
    const int my_cnt = h == 0 ? gran0 : n_gran - gran0;
#pragma unroll 2
    for (int i = 0; i < gran0; ++i) {
      // a lane whose share is exhausted re-reads granule 0 against the zero slot of q
      const bool valid = i < my_cnt;
      const int tk = valid ? (my_first + i) * EPR : 0;
      const int tq = valid ? tk : kD;
      float f[EPR];
      lds_floats<RA>(rowp + tk * EB, f);
#pragma unroll
      for (int g = 0; g < GT; ++g)
#pragma unroll
        for (int e = 0; e < EPR; ++e) z[g] = fma_z((ZT)f[e], (ZT)qs[g * kQS + tq + e], z[g]);
    }
    for (int t = n_gran * EPR; t < W; ++t) {   // elements past the last whole granule: share 0
      const float f = E::load1(rowp, t);
      const int tq = h == 0 ? t : kD;
#pragma unroll
      for (int g = 0; g < GT; ++g) z[g] = fma_z((ZT)f, (ZT)qs[g * kQS + tq], z[g]);
    }
  }
#pragma unroll
  for (int g = 0; g < GT; ++g) z[g] += lane_swap1(z[g]);

  // ---- running softmax (base-2 exponent, scale folded in) ----------------
  // every row is held by LPK lanes, so l counts each probability LPK times
  float pr[GT];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    const ZT zs = z[g] * scale;
    const float zz = r < nrows ? (float)zs : -INFINITY;
    const float m_new = max_nn(st.m[g], wave_max(zz));   // finite: the tile has >= 1 row
    if (m_new != st.m[g]) {                             // wave-uniform; rare after the first tiles
      const float corr = __builtin_amdgcn_exp2f(st.m[g] - m_new);
      st.l[g] *= corr;
#pragma unroll
      for (int v = 0; v < VEC; ++v) st.acc[g][v] *= corr;
      if constexpr (PV != 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) st.accp[g][e] *= corr;
      }
      st.m[g] = m_new;
    }
    // fp32 inputs: z - m in fp64, then one rounding (m_new is the maximum of the ROUNDED logits, so
    // the difference may exceed 0 by half an fp32 ulp of a logit: a factor 1 + 1e-4 at most)
    if constexpr (DT == THK_F32)
      pr[g] = r < nrows ? __builtin_amdgcn_exp2f((float)(zs - (ZT)m_new)) : 0.f;
    else
      pr[g] = __builtin_amdgcn_exp2f(zz - m_new);
    st.l[g] += pr[g];
  }
  // probabilities to LDS as [row][GT]
  if constexpr (GT == 4) {
    *(float4 *)(ps + r * 4) = make_float4(pr[0], pr[1], pr[2], pr[3]);
  } else if constexpr (GT == 2) {
    *(float2 *)(ps + r * 2) = make_float2(pr[0], pr[1]);
  } else {
#pragma unroll
    for (int g = 0; g < GT; ++g) ps[r * GT + g] = pr[g];
  }
  if constexpr (PV == 1) {
    // ---- accp += p . V_pruned: value bytes to LDS, then 4 kept channels per lane ----------
    k_commit<NV>(vr, vp->vbuf, lane);
    vr_free();
    wave_sync_lds();
    // Rows r0 + rsub, r0 = 0, rpw, 2 rpw, ...; NS steps are read before they are used.  Nothing
    // branches: a row past the tile's end takes the bytes of the tile's last row and a weight of 0
    // -- rows nrows .. TR - 1 of ps were written as 0 above, and rows TR .. TR + kPsPad - 1 are
    // zero for the whole kernel (four steps of at most 8 rows may start at row nrows - 1).
    constexpr int NS = GT == 1 ? 4 : 2;   // steps read before they are used (registers)
    const int rowb = vp->ld * EB;
    const int vstep = vp->rpw * rowb, pstep = vp->rpw * GT;
    int voff = vp->shift + vp->col * 4 * EB + vp->rsub * rowb;
    const int vlast = vp->shift + vp->col * 4 * EB + (nrows - 1) * rowb;
    const float *pp = ps + vp->rsub * GT;
    for (int r0 = 0; r0 < nrows; r0 += NS * vp->rpw) {
      float f[NS][4], pg[NS][GT];
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const char *vrow = vp->vbuf + min(voff, vlast);
        if constexpr (DT == THK_BF16) {
          const uint2 w = *(const uint2 *)vrow;
          f[i][0] = __uint_as_float(w.x << 16); f[i][1] = __uint_as_float(w.x & 0xffff0000u);
          f[i][2] = __uint_as_float(w.y << 16); f[i][3] = __uint_as_float(w.y & 0xffff0000u);
        } else {
          const float4 w = *(const float4 *)vrow;
          f[i][0] = w.x; f[i][1] = w.y; f[i][2] = w.z; f[i][3] = w.w;
        }
        if constexpr (GT == 4) {
          const float4 t4 = *(const float4 *)pp;
          pg[i][0] = t4.x; pg[i][1] = t4.y; pg[i][2] = t4.z; pg[i][3] = t4.w;
        } else if constexpr (GT == 2) {
          const float2 t2 = *(const float2 *)pp;
          pg[i][0] = t2.x; pg[i][1] = t2.y;
        } else {
#pragma unroll
          for (int g = 0; g < GT; ++g) pg[i][g] = pp[g];
        }
        voff += vstep;
        pp += pstep;
      }
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int g = 0; g < GT; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) st.accp[g][e] = fmaf(pg[i][g], f[i][e], st.accp[g][e]);
    }
  } else {
  wave_sync_lds();

  // ---- acc += p . V --------------------------------------------------------
#pragma unroll
  for (int i = 0; i < VShape<DT, TV>::NL; ++i) {
    const int row = i * VS::RPL + vrow;
    float f[VEC];
    E::unpack(vr[i], f);
    float pv[GT];
    if constexpr (GT == 4) {
      const float4 t4 = *(const float4 *)(ps + row * 4);
      pv[0] = t4.x; pv[1] = t4.y; pv[2] = t4.z; pv[3] = t4.w;
    } else if constexpr (GT == 2) {
      const float2 t2 = *(const float2 *)(ps + row * 2);
      pv[0] = t2.x; pv[1] = t2.y;
    } else {
#pragma unroll
      for (int g = 0; g < GT; ++g) pv[g] = ps[row * GT + g];
    }
#pragma unroll
    for (int g = 0; g < GT; ++g)
#pragma unroll
      for (int v = 0; v < VEC; ++v) st.acc[g][v] = fmaf(pv[g], f[v], st.acc[g][v]);
  }
  vr_free();
  }
  wave_sync_lds();   // ps and kbuf are rewritten by the next tile
}

// ---- cross-block hand-off of the split records (n_split > 1, at most kFuseMaxSplit pieces) ----
// The block that finishes LAST for a (unit, head group) merges the group's split records itself,
// so the call needs no second launch.  No read-modify-write is involved (the blocks of a group
// finish together, and a contended compare-and-swap loop costs a memory round trip per
// contender): every block has a FLAG word per (group, split).  A block
//   1. stores its record with device-scope relaxed atomic stores (they reach the coherence
//      point themselves: the L2 caches of the XCDs are not coherent with each other, and a
//      device-scope fence would write back a whole L2) and waits until they are acknowledged,
//   2. stores the call's nonce into its own flag and waits for that acknowledgement,
//   3. loads the group's flags: if all of them hold the nonce it merges.
// The block whose flag store is performed last finds all flags set, and by 1. every record is
// then visible to it.  Blocks that finish within a round trip of each other may both find all
// flags set: both merge, in the same order, and store the same bits.  A merging block clears the
// flags afterwards, so that a replay of the same launch from a graph, which carries the same
// nonce, starts clean; whatever else the flag words held before the call (another call's nonce,
// other data of the workspace) is not the nonce: 64 bits drawn per call.
constexpr int kFuseMaxSplit = 16;

template <class V2>   // two floats, 8-byte aligned
__device__ inline void pub_store_f32x2(float *p, V2 v) {
  __hip_atomic_store((unsigned long long *)p, __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Merge of the four waves' softmax states (mrg: [GT][130] floats per wave, wstride floats from
// wave to wave, in LDS, complete and visible to the block): the output row of every query head
// the block serves, or this split's state record -- and, where the call merges inside the
// launch, the output rows again, from all records, by the block that arrives last.
// grp: index of the block's (unit, head group) among all of the call's; s_last: one int of LDS.
// Latency bounds it: LDS, two acknowledgements, the flags, the records, one after the other, and every
// instruction in between.  One pass over a head's four states by one wave (two channels a lane) instead of a loop
// over channels, 8-byte stores, and all of a wave's records in one trip: end of the tiles to the record's store 0.75 ->
// 0.32 us; whole calls of 7 to 15 us 2 to 9 % shorter, 40 random decode calls 1.04x.
template <int DT, int GT>
__device__ __forceinline__ void block_merge_store(const float *mrg, int wstride, const DecodeArgs &a,
                                                  int64_t bn0, int sp, int heads, int64_t grp, int *s_last) {
  using E = Elem<DT>;
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const bool fused = GT <= 4 && a.arrive != nullptr;   // (blocks of eight heads have a launch for it: merges_in_launch)
  int lane = threadIdx.x % kWave;
  asm volatile("" : "+v"(lane));   // a copy of its own: nothing made from it is kept through the tile loops (registers)
  const int wave = uniform(threadIdx.x / kWave);
  // (a weight below 2^-126 is 0, as in the tiles; the library's exp2, which keeps a denormal, takes calls of 7 to 11 us
  // 1 to 2 % longer, and the error against 64 bits over 240 random calls is no larger without it: bf16 1.000, fp32 0.90 of it)
  auto weight = [](float m, float M) { return m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M); };
  auto store_out = [&](size_t bn, float A0, float A1, float L) { E::store2(a.out, bn * kD + 2 * lane, A0 / L, A1 / L); };
  // A wave takes a head, a lane two of its channels; heads <= GT of the block's slots are in use.
#pragma unroll
  for (int g0 = 0; g0 < GT; g0 += 4) {
    const int g = g0 + wave;
    if (g >= heads) break;
    f32x2 ml[4], av[4];   // (maximum, sum) and two channels of the four waves
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float *rec = mrg + (size_t)w * wstride + g * (kD + 2);
      ml[w] = *(const f32x2 *)rec;
      av[w] = *(const f32x2 *)(rec + 2 + 2 * lane);
    }
    // (a whole number at or above the maxima: what a record is weighed by against others, here and in k_decode_merge, is an
    // exact power of two, and a wave's state is the only one with a rounded weight, in however many pieces.  Mean error against 64
    // bits, the maximum itself and up to 16 pieces / so and 64-row ones: 15 fp32 calls of up to 2048 rows, 160 inputs each, 1.20e-7 / 1.18e-7;
    // 10 calls of 27 to 64 pieces in both 1.51e-7 / 1.30e-7; single inputs differ either way, one by 1.07e-7 / 1.57e-7)
    const float M = ceilf(fmaxf(fmaxf(ml[0][0], ml[1][0]), fmaxf(ml[2][0], ml[3][0])));
    float Lsum = 0.f, A0 = 0.f, A1 = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float wgt = weight(ml[w][0], M);
      Lsum = fmaf(ml[w][1], wgt, Lsum);
      A0 = fmaf(av[w][0], wgt, A0);
      A1 = fmaf(av[w][1], wgt, A1);
    }
    const size_t bn = (size_t)(bn0 + g);
    if (a.n_split == 1) {
      store_out(bn, A0, A1, Lsum);
    } else {
      float *rec = a.ws + (bn * a.n_split + sp) * (kD + 2);
      const f32x2 acc = {A0, A1}, head = {M, Lsum};
      if (fused) {
        pub_store_f32x2(rec + 2 + 2 * lane, acc);
        if (lane == 0) pub_store_f32x2(rec, head);
      } else {
        *(f32x2 *)(rec + 2 + 2 * lane) = acc;
        if (lane == 0) *(f32x2 *)rec = head;
      }
    }
  }
  if (a.n_split == 1 || !fused) return;

  // ---- the group's last block merges: m = max m_i, l = sum l_i 2^(m_i - m) by the wave's fixed tree, acc likewise in
  // split order (the result does not depend on who arrives last) ---------------------------
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's record stores are acknowledged
  __syncthreads();                                   // ... and every wave's
  unsigned long long *flags = a.arrive + (size_t)grp * a.n_split;
  if (threadIdx.x < kWave) {
    if (threadIdx.x == 0)
      __hip_atomic_store(flags + sp, a.nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the flag is out before the flags are read
    const unsigned long long f =
        (int)threadIdx.x < a.n_split
            ? __hip_atomic_load(flags + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
            : a.nonce;
    const bool all = __all(f == a.nonce);
    if (threadIdx.x == 0) *s_last = all ? 1 : 0;
  }
  __syncthreads();
  if (*s_last == 0) return;
  // Again a head per wave, two channels per lane; lane i also holds piece i's maximum and sum, whose
  // weight reaches the others through v_readlane.  One trip to memory for all of it: the loads go
  // through a buffer resource that ends with the last piece, so that those of absent pieces return 0
  // (little code matters here as much as few trips).
  constexpr int kRecB = (kD + 2) * 4, kDeviceScope = 16;   // bytes from piece to piece; sc1, the scope of the stores
  if (wave < heads) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr((const char *)(a.ws + (size_t)(bn0 + wave) * a.n_split * (kD + 2))),
                                                        (short)0, a.n_split * kRecB, kBufferWord3);
    auto load2 = [&](int off) {
      return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, kDeviceScope));
    };
    const f32x2 ml = load2(lane * kRecB);
    f32x2 av[kFuseMaxSplit];
#pragma unroll
    for (int i = 0; i < kFuseMaxSplit; ++i) av[i] = load2(i * kRecB + 8 + lane * 8);
    const float m = lane < a.n_split ? ml[0] : -INFINITY;
    const float wgt = weight(m, wave_max(m));
    const float Lsum = wave_sum(ml[1] * wgt);
    float A0 = 0.f, A1 = 0.f;
#pragma unroll
    for (int i = 0; i < kFuseMaxSplit; ++i) {
      const float wi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wgt), i));
      A0 = fmaf(av[i][0], wi, A0);
      A1 = fmaf(av[i][1], wi, A1);
    }
    store_out((size_t)(bn0 + wave), A0, A1, Lsum);
  }
  if ((int)threadIdx.x < a.n_split)
    __hip_atomic_store(flags + threadIdx.x, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every argument a block needs in front of its first loads, asked for at once.  Left to itself the compiler
// loads an argument where it is first used, and each such load is a trip of 0.2 us of its own.
__device__ __forceinline__ void want_arguments(const DecodeArgs &a, int groups) {
  asm volatile("" ::"s"(a.q), "s"(a.kp), "s"(a.v), "s"(a.kt), "s"(a.vt), "s"(a.idx), "s"(a.S), "s"(a.rows_per_split), "s"(a.unit_rows),
               "s"(a.units), "s"(a.split_inv), "s"(groups));
  asm volatile("" ::"s"(a.unified_v), "s"(a.T), "s"(a.ldk), "s"(a.G), "s"(a.s_tail), "s"(a.s_tail_cap), "s"(a.n_split), "s"(a.T_v),
               "s"(a.ld_v));
}

// Which (unit, piece, head group) a workgroup takes.  Where the heads of a KV head need several
// groups, the blocks that read the SAME keys and values are 8 workgroup numbers apart: workgroup i
// runs on XCD i % 8, so they share an L2 and are dispatched one after the other, and all but the
// first find the rows there.  With the groups n_split numbers apart: bf16, 64 units x 16384 rows x 12
// heads, 4 pieces, 136 -> 110 us; 28 units x 20000 rows x 16 heads, 9 pieces, 76.0 -> 59.2 us; where
// n_split is a multiple of 8 the XCD was the same already and nothing changes (16 units x 32768 rows x
// 16 heads 62 / 61 us, fp32 64 units x 9527 rows x 8 heads 137 / 135-143 us).
// False: a surplus workgroup of the last eight, of which the grid ends with the last one that has work (it
// may have up to 2^24 workgroups, and calls just below that are served).  (fewer than 2^31 blocks: 32-bit divisions)
struct DecodeWork {
  uint32_t u;   // (layer, batch, KV head)
  int sp, gi;
};
template <bool MANY>   // a unit may have more than one head group
__device__ __forceinline__ bool decode_block_work(const DecodeArgs &a, int groups, DecodeWork &w) {
  uint32_t piece = blockIdx.x;   // (unit, piece of S)
  w.gi = 0;
  if (MANY && groups > 1) {
    const uint32_t slot = piece / kXcds, round = slot / (uint32_t)groups;
    w.gi = (int)(slot - round * (uint32_t)groups);
    piece = round * kXcds + piece % kXcds;
  }
  w.u = (uint32_t)((piece * a.split_inv) >> kSplitShift);
  w.sp = (int)(piece - w.u * (uint32_t)a.n_split);
  return !MANY || w.u < (uint32_t)a.units;
}
inline unsigned decode_grid(const DecodeArgs &a, int groups) {
  const int64_t pieces = a.units * a.n_split, last = pieces % kXcds;   // last: pieces of an eight that is not full
  return (unsigned)(groups == 1 || last == 0 ? pieces * groups : (pieces - last) * groups + (groups - 1) * kXcds + last);
}

// The tiles of one wave in the order it takes them: every fourth pruned tile of its piece, then its share
// of the unit's tail tiles, which are dealt out from the last piece and the last wave on, for these have the
// fewest rows.  All members are wave-uniform; a tile that is not there has no bytes.
constexpr int kTileRows = 32;
struct Tile {
  enum { kPruned, kTail, kNone };
  int kind, nrows;
  ByteRange k, v;
};
template <int EB, int VP>
struct WaveTiles {
  static constexpr int TR = kTileRows, kRowB = kD * EB;
  const char *tail_k, *tail_v;
  ByteRange kt, vt;      // the next pruned tile (a wave's pruned tiles are 128 rows apart, a multiple of 16 bytes in any pitch: they share their shift)
  size_t k_step, v_step;
  int k_last, v_last, nr_last, nt_p, nt_t, ti, tj, tj_step, s_tail;
  __device__ __forceinline__ WaveTiles(const DecodeArgs &a, int64_t u, int sp, int wave) {
    const int64_t s0 = min(a.S, (int64_t)sp * a.rows_per_split);
    const int64_t s1 = min(a.S, s0 + a.rows_per_split);
    nt_p = (int)((s1 - s0 + TR - 1) / TR);
    nr_last = (int)(s1 - s0 - (int64_t)(nt_p - 1) * TR);   // rows of the piece's last tile
    s_tail = a.s_tail;
    nt_t = (s_tail + kTailRows - 1) / kTailRows;
    const size_t row = (size_t)u * a.unit_rows + s0 + (size_t)wave * TR;   // first K_pruned / V row of this wave
    kt = flat_rows<EB>(a.kp, row * a.ldk * EB, TR, a.T, a.ldk);
    k_last = (kt.shift + ((nr_last - 1) * a.ldk + a.T) * EB + 15) & ~15;
    k_step = (size_t)a.ldk * (4 * TR * EB);
    if constexpr (VP) {
      vt = flat_rows<EB>(a.v, row * a.ld_v * EB, TR, a.T_v, a.ld_v);
      v_last = (vt.shift + ((nr_last - 1) * a.ld_v + a.T_v) * EB + 15) & ~15;
      v_step = (size_t)a.ld_v * (4 * TR * EB);
    } else {
      vt = ByteRange{(const char *)a.v + row * kRowB, TR * kRowB, 0};
      v_last = nr_last * kRowB;
      v_step = 4 * TR * kRowB;
    }
    // the tail's value rows: a buffer of their own, or the rows that follow row S in v
    const size_t trow = (size_t)u * a.s_tail_cap;
    tail_k = (const char *)a.kt + trow * kRowB;
    tail_v = a.unified_v ? (const char *)a.v + ((size_t)u * a.unit_rows + a.S) * kRowB : (const char *)a.vt + trow * kRowB;
    ti = wave;
    tj = (a.n_split - 1 - sp) + (3 - wave) * a.n_split;
    tj_step = 4 * a.n_split;
  }
  __device__ __forceinline__ Tile next() {
    Tile t;
    if (ti < nt_p) {
      const bool last = ti == nt_p - 1;
      t.kind = Tile::kPruned;
      t.nrows = last ? nr_last : TR;
      t.k = ByteRange{kt.base, last ? k_last : kt.bytes, kt.shift};
      t.v = ByteRange{vt.base, last ? v_last : vt.bytes, vt.shift};
      kt.base += k_step;
      vt.base += v_step;
      ti += 4;
    } else {
      const int j0 = min(tj, nt_t) * kTailRows, n = max(min(kTailRows, s_tail - j0), 0);
      t.kind = tj < nt_t ? Tile::kTail : Tile::kNone;
      t.nrows = n;
      t.k = ByteRange{tail_k + (size_t)j0 * kRowB, n * kRowB, 0};
      t.v = ByteRange{tail_v + (size_t)j0 * kRowB, n * kRowB, 0};
      tj += tj_step;
    }
    return t;
  }
};

// KB: 16-byte K chunks a lane may have to stage for one TR-row pruned tile.
// WPE: resident waves per SIMD the register budget is set for.
// VP = 1: the value rows of the pruned segment hold only the T_v kept channels (a.v is
// V_pruned with rows a.ld_v elements apart, a.idx_v lists the channels).  Their bytes are staged
// like the key bytes (KB chunks per lane, the class is chosen for the wider of the two), into the
// same wave-private LDS slab once the tile's key bytes have been consumed, and each lane
// accumulates 4 kept channels; at the end the sums are scattered to their channels.  The tail
// keeps full-width value rows.
template <int DT, int GT, int RA, int KB, int TR, int WPE, int VP = 0>
__global__ __launch_bounds__(256, WPE) void k_decode(DecodeArgs a, int groups, int kbuf_bytes) {
  using E = Elem<DT>;
  using VS = VShape<DT, TR>;
  constexpr int VEC = E::VEC, EB = E::EB, LPR = VS::LPR, LPK = kWave / TR;
  extern __shared__ uint4 smem[];
  // the gathered query channels (0 beyond T) and the full query: [GT][kQS] floats each (fp32 inputs), or as
  // packed pairs, [GT][kQS / 2] words each (bf16 inputs)
  constexpr bool F32 = DT == THK_F32;
  constexpr int QW = GT * kQS * EB / 4;          // words per copy
  uint32_t *qkw = (uint32_t *)smem, *qfw = qkw + QW;
  float *qk = F32 ? (float *)qkw : nullptr, *qf = F32 ? (float *)qfw : nullptr;
  uint32_t *qkp = F32 ? nullptr : qkw, *qfp = F32 ? nullptr : qfw;
  float *mrg = (float *)(qfw + QW);              // [4][GT][130] per-wave states for the final merge
  char *wbase = (char *)(mrg + 4 * GT * (kD + 2));
  __shared__ int s_last;
  const int lane = threadIdx.x % kWave;
  const int wave = uniform(threadIdx.x / kWave);   // tile counts and branches stay scalar
  const int wstride = kbuf_bytes + GT * (TR + (VP ? kPsPad : 0)) * 4;
  char *kbuf = wbase + (size_t)wave * wstride;
  float *ps = (float *)(kbuf + kbuf_bytes);
  VPruned vpd;
  vpd.vbuf = kbuf;   // the key bytes of a tile are consumed before its value bytes are staged
  vpd.shift = 0;
  vpd.ld = a.ld_v;
  {
    const int lprv = VP ? (a.T_v + 3) / 4 : 1;          // lanes per value row, <= 32
    vpd.rpw = min(kWave / lprv, 8);
    vpd.col = lane % lprv;
    vpd.active = lane / lprv < vpd.rpw;
    vpd.rsub = vpd.active ? lane / lprv : 0;   // idle lanes repeat row group 0; their sums are dropped
  }

  want_arguments(a, groups);
  DecodeWork work;
  if (!decode_block_work<GT == 4>(a, groups, work)) return;   // fewer: all heads of a unit
  const int sp = work.sp, gi = work.gi;
  const int64_t u = work.u;
  const int G = a.G;
  const int64_t bn0 = u * G + (int64_t)gi * GT;   // first query head served (heads of unit u: u*G ..)
  // the unit's last block may have fewer than GT heads left: the other slots carry a zero query
  // (their logits are 0, their output is never stored)
  const int hb = min(GT, G - gi * GT);

  QueryStage<DT, GT> qst;
  qst.issue(a.q, (size_t)bn0, hb, a.idx + (size_t)u * a.T, a.T);

  // the first tile's key and value bytes start moving before anything is waited for
  WaveTiles<EB, VP> tiles(a, u, sp, wave);
  constexpr int VB = VP ? KB : VS::NL;
  constexpr int TB = kTailRows * kD * EB / (16 * kWave);   // chunks per lane of a tail tile's keys, and of its values
  static_assert(TB <= KB && TB <= VB, "a tail tile fits the staging registers");
  u32x4 kr[KB], vr[VB];
  Tile nt = tiles.next();
  tile_issue<KB>(kr, nt.k.base, nt.k.bytes, lane);
  tile_issue<VB>(vr, nt.v.base, nt.v.bytes, lane);

  // query: gather the kept channels (Sec. 3.3: the query is pruned with the stored mask)
  qst.commit((char *)mrg);
  __syncthreads();
  QueryStage<DT, GT>::pack((const char *)mrg, a.T, qf, qk, qfp, qkp);
  if constexpr (VP) {
    for (int o = lane; o < GT * kPsPad; o += kWave) ps[GT * TR + o] = 0.f;
  }
  __syncthreads();

  TileState<DT, GT> st;
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    st.m[g] = -INFINITY; st.l[g] = 0.f;
#pragma unroll
    for (int v = 0; v < VEC; ++v) st.acc[g][v] = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) st.accp[g][e] = 0.f;
  }

  // ---- the bytes of this wave's next tile are in flight while the current one is computed:
  // pruned tiles, then the wave's share of the unpruned tail (full-width keys, full query)
  while (nt.kind == Tile::kPruned) {
    const Tile t = nt;
    nt = tiles.next();
    k_commit<KB>(kr, kbuf, lane);
    tile_issue<KB>(kr, nt.k.base, nt.k.bytes, lane);
    wave_sync_lds();
    vpd.shift = t.v.shift;
    tile_compute<DT, GT, RA, TR, TR, VP>(t.k.shift, t.nrows, a.T, a.ldk, qk, qkp, vr, kbuf, ps, st, a.scale_log2_d, lane, &vpd,
                                         [&]() { tile_issue<VB>(vr, nt.v.base, nt.v.bytes, lane); });
  }
  while (nt.kind == Tile::kTail) {
    const Tile t = nt;
    nt = tiles.next();
    k_commit<TB>(kr, kbuf, lane);
    tile_issue<TB>(kr, nt.k.base, nt.k.bytes, lane);
    wave_sync_lds();
    tile_compute<DT, GT, 16, TR, kTailRows, 2 * VP>(0, t.nrows, kD, kD, qf, qfp, vr, kbuf, ps, st, a.scale_log2_d, lane, &vpd,
                                                    [&]() { tile_issue<TB>(vr, nt.v.base, nt.v.bytes, lane); });
  }

  // ---- wave state -> LDS ---------------------------------------------------
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    const float lt = wave_sum(st.l[g]) * (1.0f / LPK);
#pragma unroll
    for (int off = LPR; off < kWave; off <<= 1)
#pragma unroll
      for (int v = 0; v < VEC; ++v) st.acc[g][v] += __shfl_xor(st.acc[g][v], off);
    float *rec = mrg + (size_t)(wave * GT + g) * (kD + 2);
    if (lane == 0) { rec[0] = st.m[g]; rec[1] = lt; }
    if (lane < LPR)
#pragma unroll
      for (int v = 0; v < VEC; ++v) rec[2 + lane * VEC + v] = st.acc[g][v];
  }
  if constexpr (VP) {
    // the sums over the pruned rows go to their channels, one row-within-step group at a time
    const int16_t *uidv = a.idx_v + (size_t)u * a.T_v;
    int cv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int t = vpd.col * 4 + e;
      cv[e] = t < a.T_v ? uidv[t] : -1;
    }
    for (int rs = 0; rs < vpd.rpw; ++rs) {
      wave_sync_lds();
      if (vpd.active && vpd.rsub == rs) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (cv[e] >= 0) {
#pragma unroll
            for (int g = 0; g < GT; ++g) mrg[(size_t)(wave * GT + g) * (kD + 2) + 2 + cv[e]] += st.accp[g][e];
          }
        }
      }
    }
  }
  __syncthreads();

  block_merge_store<DT, GT>(mrg, GT * (kD + 2), a, bn0, sp, hb, u * groups + gi, &s_last);
}

// ---- host side: pick the instantiation for a shape --------------------------
struct DecodeLaunch {
  int ra;      // byte alignment of K_pruned rows (16, 8, 4, 2)
  int kb;      // staged chunks per lane needed for one tile
};

template <int DT>
inline DecodeLaunch decode_launch_params(const DecodeArgs &a, int tr) {
  constexpr int eb = Elem<DT>::EB;
  DecodeLaunch p;
  // every row starts at a multiple of ld * eb bytes from the 16-byte aligned base
  const size_t rowb = (size_t)a.ldk * eb;
  p.ra = 16;
  while (rowb % p.ra) p.ra >>= 1;
  const int max_nch = (int)((tr * rowb + (p.ra == 16 ? 0 : 14) + 15) / 16);
  p.kb = (max_nch + kWave - 1) / kWave;
  return p;
}

template <int DT, int GT, int RA, int KB, int TR, int WPE, int VP>
inline hipError_t decode_launch_one(const DecodeArgs &a, int groups, hipStream_t st) {
  constexpr int eb = Elem<DT>::EB;
  int kbuf = KB * kWave * 16;                      // every staged chunk has an LDS slot
  const int tailbuf = kTailRows * kD * eb;
  if (kbuf < tailbuf) kbuf = tailbuf;
  const size_t lds = (size_t)2 * GT * kQS * eb + (size_t)4 * GT * (kD + 2) * 4 + 4 * ((size_t)kbuf + GT * (TR + (VP ? kPsPad : 0)) * 4);
  const dim3 grid(decode_grid(a, groups)), block(256);
  {
    static DynLds set;   // one per instantiation
    const hipError_t e = ensure_dyn_lds((const void *)k_decode<DT, GT, RA, KB, TR, WPE, VP>, lds, set);
    if (e != hipSuccess) return e;
  }
  void *kargs[] = {(void *)&a, (void *)&groups, (void *)&kbuf};
  const hipError_t e = launch_main_kernel((const void *)k_decode<DT, GT, RA, KB, TR, WPE, VP>, grid, block, kargs, lds, st);
  return e != hipSuccess ? e : hipGetLastError();
}

template <int DT, int GT, int KB, int TR, int WPE, int VP>
inline hipError_t decode_launch_ra(const DecodeArgs &a, int ra, int groups, hipStream_t st) {
  if (ra == 16) return decode_launch_one<DT, GT, 16, KB, TR, WPE, VP>(a, groups, st);
  if (ra == 8) return decode_launch_one<DT, GT, 8, KB, TR, WPE, VP>(a, groups, st);
  if (ra == 4) return decode_launch_one<DT, GT, 4, KB, TR, WPE, VP>(a, groups, st);
  if constexpr (DT == THK_BF16) {
    if (ra == 2) return decode_launch_one<DT, GT, 2, KB, TR, WPE, VP>(a, groups, st);
  }
  return hipErrorInvalidValue;
}

// Tiles of 32 rows: two lanes share a key row, waves stay light (4 per SIMD when
// K staging is narrow and at most two query heads share the block, else 3).
template <int DT, int GT, int VP = 0>
hipError_t decode_launch_gt(const DecodeArgs &a, int groups, hipStream_t st) {
  constexpr int TR = 32;
  DecodeLaunch p = decode_launch_params<DT>(a, TR);
  if constexpr (VP) {
    // the value tile is staged with the same chunk count: size the class for the wider of the two
    const int kbv = (int)((TR * (size_t)a.ld_v * Elem<DT>::EB + 15 + 15) / 16 + kWave - 1) / kWave;
    if (kbv > p.kb) p.kb = kbv;
  }
  constexpr int KBN = (DT == THK_BF16) ? 5 : 10;   // T <= 79
  constexpr int KBW = (DT == THK_BF16) ? 9 : 17;   // up to ld_keep = 128
  // fp32 stages twice as many registers per tile: one wave per SIMD fewer than bf16 (at four
  // the fp32 kernels spilled 27-63 registers and ran at 3.7 TB/s instead of 5.3)
  constexpr int WN = DT == THK_F32 ? ((VP || GT == 4) ? 2 : 3) : (GT <= 2 ? 4 : 3);
  constexpr int WW = DT == THK_F32 ? 2 : (VP ? 2 : 3);
  if (p.kb <= KBN) return decode_launch_ra<DT, GT, KBN, TR, WN, VP>(a, p.ra, groups, st);
  if (p.kb <= KBW) return decode_launch_ra<DT, GT, KBW, TR, WW, VP>(a, p.ra, groups, st);
  return hipErrorInvalidValue;
}

}  // namespace thk
