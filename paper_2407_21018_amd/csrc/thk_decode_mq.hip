// Decode attention over the pruned key cache for bf16 caches whose KV heads serve three or more
// query heads each (Sec. 3.3, Fig. 2; attention formula of Sec. 3.2) -- gfx950, wave64.
//
// With four query heads per key row the two products of a tile are skinny matrix products
// (4 x T by T x 32, then 4 x 32 by 32 x 128) and go to the matrix cores as batches of 4 x 4
// blocks (v_mfma_f32_4x4x4_16B_bf16: 16 independent blocks per instruction; lane 4 b + x holds
// row x of A_b, column x of B_b and column x of D_b).  Work split, tile size, staging of the key
// bytes, split records and the final merge are those of k_decode; what differs is one tile:
//
//   logits   block b <-> key rows 4 (b % 8) .. + 3 and one half (b / 8) of the kept channels.
//            A_b = four key rows x four channels, 8 bytes per lane straight from the staged
//            bytes in LDS; B_b = the four query heads' same four channels; D_b[i][j] is the
//            partial logit of row i and head j.  The blocks of one half walk the channel chunks
//            in rotated order so that the row reads spread over the LDS banks; the two halves
//            are added with one cross-half exchange.
//   softmax  lane 4 b + j owns head j and four rows: the running maximum is a per-lane scalar,
//            reduced over the lanes of equal j.  A probability is split into bf16 terms of 8 bits
//            each: two (p = hi + lo, exact to 2^-16) for key rows a multiple of 4 elements apart;
//            three, which are all of p's 24 bits, for other pitches: those calls came from the
//            general kernel, whose product with V is fp32.  The third term costs a half more
//            matrix instructions and probability reads in the second product (64 units, T = 51:
//            32768 rows, G = 4 123.4 -> 124.2 us, G = 8 122.7 -> 124.4; 8191 rows, G = 8, 76 value
//            channels 32.2 -> 34.6).
//   values   block b <-> output channels 4 b .. + 3 (two instructions cover 128 channels).
//            A_b = the four heads' probabilities of four rows, the same for every block (read
//            back from an LDS line of 256 bytes per term); B_b = four value rows x four channels, which is a
//            transposed read of the row-major value tile: ds_read_b64_tr_b16 out of LDS, where
//            the tile is staged with the two 128-byte halves of odd rows swapped (the four rows
//            of one read then cover all banks).  D_b[i][j] accumulates head i, channel 4 b + j:
//            lane l ends with channels l and 64 + l of all four heads.
//   VP = 1   channel-pruned value rows (T_v kept channels, rows ld_v elements apart): their bytes
//            are staged like the key bytes, as a flat range, and the same transposing reads walk
//            them with the row pitch ld_v; lane l then sums kept channels l and 64 + l, which
//            are scattered to their output channels at the end.  The tail keeps full-width rows.
//   NH = 2   eight query heads per KV head in one block: two groups of four share every key
//            and value operand read from LDS; queries, probabilities and accumulators double.
//
// The kernel streams at the rate of a plain read of the same bytes only while its instruction
// stream stays short (a wave64 instruction holds its SIMD for four cycles, and three or four
// waves share one): the wave index is made uniform so that tile counts, row counts and their
// branches live in scalar registers; a whole tile (32 rows, all but a block's last) takes
// a straight-line path -- the eight 4-row
// steps of the second product without a test between them so that later reads overlap earlier
// products; the logit loop covers the chunks that both halves have without masks or range checks, and
// what is left of a row (an odd chunk, a partial one) is one masked step behind it; tiles of at
// most 4 KB of keys get a staging class of their own (no fifth, duplicate chunk).  Together: 805 MB (64 units x 32768 rows, G = 4) 130.4 -> 125.9 us, 403 MB
// (8 units x 131072 rows) 68.0 -> 65.0 us; with no arithmetic at all the same loads take 123 us.
#include <stdlib.h>

#include <type_traits>

#include "thk_decode_impl.h"

namespace thk {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMqRows = kTileRows;                // rows per tile
constexpr int kMqVBytes = kMqRows * kD * 2;       // a value tile in LDS
constexpr int kMqVChunks = kMqVBytes / 16 / kWave;   // 16-byte value chunks per lane and tile

struct MqState {
  float m;        // running maximum of this lane's head (lane % 4), log2 domain
  float l;        // this lane's share of its head's probability sum
  f32x4 acc[2];   // acc[h][i]: head i, channel 64 h + lane
  f32x4 accp[2];  // channel-pruned values only: accp[h][i]: head i, kept channel number 64 h + lane
};

__device__ __forceinline__ f32x4 mfma4(s16x4 a, s16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, b, c, 0, 0, 0);
}

// x combined over the lanes of equal lane % 4 inside each half of the wave (rotations by 4 and 8
// inside the 16-lane rows, then the neighbouring row).
template <bool MAX>
__device__ __forceinline__ float quad_column_reduce(float x) {
  float y = dpp_move<0x124, 0xf>(x, x);   // row_ror:4
  x = MAX ? max_nn(x, y) : x + y;
  y = dpp_move<0x128, 0xf>(x, x);         // row_ror:8
  x = MAX ? max_nn(x, y) : x + y;
  const LanePair p = pair16(x);
  return MAX ? max_nn(p.a, p.b) : p.a + p.b;
}

// Value rows of a tile (chunk j * 64 + lane is 16 bytes of row 4 j + lane / 16) into the slab: rows 256 bytes
// apart, the two halves of odd rows swapped.
template <int N, int M>
__device__ __forceinline__ void mq_v_commit(const u32x4 (&vr)[M], char *slab, int lane) {
  const int rsub = lane >> 4, col = (lane & 15) ^ ((rsub & 1) << 3);
#pragma unroll
  for (int j = 0; j < N; ++j) *(u32x4 *)(slab + (4 * j + rsub) * 256 + col * 16) = vr[j];
}

// Logits of a tile whose key bytes are in the slab, for NH groups of four heads.  qrow: this lane's
// head of the first group as packed bf16, zero from channel W on (the same head of the next group
// follows 4 * kQS / 2 words later).  d[g] receives,
// in both halves of the wave, the dot products of rows 4 ((lane / 4) % 8) + r, r = 0 .. 3, with
// head 4 g + lane % 4: the key operand is read once for all groups.
// W: elements per key row.
// AL: alignment of the rows' start in bytes.  8: a chunk is one read.  4 (T = 70, 78, ...): two words.
// 2 (dense rows of an odd T: 51 is lambda = 0.6): three words from the boundary below, of which a
// lane takes the upper or the lower halves -- its row starts on a word or in the middle of
// one, the same for every chunk of the row.
template <int AL>
__device__ __forceinline__ uint2 key_chunk(const char *p, uint32_t shift_bytes) {
  if constexpr (AL == 8) {
    return *(const uint2 *)p;
  } else {
    const uint32_t *w = (const uint32_t *)p;
    if constexpr (AL == 4) return uint2{w[0], w[1]};
    const uint32_t a = w[0], b = w[1], c = w[2];
    return uint2{__builtin_amdgcn_alignbyte(b, a, shift_bytes), __builtin_amdgcn_alignbyte(c, b, shift_bytes)};
  }
}
template <int NH, int AL>
__device__ __forceinline__ void mq_logits(const char *slab, int shift, int nrows, int W, int pitch_bytes,
                                          const uint32_t *qrow, int lane, f32x4 (&d)[NH]) {
  const int b = lane >> 2, x = lane & 3, half = b >> 3, bb = b & 7;
  int row_off = shift + __umul24(min(4 * bb + x, nrows - 1), pitch_bytes);
  const uint32_t sb = AL == 2 ? (uint32_t)row_off & 2u : 0u;
  if constexpr (AL == 2) row_off &= ~3;
  const char *rowp = slab + row_off;
  const char *qb = (const char *)qrow;
  const int n_full = W >> 2;               // whole chunks; lanes of half 0 take the first h0 of them
  const int h0 = (n_full + 1) >> 1, common = n_full - h0;
  f32x4 d0[NH], d1[NH];
#pragma unroll
  for (int g = 0; g < NH; ++g) {
    d0[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    d1[g] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  {
    // The chunks both halves have, without masks or range checks: off walks this lane's chunks as
    // a byte offset from its block's place on, wrapping inside the half's range.
    const int lo = half ? h0 * 8 : 0, hi = lo + common * 8;
    int off = lo + (common < 4 ? 0 : bb < common ? bb : bb - common) * 8;
    auto pstep = [&](f32x4 (&acc)[NH]) {
      const s16x4 ka = __builtin_bit_cast(s16x4, key_chunk<AL>(rowp + off, sb));
#pragma unroll
      for (int g = 0; g < NH; ++g) acc[g] = mfma4(ka, *(const s16x4 *)(qb + off + g * 4 * (kQS / 2) * 4), acc[g]);
      off = off + 8 == hi ? lo : off + 8;
    };
    int ks = 0;
    for (; ks + 4 <= common; ks += 4) { pstep(d0); pstep(d1); pstep(d0); pstep(d1); }
    for (; ks + 2 <= common; ks += 2) { pstep(d0); pstep(d1); }
    if (ks < common) pstep(d0);
  }
  if (h0 > common || (W & 3) != 0) {
    // What is left over, one step: half 0 takes its odd chunk, half 1 the row's last, partial chunk,
    // whose elements past W (row padding, or whatever follows the tile) are masked; a half with
    // nothing left takes zeros.
    const bool any = half == 0 ? h0 > common : (W & 3) != 0;
    const int c = half == 0 ? common : n_full;
    uint2 kw = key_chunk<AL>(rowp + (any ? c * 8 : 0), sb);
    // elements this lane's chunk has: 4, the partial chunk's W & 3, or none
    const int ne = !any ? 0 : half == 0 ? 4 : W & 3;
    kw.x &= ne >= 2 ? 0xffffffffu : ne == 1 ? 0x0000ffffu : 0u;
    kw.y &= ne == 4 ? 0xffffffffu : ne == 3 ? 0x0000ffffu : 0u;
    const s16x4 ka = __builtin_bit_cast(s16x4, kw);
    const char *qp = qb + (any ? c * 8 : kD * 2);
#pragma unroll
    for (int g = 0; g < NH; ++g) d1[g] = mfma4(ka, *(const s16x4 *)(qp + g * 4 * (kQS / 2) * 4), d1[g]);
  }
#pragma unroll
  for (int g = 0; g < NH; ++g)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const LanePair t = pair32(d0[g][r] + d1[g][r]);
      d[g][r] = t.a + t.b;
    }
}

// Running softmax over the tile's logits; the probabilities go to pline as NT bf16 terms:
// bytes [0, 256) the leading terms, [256, 512) the next, then the third, entry 4 ks + head holding
// the four rows 4 ks .. 4 ks + 3.
template <int VP, int NT>
__device__ __forceinline__ void mq_softmax(const f32x4 &d, int nrows, float scale, MqState &st, char *pline,
                                           int lane) {
  const int bb = (lane >> 2) & 7;
  float zz[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) zz[r] = (nrows == kMqRows || 4 * bb + r < nrows) ? d[r] * scale : -INFINITY;
  const float mx = quad_column_reduce<true>(max_nn(max_nn(zz[0], zz[1]), max_nn(zz[2], zz[3])));
  const float m_new = max_nn(st.m, mx);             // finite: the tile has at least one row
  if (__builtin_amdgcn_ballot_w64(m_new != st.m) != 0) {   // rare after the first tiles
    const float corr = __builtin_amdgcn_exp2f(st.m - m_new);
    st.l *= corr;
    st.m = m_new;
    // every lane carries channels of all four heads: the heads' factors sit in the lane's quad
    const float c0 = dpp_move<0x00, 0xf>(corr, corr), c1 = dpp_move<0x55, 0xf>(corr, corr);
    const float c2 = dpp_move<0xAA, 0xf>(corr, corr), c3 = dpp_move<0xFF, 0xf>(corr, corr);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      st.acc[h][0] *= c0; st.acc[h][1] *= c1; st.acc[h][2] *= c2; st.acc[h][3] *= c3;
      if constexpr (VP) {
        st.accp[h][0] *= c0; st.accp[h][1] *= c1; st.accp[h][2] *= c2; st.accp[h][3] *= c3;
      }
    }
  }
  uint32_t hi[4], lo[4], lo2[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float p = __builtin_amdgcn_exp2f(zz[r] - m_new);
    st.l += p;
    hi[r] = __float_as_uint(p) & 0xffff0000u;
    const float rem = p - __uint_as_float(hi[r]);
    lo[r] = __float_as_uint(rem) & 0xffff0000u;
    if constexpr (NT == 3) lo2[r] = __float_as_uint(rem - __uint_as_float(lo[r]));   // 8 bits are left: exact
  }
  // the lower half of the wave writes the leading terms, the upper half the remainders
  const bool up = lane >= 32;
  uint2 w;
  w.x = up ? ((lo[0] >> 16) | lo[1]) : ((hi[0] >> 16) | hi[1]);
  w.y = up ? ((lo[2] >> 16) | lo[3]) : ((hi[2] >> 16) | hi[3]);
  *(uint2 *)(pline + lane * 8) = w;
  if constexpr (NT == 3)
    if (!up) *(uint2 *)(pline + 512 + lane * 8) = uint2{(lo2[0] >> 16) | (lo2[1] & 0xffff0000u), (lo2[2] >> 16) | (lo2[3] & 0xffff0000u)};
}

// acc += P . V for the tile whose value rows are in the slab; the probabilities of head group g
// are in the 256 NT bytes at pline + 256 NT g, term by term.  The value operand is read once for all
// groups.
template <int NH, int NT, bool RAGGED = false>
__device__ __forceinline__ void mq_values(const char *slab, const char *pline, int nrows, MqState (&st)[NH],
                                          int lane) {
  const int x = lane & 3, grp = lane >> 4, j = lane & 15, r = j >> 2, seg = j & 3;
  const int cc = 2 * grp + (seg >> 1), swz = (r & 1) << 3;
  const char *vb0 = slab + r * 256 + ((cc ^ swz) << 4) + (seg & 1) * 8;        // channels 0 .. 63
  const char *vb1 = slab + r * 256 + (((8 + cc) ^ swz) << 4) + (seg & 1) * 8;  // channels 64 .. 127
  const char *pa = pline + x * 8;
  auto rows4 = [&](const int ks) {
    const s16x4 b0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4 *)(vb0 + ks * 1024));
    const s16x4 b1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4 *)(vb1 + ks * 1024));
    s16x4 a[NT][NH];
#pragma unroll
    for (int g = 0; g < NH; ++g)
#pragma unroll
      for (int i = 0; i < NT; ++i) a[i][g] = *(const s16x4 *)(pa + (g * NT + i) * 256 + ks * 32);
    // (three terms of eight heads: a read that runs ahead of the step before would not find registers)
    if constexpr (NT * NH == 6) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int g = 0; g < NH; ++g) {
        st[g].acc[0] = mfma4(a[i][g], b0, st[g].acc[0]);
        st[g].acc[1] = mfma4(a[i][g], b1, st[g].acc[1]);
      }
  };
  // a whole tile: straight-line code, the reads of later rows overlap the products
  if (RAGGED || nrows < kMqRows) {
    const int nks = (nrows + 3) >> 2;
    for (int ks = 0; ks < nks; ++ks) rows4(ks);
  } else {
#pragma unroll
    for (int ks = 0; ks < kMqRows / 4; ++ks) rows4(ks);
  }
}

// accp += P . V_pruned for the tile whose value bytes sit in the slab as staged (first row at
// byte `shift`, rows pitch_bytes apart).  A read past a row's T_v channels lands in the next row,
// or within the bytes that follow every slab, and only feeds kept-channel numbers >= T_v,
// which nobody collects; a row past a ragged tile's end is read as the tile's last row, with
// probability 0.
template <int NH, int NT>
__device__ __forceinline__ void mq_values_pruned(const char *slab, int shift, int pitch_bytes, int T_v,
                                                 const char *pline, int nrows, MqState (&st)[NH], int lane) {
  const int x = lane & 3, grp = lane >> 4, j = lane & 15, r = j >> 2, seg = j & 3;
  const char *vb = slab + shift + (16 * grp + 4 * seg) * 2;
  const char *pa = pline + x * 8;
  auto rows4 = [&](const int ks, const char *vrow, auto wide) {
    const s16x4 b0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(vrow));
    s16x4 b1 = b0;
    if constexpr (wide)
      b1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(vrow + 128));
    s16x4 a[NT][NH];
#pragma unroll
    for (int g = 0; g < NH; ++g)
#pragma unroll
      for (int i = 0; i < NT; ++i) a[i][g] = *(const s16x4 *)(pa + (g * NT + i) * 256 + ks * 32);
    if constexpr (NT * NH == 6) __builtin_amdgcn_sched_barrier(0);   // as in mq_values
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int g = 0; g < NH; ++g) {
        st[g].accp[0] = mfma4(a[i][g], b0, st[g].accp[0]);
        if constexpr (wide) st[g].accp[1] = mfma4(a[i][g], b1, st[g].accp[1]);
      }
  };
  auto tile = [&](auto wide) {
    if (nrows == kMqRows) {   // straight-line code, the reads of later rows overlap the products
#pragma unroll
      for (int ks = 0; ks < kMqRows / 4; ++ks) rows4(ks, vb + (4 * ks + r) * pitch_bytes, wide);
      return;
    }
    const int nks = (nrows + 3) >> 2;
    for (int ks = 0; ks < nks; ++ks) rows4(ks, vb + min(4 * ks + r, nrows - 1) * pitch_bytes, wide);
  };
  if (T_v > 64) tile(std::true_type{});
  else tile(std::false_type{});
}

constexpr int mq_terms(int AL) { return AL == 8 ? 2 : 3; }   // bf16 terms of a probability

// KB: 16-byte key chunks a lane may have to stage for one tile.  slab_bytes: the wave's LDS slab,
// which holds a tile's key bytes and, once the logits are done, its value rows.
// VP = 1: the value rows of the pruned segment are channel-pruned (a.v = V_pruned, a.ld_v, a.idx_v).
// NH: groups of four query heads served by one block (1, or 2 when N_q / N_kv is a multiple of 8:
// the key and value operands are then read from LDS once for eight heads).
// AL: alignment of the key rows in bytes (mq_logits).
template <int KB, int WPE, int VP, int NH, int AL>
__global__ __launch_bounds__(256, WPE) void k_decode_mq(DecodeArgs a, int groups, int slab_bytes) {
  constexpr int DT = THK_BF16, GT = 4 * NH, EB = 2, TR = kMqRows;
  constexpr int NT = mq_terms(AL), PB = 256 * NT;
  extern __shared__ uint4 smem[];
  uint32_t *qkp = (uint32_t *)smem;                 // [GT][kQS/2] kept query channels, packed bf16, 0 beyond T
  uint32_t *qfp = qkp + GT * (kQS / 2);             // [GT][kQS/2] full query
  char *wbase = (char *)(qfp + GT * (kQS / 2));
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);   // uniform: tile counts and branches stay scalar
  char *slab = wbase + (size_t)wave * (slab_bytes + PB * NH);
  char *pline = slab + slab_bytes;               // PB bytes of probabilities per head group
  __shared__ int s_last;

  want_arguments(a, groups);
  DecodeWork work;
  if (!decode_block_work<NH == 2>(a, groups, work)) return;   // four slots: all heads of a unit
  const int sp = work.sp, gi = work.gi;
  const int64_t u = work.u;
  const int G = a.G;
  const int64_t bn0 = u * G + (int64_t)gi * GT;
  const int hb = min(GT, G - gi * GT);   // head slots in use; the others carry a zero query

  QueryStage<DT, GT> qs;
  qs.issue(a.q, (size_t)bn0, hb, a.idx + (size_t)u * a.T, a.T);

  // the first tile's key and value bytes start moving before anything is waited for
  constexpr int VB = VP ? KB : kMqVChunks;
  static_assert(kTailRows * 16 <= 4 * kWave && KB >= 4, "a tail tile is four chunks per lane");
  u32x4 kr[KB], vr[VB];
  WaveTiles<EB, VP> tiles(a, u, sp, wave);
  Tile nt = tiles.next();
  tile_issue<KB>(kr, nt.k.base, nt.k.bytes, lane);
  tile_issue<VB>(vr, nt.v.base, nt.v.bytes, lane);

  // query: gather the kept channels (Sec. 3.3: the query is pruned with the stored mask), out of
  // LDS (the slabs are idle until the barrier below)
  qs.commit(wbase);
  __syncthreads();
  QueryStage<DT, GT>::pack(wbase, a.T, nullptr, nullptr, qfp, qkp);
  __syncthreads();

  MqState st[NH];
#pragma unroll
  for (int g = 0; g < NH; ++g) {
    st[g].m = -INFINITY;
    st[g].l = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      st[g].acc[h] = f32x4{0.f, 0.f, 0.f, 0.f};
      st[g].accp[h] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  const int x = lane & 3;

  // ---- the bytes of this wave's next tile are in flight while the current one is computed:
  // pruned tiles, then the wave's share of the unpruned tail (full-width keys, full query)
  while (nt.kind == Tile::kPruned) {
    const Tile t = nt;
    nt = tiles.next();
    k_commit<KB>(kr, slab, lane);
    tile_issue<KB>(kr, nt.k.base, nt.k.bytes, lane);
    wave_sync_lds();
    f32x4 d[NH];
    mq_logits<NH, AL>(slab, t.k.shift, t.nrows, a.T, a.ldk * EB, qkp + x * (kQS / 2), lane, d);
#pragma unroll
    for (int g = 0; g < NH; ++g) mq_softmax<VP, NT>(d[g], t.nrows, a.scale_log2, st[g], pline + PB * g, lane);
    wave_sync_lds();   // the key bytes are consumed: the slab takes the value rows
    if constexpr (VP) k_commit<KB>(vr, slab, lane);
    else mq_v_commit<VB>(vr, slab, lane);
    tile_issue<VB>(vr, nt.v.base, nt.v.bytes, lane);
    wave_sync_lds();
    if constexpr (VP) mq_values_pruned<NH, NT>(slab, t.v.shift, a.ld_v * EB, a.T_v, pline, t.nrows, st, lane);
    else mq_values<NH, NT>(slab, pline, t.nrows, st, lane);
    wave_sync_lds();   // slab and pline are rewritten by the next tile
  }
  while (nt.kind == Tile::kTail) {
    const Tile t = nt;
    nt = tiles.next();
    k_commit<4>(kr, slab, lane);
    tile_issue<4>(kr, nt.k.base, nt.k.bytes, lane);
    wave_sync_lds();
    f32x4 d[NH];
    mq_logits<NH, 8>(slab, 0, t.nrows, kD, kD * EB, qfp + x * (kQS / 2), lane, d);
#pragma unroll
    for (int g = 0; g < NH; ++g) mq_softmax<VP, NT>(d[g], t.nrows, a.scale_log2, st[g], pline + PB * g, lane);
    wave_sync_lds();
    mq_v_commit<4>(vr, slab, lane);
    tile_issue<4>(vr, nt.v.base, nt.v.bytes, lane);
    wave_sync_lds();
    mq_values<NH, NT, true>(slab, pline, t.nrows, st, lane);
    wave_sync_lds();
  }

  // ---- wave state -> LDS: [GT][130] floats at the start of the wave's own slab -------------
  {
    float *mrg = (float *)slab;
#pragma unroll
    for (int g = 0; g < NH; ++g) {
      const float lt = quad_column_reduce<false>(st[g].l);   // both halves of the wave saw every row
      if (lane < 4) {
        float *rec = mrg + (4 * g + lane) * (kD + 2);
        rec[0] = st[g].m;
        rec[1] = lt;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float *rec = mrg + (4 * g + i) * (kD + 2) + 2;
        rec[lane] = st[g].acc[0][i];
        rec[64 + lane] = st[g].acc[1][i];
      }
    }
    if constexpr (VP) {
      // the sums over the pruned rows go to their channels (distinct for distinct kept numbers)
      wave_sync_lds();
      const int16_t *uidv = a.idx_v + (size_t)u * a.T_v;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int t = 64 * h + lane;
        if (t < a.T_v) {
          const int c = uidv[t];
#pragma unroll
          for (int g = 0; g < NH; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) mrg[(4 * g + i) * (kD + 2) + 2 + c] += st[g].accp[h][i];
        }
      }
    }
  }
  __syncthreads();
  block_merge_store<DT, GT>((const float *)wbase, (slab_bytes + PB * NH) / 4, a, bn0, sp, hb, u * groups + gi, &s_last);
}

// Four blocks per compute unit with the narrow staging class and four heads per block (37 KB of
// LDS and at most 128 registers per lane each), two with the wide class and eight heads, three
// otherwise.
template <int KB, int VP, int NH, int AL>
static hipError_t mq_launch(const DecodeArgs &a, int groups, hipStream_t st) {
  constexpr int WPE = (KB <= 5 && NH == 1) ? 4 : (KB > 5 && NH == 2) ? 2 : 3;
  const int slab = KB * kWave * 16 > kMqVBytes ? KB * kWave * 16 : kMqVBytes;
  const size_t lds = (size_t)(2 * 4 * NH * (kQS / 2)) * 4 + 4 * ((size_t)slab + 256 * mq_terms(AL) * NH);
  const dim3 grid(decode_grid(a, groups)), block(256);
  {
    static DynLds set;   // one per instantiation
    const hipError_t e = ensure_dyn_lds((const void *)k_decode_mq<KB, WPE, VP, NH, AL>, lds, set);
    if (e != hipSuccess) return e;
  }
  void *kargs[] = {(void *)&a, (void *)&groups, (void *)&slab};
  const hipError_t e = launch_main_kernel((const void *)k_decode_mq<KB, WPE, VP, NH, AL>, grid, block, kargs, lds, st);
  return e != hipSuccess ? e : hipGetLastError();
}

// Staged 16-byte chunks per lane for one tile: the wider of the key rows and, when they are
// channel-pruned, the value rows.
static int mq_chunks(const DecodeArgs &a) {
  int kb = decode_launch_params<THK_BF16>(a, kMqRows).kb;
  if (a.T_v > 0) {
    const int kbv = (int)((kMqRows * (size_t)a.ld_v * 2 + 15 + 15) / 16 + kWave - 1) / kWave;
    if (kbv > kb) kb = kbv;
  }
  return kb;
}

// True when the shape is one this kernel serves: bf16 and at least three query heads per KV head
// (one or two share a key row cheaply enough on the vector units).  Key rows of any pitch: where it
// is not a multiple of four elements an operand is put together from two or three words
// (AL = 4, 2) and a probability kept in three terms, which leaves the general kernel (four heads per
// block, vector arithmetic) far behind: T = 51 dense, 64 units x 32768 rows, G = 4 142.5 -> 124.2 us,
// G = 8 233 -> 124.4 us; G = 7, 216 units x 1700 rows 68.0 -> 33.6 us; T = 70, G = 4, 144 units x 6847
// rows 84.5 -> 69.3 us (the last with seven pieces instead of four).
// THK_DECODE_MFMA=0 in the environment keeps all shapes on k_decode.
bool decode_mq_serves(const DecodeArgs &a) {
  if (a.dtype != THK_BF16 || a.N_kv <= 0) return false;
  const int G = a.N_q / a.N_kv;
  if (G < 3) return false;
  if (a.T_v > 0 && a.ld_v % 4 != 0) return false;
  if (mq_chunks(a) > 9) return false;
  return !env_switches().decode_mfma_off;
}

// Head slots per block: four for three or four query heads per KV head, else eight; a unit
// takes ceil(G / slots) blocks per split and the last one may leave slots empty.
int decode_mq_heads(const DecodeArgs &a) { return (a.N_q / a.N_kv) <= 4 ? 4 : 8; }

// Staging classes: 4 chunks per lane (a 32-row tile of at most 4 KB: T <= 64 with 16-byte rows),
// 5 (T <= 79) and 9 (up to 128 kept channels).
template <int VP, int NH, int AL>
static hipError_t mq_launch_class(const DecodeArgs &a, int groups, hipStream_t st) {
  const int kb = mq_chunks(a);
  if constexpr (AL == 8)   // rows of other pitches: one class for the narrow ones
    if (kb <= 4) return mq_launch<4, VP, NH, AL>(a, groups, st);
  if (kb <= 5) return mq_launch<5, VP, NH, AL>(a, groups, st);
  return mq_launch<9, VP, NH, AL>(a, groups, st);
}
template <int VP, int NH>
static hipError_t mq_launch_aligned(const DecodeArgs &a, int groups, hipStream_t st) {
  if (a.ldk % 4 == 0) return mq_launch_class<VP, NH, 8>(a, groups, st);
  return a.ldk % 2 == 0 ? mq_launch_class<VP, NH, 4>(a, groups, st) : mq_launch_class<VP, NH, 2>(a, groups, st);
}

hipError_t decode_mq_launch(const DecodeArgs &a, hipStream_t st) {
  const int G = a.N_q / a.N_kv;
  if (decode_mq_heads(a) == 8) {
    const int groups = (G + 7) / 8;
    return a.T_v > 0 ? mq_launch_aligned<1, 2>(a, groups, st) : mq_launch_aligned<0, 2>(a, groups, st);
  }
  const int groups = (G + 3) / 4;
  return a.T_v > 0 ? mq_launch_aligned<1, 1>(a, groups, st) : mq_launch_aligned<0, 1>(a, groups, st);
}

}  // namespace thk
