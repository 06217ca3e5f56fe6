// Key compaction K_pruned[s][t] = K[s][idx[t]] (Fig. 1; Sec. 3.3), full-width row
// copies and the tail append (gfx950, wave64).  Pure byte movement: no arithmetic
// on values.
#include "thk_prune_device.h"

namespace thk {

// A run of rows of K_pruned is a run of bytes (dense rows, or rows with padding behind them,
// which is written as zeros); the unit may start and end anywhere (see compact_rows).
// A unit's list on its way to the gather table (compact_build_tab, with the loads apart from their use):
// 32 threads per row of the table's period, entries thread % 32 + 32 n.
struct ChannelList {
  int ch[4];
  __device__ __forceinline__ void request(const int16_t *uidx, int T) {
#pragma unroll
    for (int n = 0; n < 4; ++n) ch[n] = uidx[min((int)(threadIdx.x & 31) + 32 * n, T - 1)];
    __builtin_amdgcn_sched_barrier(0);   // what is requested next stays behind
  }
  // The entries are waited for here, all four at once (left alone, the compiler moves each load to its
  // use, behind the rows: four trips one after the other).
  __device__ __forceinline__ void arrived() {
    asm volatile("" : "+v"(ch[0]), "+v"(ch[1]), "+v"(ch[2]), "+v"(ch[3]));
  }
  template <int DT>
  __device__ __forceinline__ void build_tab(int16_t *tab, int T, int ld, int sh) const {
    const int period = 8 * ld, row = threadIdx.x >> 5;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int t = (int)(threadIdx.x & 31) + 32 * n;
      if (t >= ld) break;
      int i = row * ld + t + sh, back = 0;
      if (i >= period) { i -= period; back = 8 * Tile<DT>::ROW_ELEMS; }
      tab[i] = (int16_t)((row * Tile<DT>::ROW_ELEMS + (t < T ? ch[n] : kD) - back) * (int)sizeof(typename Elem<DT>::Bits));
    }
  }
};

template <int DT>
__device__ __forceinline__ void compact_flat_block(const CompactArgs &a, uint32_t block, u32x4 *smem) {
  using E = Elem<DT>;
  constexpr int CPR = kD / E::VEC, TR = kCompactTileRows, NLD = TR * CPR / kWave;
  int16_t *tab = (int16_t *)smem;                         // [8 * T], padded to 2 KiB
  const uint32_t u = block / (uint32_t)a.blocks_per_unit;
  const int blk = (int)(block - u * (uint32_t)a.blocks_per_unit);
  const int64_t s0 = (int64_t)blk * a.rows_per_block;
  const int n_rows = (int)min(a.n_rows - s0, a.rows_per_block);
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const char *src = (const char *)a.src + ((size_t)u * a.src_unit_rows + a.src_row0 + s0) * kD * E::EB;
  u32x4 *tile = smem + 128 + wave * Tile<DT>::CHUNKS;
  // A tile's rows are requested before the tile in front of it is gathered, the first tile's before the
  // table is built: a short call is a chain of trips (64 units x 487 bf16 rows, T = 51: 7.7 -> 4.6 us),
  // a long one is bounded by memory (64 x 32768 rows, T = 64: 5.7 TB/s).
  u32x4 r[NLD];
  // (rows past the end of a ragged tile repeat its last chunk, never gathered; a wave without rows the block's first)
  auto request = [&](int row) {
    const uint32_t last = row < n_rows ? (uint32_t)min(TR, n_rows - row) * CPR - 1u : 0u;
    row = row < n_rows ? row : 0;
#pragma unroll
    for (int j = 0; j < NLD; ++j)
      r[j] = ld_stream((const u32x4 *)(src + (size_t)row * (kD * E::EB) + min((uint32_t)(j * kWave + lane), last) * 16u));
  };
  // The list goes first: loads return in order, and the table is to be built while the rows travel (the
  // other way round, calls of a few rounds of blocks lose: 448 units x 512 fp32 rows 31.6 instead of 28.0
  // us, 224 x 896 bf16 rows, T = 86, 19.0 instead of 15.7).
  ChannelList list;
  list.request(a.idx + (size_t)u * a.T, a.T);
  int row = wave * TR;
  request(row);   // no branch around it: how many loads are behind the list is known
  list.arrived();
  const FlatOut<DT> out((char *)a.dst + ((size_t)u * a.dst_unit_rows + a.dst_row0) * a.ld * E::EB);
  list.build_tab<DT>(tab, a.T, a.ld, out.sh);
  if (a.ld != a.T) tile_clear_padding<DT>(tile, lane);
  __syncthreads();
  for (; row < n_rows; row += 4 * TR) {
#pragma unroll
    for (int j = 0; j < NLD; ++j) tile[Tile<DT>::slot(j * kWave + lane)] = r[j];
    if (row + 4 * TR < n_rows) request(row + 4 * TR);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    compact_emit_tile<DT>(tile, out, s0 + row, min(TR, n_rows - row), a.ld, tab, lane);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

template <int DT>
__global__ __launch_bounds__(256) void k_compact_flat(CompactArgs a) {
  extern __shared__ u32x4 smem[];
  compact_flat_block<DT>(a, blockIdx.x, smem);
}

// A whole tail leaves for the pruned cache: the first n_compact blocks compact the keys, the others
// copy the values, kFlushRows rows of a unit each (the other order is 10 % slower: the longer blocks
// would come last).  One launch instead of two: the second one's dispatch and ramp weigh most on
// small tails (from a graph): 192 units x 128 rows 7.4 -> 5.3 us, 64 x 32 rows 5.4 -> 3.4 us; whole calls of
// 1024 x 128 rows 24.4 -> 22.8 us (bounded by memory: 121 MB, 5.3 TB/s).
constexpr int kFlushRows = 64;
struct FlushCopy {
  const void *src;
  void *dst;
  int64_t src_unit_rows, dst_unit_rows, dst_row0;
  int32_t n_rows, blocks_per_unit;
};
template <int DT>
__global__ __launch_bounds__(256) void k_flush(CompactArgs a, FlushCopy c, uint32_t n_compact) {
  extern __shared__ u32x4 smem[];
  // all arguments at once, as the blocks of either kind need them: one trip instead of two (bf16, 96 units x 128 rows 4.00
  // -> 3.81 us, 1024 x 128 20.97 -> 20.80; fp32, 64 x 64 4.18 -> 4.06; medians of 15 turns in alternation, of which
  // every one has this sign; two runs of one side can differ by as much on the larger ones)
  asm volatile("" ::"s"(a.src), "s"(a.dst), "s"(a.idx), "s"(a.src_unit_rows), "s"(a.src_row0), "s"(a.dst_unit_rows), "s"(a.dst_row0),
               "s"(a.n_rows), "s"(a.rows_per_block), "s"(a.T), "s"(a.ld), "s"(a.blocks_per_unit), "s"(c.src), "s"(c.dst),
               "s"(c.src_unit_rows), "s"(c.dst_unit_rows), "s"(c.dst_row0), "s"(c.n_rows), "s"(c.blocks_per_unit));
  if (blockIdx.x < n_compact) {
    compact_flat_block<DT>(a, blockIdx.x, smem);
    return;
  }
  constexpr int CPR = kD / Elem<DT>::VEC, PER = kFlushRows * CPR / 256;   // 16-byte chunks per row, per thread
  const uint32_t block = blockIdx.x - n_compact;
  const uint32_t u = block / (uint32_t)c.blocks_per_unit;
  const int r0 = (int)(block - u * (uint32_t)c.blocks_per_unit) * kFlushRows;
  const int total = min(kFlushRows, c.n_rows - r0) * CPR;
  const u32x4 *s = (const u32x4 *)c.src + ((size_t)u * c.src_unit_rows + r0) * CPR;
  u32x4 *d = (u32x4 *)c.dst + ((size_t)u * c.dst_unit_rows + c.dst_row0 + r0) * CPR;
  u32x4 r[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) r[j] = ld_stream(s + min(j * 256 + (int)threadIdx.x, total - 1));
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (j * 256 + (int)threadIdx.x < total) st_stream(d + j * 256 + threadIdx.x, r[j]);
}

// Full-width row copy dst[u][dst_row0 + r][:] = src[u][src_row0 + r][:], r < n_rows.
// One block per unit; rows move in ascending chunks, each chunk loaded completely
// before any of it is stored, so a downward shift inside one buffer
// (dst_row0 <= src_row0) is safe.  src and dst may alias: neither is declared restrict.
template <int DT>
__global__ __launch_bounds__(256) void k_copy_rows(const void *src, void *dst,
                                                   int64_t src_unit_rows, int64_t src_row0,
                                                   int64_t dst_unit_rows, int64_t dst_row0,
                                                   int64_t n_rows) {
  using E = Elem<DT>;
  constexpr int CPR = kD / E::VEC;     // 16-byte chunks per row
  constexpr int PER = 8;               // chunks per thread per pass
  const int64_t u = blockIdx.x;
  const u32x4 *s = (const u32x4 *)src + ((size_t)u * src_unit_rows + src_row0) * CPR;
  u32x4 *d = (u32x4 *)dst + ((size_t)u * dst_unit_rows + dst_row0) * CPR;
  const int64_t total = n_rows * CPR;
  for (int64_t c0 = 0; c0 < total; c0 += 256 * PER) {
    u32x4 r[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int64_t c = c0 + (int64_t)j * 256 + threadIdx.x;
      if (c < total) r[j] = s[c];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int64_t c = c0 + (int64_t)j * 256 + threadIdx.x;
      if (c < total) d[c] = r[j];
    }
    __syncthreads();
  }
}

// The same copy when source and destination ranges cannot touch each other: many blocks per
// unit, each streaming its own run of rows (eight 16-byte chunks in flight per thread).
template <int DT>
__global__ __launch_bounds__(256) void k_copy_rows_wide(const void *__restrict__ src, void *__restrict__ dst,
                                                        int64_t src_unit_rows, int64_t src_row0,
                                                        int64_t dst_unit_rows, int64_t dst_row0,
                                                        int64_t n_rows, int64_t rows_per_block, int blocks_per_unit) {
  using E = Elem<DT>;
  constexpr int CPR = kD / E::VEC;
  constexpr int PER = 8;
  const int64_t u = blockIdx.x / blocks_per_unit;
  const int64_t r0 = (int64_t)(blockIdx.x % blocks_per_unit) * rows_per_block;
  const int64_t r1 = min(n_rows, r0 + rows_per_block);
  const u32x4 *s = (const u32x4 *)src + ((size_t)u * src_unit_rows + src_row0 + r0) * CPR;
  u32x4 *d = (u32x4 *)dst + ((size_t)u * dst_unit_rows + dst_row0 + r0) * CPR;
  const int64_t total = (r1 - r0) * CPR;
  for (int64_t c0 = 0; c0 < total; c0 += 256 * PER) {
    u32x4 r[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int64_t c = c0 + (int64_t)j * 256 + threadIdx.x;
      if (c < total) r[j] = ld_stream(s + c);
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int64_t c = c0 + (int64_t)j * 256 + threadIdx.x;
      if (c < total) st_stream(d + c, r[j]);
    }
  }
}

// One new token per unit: K_tail[u][k_row] = k_new[u], Vdst[u][v_row] = v_new[u].
template <int DT>
__global__ __launch_bounds__(256) void k_tail_append(const void *__restrict__ k_new,
                                                     const void *__restrict__ v_new,
                                                     void *__restrict__ k_dst, void *__restrict__ v_dst,
                                                     int64_t U, int64_t k_unit_rows, int64_t k_row,
                                                     int64_t v_unit_rows, int64_t v_row) {
  using E = Elem<DT>;
  constexpr int CPR = kD / E::VEC;   // 16-byte chunks per row
  // Every argument at once: behind the return below they were a second trip in front of the first load.
  // 32 x (append + decode), medians of 15 turns in alternation: 8 units x 1000 rows x 4 heads 321.4 -> 314.6 us, eight
  // shapes 0.998 to 0.981 of the time, 0.991 in the mean; an append by itself is bound by the host.
  asm volatile("" ::"s"(k_new), "s"(v_new), "s"(k_dst), "s"(v_dst), "s"(k_unit_rows), "s"(k_row), "s"(v_unit_rows), "s"(v_row));
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= U * CPR) return;
  const int64_t u = i / CPR;
  const int c = (int)(i % CPR);
  ((u32x4 *)k_dst)[((size_t)u * k_unit_rows + k_row) * CPR + c] = ((const u32x4 *)k_new)[i];
  ((u32x4 *)v_dst)[((size_t)u * v_unit_rows + v_row) * CPR + c] = ((const u32x4 *)v_new)[i];
}

static CompactArgs compact_args(const void *src, int64_t src_unit_rows, int64_t src_row0, const int16_t *idx, void *dst,
                                int64_t dst_unit_rows, int64_t dst_row0, int64_t U, int64_t n_rows, int T, int ld_keep) {
  CompactArgs a;
  a.src = src; a.dst = dst; a.idx = idx;
  a.src_unit_rows = src_unit_rows; a.src_row0 = src_row0;
  a.dst_unit_rows = dst_unit_rows; a.dst_row0 = dst_row0; a.n_rows = n_rows;
  a.T = T; a.ld = ld_keep;
  // 4 waves x 4 tiles of 32 rows; smaller blocks (down to one tile per wave) while the call has
  // fewer than four blocks per compute unit: a wave's tiles go load -> LDS -> gather -> store one
  // after the other, so a small call is as long as its longest block
  a.rows_per_block = 512;
  while (a.rows_per_block > 128 && U * ((n_rows + a.rows_per_block - 1) / a.rows_per_block) < 4 * kCUs) a.rows_per_block /= 2;
  a.blocks_per_unit = (int)((n_rows + a.rows_per_block - 1) / a.rows_per_block);
  return a;
}

hipError_t launch_compact(int dtype, const void *src, int64_t src_unit_rows, int64_t src_row0,
                          const int16_t *idx, void *dst, int64_t dst_unit_rows, int64_t dst_row0,
                          int64_t U, int64_t n_rows, int T, int ld_keep, hipStream_t st) {
  clear_stale_hip_error();
  if (n_rows <= 0) return hipSuccess;
  const int eb = dtype == THK_BF16 ? 2 : 4;
  CompactArgs a = compact_args(src, src_unit_rows, src_row0, idx, dst, dst_unit_rows, dst_row0, U, n_rows, T, ld_keep);
  const dim3 grid((unsigned)(U * a.blocks_per_unit)), block(256);
  const size_t lds = 2048 + 4 * compact_tile_bytes(eb);
  void *kargs[] = {(void *)&a};
  const void *fn = dtype == THK_BF16 ? (const void *)k_compact_flat<THK_BF16> : (const void *)k_compact_flat<THK_F32>;
  const hipError_t e = launch_main_kernel(fn, grid, block, kargs, lds, st);
  return e != hipSuccess ? e : hipGetLastError();
}

// The whole key tail compacted and the whole value tail copied.  false: not a call for one launch
// (ranges that may touch, more rows than the copy numbers, more blocks than a grid: a launch of 2^32
// work-items or more is cut short without an error); nothing is done then.
bool launch_flush(int dtype, const void *k_tail, const void *v_tail, int64_t tail_cap, const int16_t *idx, void *k_pruned,
                  void *v, int64_t unit_rows, int64_t dst_row0, int64_t U, int64_t n_rows, int T, int ld_keep,
                  hipStream_t st, hipError_t *err) {
  const size_t eb = dtype == THK_BF16 ? 2 : 4;
  const auto apart = [](const void *x, size_t nx, const void *y, size_t ny) {
    return (const char *)x + nx <= (const char *)y || (const char *)y + ny <= (const char *)x;
  };
  const size_t n_tail = (size_t)U * tail_cap * kD * eb, n_v = (size_t)U * unit_rows * kD * eb;
  const size_t n_k = (size_t)U * unit_rows * ld_keep * eb;
  if (n_rows < 1 || n_rows > (1 << 20)) return false;
  // one after the other, the two launches also serve buffers that share memory
  if (!apart(v_tail, n_tail, v, n_v) || !apart(k_tail, n_tail, v, n_v) || !apart(v_tail, n_tail, k_pruned, n_k) ||
      !apart(v, n_v, k_pruned, n_k))
    return false;
  CompactArgs a = compact_args(k_tail, tail_cap, 0, idx, k_pruned, unit_rows, dst_row0, U, n_rows, T, ld_keep);
  FlushCopy c;
  c.src = v_tail; c.dst = v; c.src_unit_rows = tail_cap; c.dst_unit_rows = unit_rows; c.dst_row0 = dst_row0;
  c.n_rows = (int32_t)n_rows;
  c.blocks_per_unit = (int)((n_rows + kFlushRows - 1) / kFlushRows);
  const int64_t n_compact = U * a.blocks_per_unit, grid = n_compact + U * c.blocks_per_unit;
  if (grid * 256 > 0xffffffffll) return false;
  clear_stale_hip_error();
  uint32_t nc = (uint32_t)n_compact;
  void *kargs[] = {(void *)&a, (void *)&c, (void *)&nc};
  const void *fn = dtype == THK_BF16 ? (const void *)k_flush<THK_BF16> : (const void *)k_flush<THK_F32>;
  const size_t lds = 2048 + 4 * compact_tile_bytes((int)eb);
  static DynLds set[2];
  hipError_t e = ensure_dyn_lds(fn, lds, set[dtype == THK_BF16 ? 1 : 0]);
  if (e == hipSuccess) e = launch_main_kernel(fn, dim3((unsigned)grid), dim3(256), kargs, lds, st);
  *err = e != hipSuccess ? e : hipGetLastError();
  return true;
}

hipError_t launch_copy_rows(int dtype, const void *src, int64_t src_unit_rows, int64_t src_row0, void *dst,
                            int64_t dst_unit_rows, int64_t dst_row0, int64_t U, int64_t n_rows,
                            hipStream_t st) {
  clear_stale_hip_error();
  if (n_rows <= 0) return hipSuccess;
  // byte ranges the call touches, over all units: disjoint ranges may be copied in any order
  auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  constexpr int64_t kMaxBlocks = 0x7fffffff;
  const size_t rowb = (size_t)kD * (dtype == THK_BF16 ? 2 : 4);
  const char *s_lo = (const char *)src + (size_t)src_row0 * rowb;
  const char *s_hi = (const char *)src + ((size_t)(U - 1) * src_unit_rows + src_row0 + n_rows) * rowb;
  const char *d_lo = (const char *)dst + (size_t)dst_row0 * rowb;
  const char *d_hi = (const char *)dst + ((size_t)(U - 1) * dst_unit_rows + dst_row0 + n_rows) * rowb;
  const bool disjoint = s_hi <= d_lo || d_hi <= s_lo;
  const dim3 block(256);
  if (disjoint && n_rows > 64) {
    // ~8 blocks per compute unit, at least 64 rows each
    int64_t bpu = ceil_div((int64_t)kCUs * 8, U);
    const int64_t cap = ceil_div(n_rows, 64);
    if (bpu > cap) bpu = cap;
    if (bpu < 1) bpu = 1;
    const int64_t rpb = ceil_div(n_rows, bpu);
    bpu = ceil_div(n_rows, rpb);
    if (U * bpu <= kMaxBlocks) {
      const dim3 grid((unsigned)(U * bpu));
      if (dtype == THK_BF16)
        hipLaunchKernelGGL((k_copy_rows_wide<THK_BF16>), grid, block, 0, st, src, dst, src_unit_rows, src_row0, dst_unit_rows, dst_row0, n_rows, rpb, (int)bpu);
      else
        hipLaunchKernelGGL((k_copy_rows_wide<THK_F32>), grid, block, 0, st, src, dst, src_unit_rows, src_row0, dst_unit_rows, dst_row0, n_rows, rpb, (int)bpu);
      return hipGetLastError();
    }
  }
  const dim3 grid((unsigned)U);
  if (dtype == THK_BF16)
    hipLaunchKernelGGL((k_copy_rows<THK_BF16>), grid, block, 0, st, src, dst, src_unit_rows, src_row0, dst_unit_rows, dst_row0, n_rows);
  else
    hipLaunchKernelGGL((k_copy_rows<THK_F32>), grid, block, 0, st, src, dst, src_unit_rows, src_row0, dst_unit_rows, dst_row0, n_rows);
  return hipGetLastError();
}

hipError_t launch_tail_append(int dtype, const void *k_new, const void *v_new, void *k_dst, void *v_dst,
                              int64_t U, int64_t k_unit_rows, int64_t k_row, int64_t v_unit_rows,
                              int64_t v_row, hipStream_t st) {
  clear_stale_hip_error();
  const int cpr = dtype == THK_BF16 ? 16 : 32;
  const dim3 grid((unsigned)((U * cpr + 255) / 256)), block(256);
  if (dtype == THK_BF16)
    hipLaunchKernelGGL((k_tail_append<THK_BF16>), grid, block, 0, st, k_new, v_new, k_dst, v_dst, U, k_unit_rows, k_row, v_unit_rows, v_row);
  else
    hipLaunchKernelGGL((k_tail_append<THK_F32>), grid, block, 0, st, k_new, v_new, k_dst, v_dst, U, k_unit_rows, k_row, v_unit_rows, v_row);
  return hipGetLastError();
}

}  // namespace thk
