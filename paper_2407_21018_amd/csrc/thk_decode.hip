// Decode attention: dispatch to the per-(dtype, group width) kernels and the
// merge of the per-split softmax states (gfx950, wave64).
#include "thk_decode_impl.h"

namespace thk {

static_assert(kFuseMaxSplit == kDecodeFuseMaxSplit, "the host and the kernels must agree on the fused merge's reach");

hipError_t decode_launch_bf16_g1(const DecodeArgs &, int, hipStream_t);
hipError_t decode_launch_bf16_g2(const DecodeArgs &, int, hipStream_t);
hipError_t decode_launch_bf16_g4(const DecodeArgs &, int, hipStream_t);
hipError_t decode_launch_f32_g1(const DecodeArgs &, int, hipStream_t);
hipError_t decode_launch_f32_g2(const DecodeArgs &, int, hipStream_t);
hipError_t decode_launch_f32_g4(const DecodeArgs &, int, hipStream_t);
hipError_t decode_kv_launch_bf16_g1(const DecodeArgs &, int, hipStream_t);
hipError_t decode_kv_launch_bf16_g2(const DecodeArgs &, int, hipStream_t);
hipError_t decode_kv_launch_bf16_g4(const DecodeArgs &, int, hipStream_t);
hipError_t decode_kv_launch_f32_g1(const DecodeArgs &, int, hipStream_t);
hipError_t decode_kv_launch_f32_g2(const DecodeArgs &, int, hipStream_t);
hipError_t decode_kv_launch_f32_g4(const DecodeArgs &, int, hipStream_t);
// four query heads per KV head on the matrix cores (bf16, full-width values)
hipError_t decode_mq_launch(const DecodeArgs &, hipStream_t);

// Merge of the per-split states: m = max m_i, l = sum l_i 2^(m_i - m),
// acc = sum acc_i 2^(m_i - m), out = acc / l.  One block of NW wavefronts per query head: wave w takes the
// pieces 16 w .. 16 w + 15 of every 16 NW, a lane two channels of them, lane i also piece i's maximum and sum,
// whose weight reaches the other lanes through v_readlane.  Latency bounds it: the maxima, the sums and the
// accumulators of a wave's 16 pieces are one trip to memory, absent pieces read 0 past the end of the buffer
// and weigh nothing, and the waves' states meet in LDS once, in wave order (the result does not depend on timing).
// (A weight below 2^-126 is 0, as in the tiles, where the library's exp2 kept a denormal.)
// Before, a block asked for the maxima, then for eight accumulators at a time, and for those past a multiple of eight
// one by one.  Whole calls, us, before / now: 4 units x 8 heads x 8000 rows (63 pieces) 11.6 / 9.5, fp32 8 x 9000 (29)
// 15.6 / 13.4, 8 x 4 heads x 131072 (64) 64.2 / 63.3, 64 x 4 heads x 32768 (16) 123.4 / 122.0, 64 x 8 heads x 8191, pruned
// values (8) 30.3 / 29.8.
template <int DT, int NW>
__global__ __launch_bounds__(64 * NW) void k_decode_merge(const float *__restrict__ ws,
                                                          void *__restrict__ out, int n_split) {
  using E = Elem<DT>;
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  constexpr int kRecB = (kD + 2) * 4, P = 16;
  __shared__ f32x2 part_ml[NW], part_a[NW][kWave];
  const int lane = threadIdx.x % kWave, wave = uniform(threadIdx.x / kWave);
  const size_t bn = blockIdx.x;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr((const char *)(ws + bn * n_split * (kD + 2))),
                                                      (short)0, n_split * kRecB, kBufferWord3);
  auto load2 = [&](int off) { return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, 0)); };
  auto weight = [](float m, float M) { return m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M); };
  float M = -INFINITY, L = 0.f, A0 = 0.f, A1 = 0.f;
  for (int i0 = wave * P; i0 < n_split; i0 += NW * P) {
    const f32x2 ml = load2((i0 + min(lane, P)) * kRecB);   // lanes from P on hold a piece that is not this wave's
    f32x2 av[P];
#pragma unroll
    for (int i = 0; i < P; ++i) av[i] = load2((i0 + i) * kRecB + 8 + lane * 8);
    const float m = lane < P && i0 + lane < n_split ? ml[0] : -INFINITY;
    const float M_new = fmaxf(M, wave_max(m));   // whole numbers: every weight here is an exact power of two
    const float wgt = weight(m, M_new), keep = weight(M, M_new);
    M = M_new;
    L = fmaf(L, keep, wave_sum(lane < P ? ml[1] * wgt : 0.f));
    A0 *= keep;
    A1 *= keep;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const float wi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wgt), i));
      A0 = fmaf(av[i][0], wi, A0);
      A1 = fmaf(av[i][1], wi, A1);
    }
  }
  if constexpr (NW > 1) {
    part_a[wave][lane] = f32x2{A0, A1};
    if (lane == 0) part_ml[wave] = f32x2{M, L};
    __syncthreads();
    if (wave != 0) return;
    f32x2 ml[NW], av[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) { ml[w] = part_ml[w]; av[w] = part_a[w][lane]; }
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, ml[w][0]);
    L = A0 = A1 = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wi = weight(ml[w][0], M);
      L = fmaf(ml[w][1], wi, L);
      A0 = fmaf(av[w][0], wi, A0);
      A1 = fmaf(av[w][1], wi, A1);
    }
  }
  E::store2(out, bn * kD + 2 * lane, A0 / L, A1 / L);
}

template <int DT>
static void launch_decode_merge(const DecodeArgs &a, hipStream_t st) {
  const dim3 heads((unsigned)(a.units / a.N_kv * a.N_q));
  // one trip up to 128 pieces; fewer waves have less to say to each other
  if (a.n_split <= 16) hipLaunchKernelGGL((k_decode_merge<DT, 1>), heads, dim3(64), 0, st, a.ws, a.out, a.n_split);
  else if (a.n_split <= 64) hipLaunchKernelGGL((k_decode_merge<DT, 4>), heads, dim3(256), 0, st, a.ws, a.out, a.n_split);
  else hipLaunchKernelGGL((k_decode_merge<DT, 8>), heads, dim3(512), 0, st, a.ws, a.out, a.n_split);
}

hipError_t launch_decode(const DecodeArgs &a, hipStream_t st) {
  clear_stale_hip_error();
  const int G = a.N_q / a.N_kv;
  // query heads per block of the general kernel: 1, 2, or 4 with the unit's last block partly
  // filled when G is not a multiple of 4 (every block of a unit streams the unit's K and V)
  const int gt = G <= 2 ? G : 4;
  const int groups = (G + gt - 1) / gt;
  hipError_t e;
  if (decode_mq_serves(a))
    e = decode_mq_launch(a, st);
  else if (a.T_v > 0 && a.dtype == THK_BF16)
    e = gt == 4 ? decode_kv_launch_bf16_g4(a, groups, st)
                : gt == 2 ? decode_kv_launch_bf16_g2(a, groups, st) : decode_kv_launch_bf16_g1(a, groups, st);
  else if (a.T_v > 0)
    e = gt == 4 ? decode_kv_launch_f32_g4(a, groups, st)
                : gt == 2 ? decode_kv_launch_f32_g2(a, groups, st) : decode_kv_launch_f32_g1(a, groups, st);
  else if (a.dtype == THK_BF16)
    e = gt == 4 ? decode_launch_bf16_g4(a, groups, st)
                : gt == 2 ? decode_launch_bf16_g2(a, groups, st) : decode_launch_bf16_g1(a, groups, st);
  else
    e = gt == 4 ? decode_launch_f32_g4(a, groups, st)
                : gt == 2 ? decode_launch_f32_g2(a, groups, st) : decode_launch_f32_g1(a, groups, st);
  if (e != hipSuccess) return e;
  if (a.n_split > 1 && a.arrive == nullptr) {
    if (a.dtype == THK_BF16) launch_decode_merge<THK_BF16>(a, st);
    else launch_decode_merge<THK_F32>(a, st);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace thk
