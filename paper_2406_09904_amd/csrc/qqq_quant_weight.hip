// Offline weight front-end: symmetric round-to-nearest int4 codes and their scales from fp16
// weights (the inputs of Sec. 3.3.1's offline scale adjustment and of the offline boxes of
// Fig. 5 in the QQQ paper).  The row of an output channel is read once, the block maxima
// (channel: workgroup reduction; group of 128 = one 16-lane row of a wave) are reduced with
// data-parallel primitives, the row is divided by the stored fp16 scale, rounded half to
// even, clamped to [-7,7] and written eight codes per word in the natural nibble format.
// Per-group, the same pass finds the channel's largest dequantised magnitude, from which the
// fp16->int8 scale s_Wc and the fused scales s*_Wg = s_Wg / s_Wc follow.  A streaming pass:
// 2 B in, 0.5 B out per weight.
#include "qqq_internal.h"

#include <type_traits>

namespace qqq {

namespace {

constexpr float kStarCap = 18.203125f;  // largest fp16 s with rne(7 * s) <= 127
constexpr int kWaves = 4;               // waves, and channels, per workgroup of the per-group kernel

__device__ __forceinline__ uint32_t row16_max_u32(uint32_t v) {  // max over a 16-lane row, in every lane
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
  return v;
}

struct GroupOut {
  uint16_t* s_wg;    // [G][N] or nullptr
  uint16_t* s_star;  // [G][N]
  int8_t* s_int;     // [G][N] or nullptr
  int G;
};

__device__ __forceinline__ uint32_t block_max(uint32_t v, uint32_t* smem) {
  v = wave_max_u32(v);
  if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = v;
  __syncthreads();
  const uint32_t r = max(max(smem[0], smem[1]), max(smem[2], smem[3]));
  __syncthreads();
  return r;
}

}  // namespace

// absmax_bits one pattern at a time.  The per-channel kernel has little to do between its loads and its reduction, and there
// this form is ahead of two at a time (N = 11008, K = 4096: 19.9 us against 20.5; N = 4096: 9.9 against 10.2); the per-group kernel is
// bound by its instructions and takes the other.
__device__ __forceinline__ uint32_t absmax_bits_each(uint4 v, uint32_t cur) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) cur = max(cur, max(w[i] & 0x7FFFu, (w[i] >> 16) & 0x7FFFu));
  return cur;
}

// Per-channel: one workgroup per channel.
// VPT > 0: the row fits in VPT 128-bit vectors per thread and stays in registers, all of them requested before the first is looked at
// (N = 4096, K = 11008 23.5 us, 28.7 with a condition on each; N = 1024, K = 32768 20.0, 24.7; N = 28672, K = 8192 110 either way: memory).
// VPT == 0: any K; the row is read twice (the second read hits L2).
template <int VPT>
__global__ __launch_bounds__(256) void quant_weight_channel_kernel(const uint4* __restrict__ w, int64_t ldw_vec,
                                                                   int nvec, uint32_t* __restrict__ w_nat,
                                                                   uint16_t* __restrict__ s_w) {
  __shared__ uint32_t smem[4];
  const int64_t n = blockIdx.x;
  const uint4* row = w + n * ldw_vec;
  uint32_t* out = w_nat + n * (int64_t)nvec;
  constexpr int kIter = VPT > 0 ? VPT : 1;
  uint4 v[kIter];
  uint32_t amax_bits = 0;
  if constexpr (VPT > 0) {
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const int idx = threadIdx.x + 256 * j;
      v[j] = row[min(idx, nvec - 1)];  // (unconditional: a load under its own condition waits for the one before)
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      amax_bits = absmax_bits_each(v[j], amax_bits);
    }
  } else {
    for (int idx = threadIdx.x; idx < nvec; idx += 256) amax_bits = absmax_bits_each(row[idx], amax_bits);
  }
  amax_bits = block_max(amax_bits, smem);
  const uint16_t sb = scale_bits(half_bits_to_float(amax_bits), 7.0f);
  const float s = half_bits_to_float(sb);
  if (threadIdx.x == 0) s_w[n] = sb;
  const float rs = __builtin_amdgcn_rcpf(s);
  float cmax;
  if (s == 0.0f) {  // uniform over the workgroup
    for (int idx = threadIdx.x; idx < nvec; idx += 256) out[idx] = 0u;
    return;
  }
  if constexpr (VPT > 0) {
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const int idx = threadIdx.x + 256 * j;
      asm volatile("" : "+v"(v[j].x), "+v"(v[j].y), "+v"(v[j].z), "+v"(v[j].w));  // (the dwords anew: not the elements
      // that the maximum took apart, eight registers a vector)
      if (idx < nvec) out[idx] = quant8<false>(v[j], s, rs, &cmax);
    }
  } else {
    for (int idx = threadIdx.x; idx < nvec; idx += 256) out[idx] = quant8<false>(row[idx], s, rs, &cmax);
  }
}

// Per-group: one wave per channel, four channels per workgroup.  A group of 128 is 16
// consecutive vectors, i.e. one 16-lane row of a wave, so its scale needs no memory of the rest of
// the channel: the wave streams the row once, four vectors per lane at a time, and leaves the group
// scales in LDS; the channel's s_Wc follows from a wave reduction at the end of the row.
// The scale tables are [G][N]: one channel owns one element of every table row.  The workgroup's
// LDS stage is [G][kWaves], and after a barrier the tables are written in runs of four elements,
// the division s_Wg / s_Wc being done there.  STAGED == false (a table too tall for LDS): the
// wave reads its row a second time (from L2) and writes its table elements one by one.
// K = 8192, N = 28672: 131 us, 4.6 TB/s; K = 4096, N = 11008: 25.6 us, 4.5 TB/s; N = 4096: 11.8.  Neither memory alone (a copy reaches
// 6.1 TB/s) nor instructions (about 8 a weight, 0.4 of these times): between a wave's requests and its codes nothing else of
// that wave runs.  The range checks are only where a row ends (per 2048 weights): with checks everywhere and eight channels a workgroup from N = 18432 on 131 was 137, 25.6 27.0, 11.8 12.9, and K = 11008, N = 6656
// 49.3 us 53.1.  Four channels throughout: eight are 1 to 9 % slower from K = 4096 on (K = 8192, N = 8704: 45.4 us against 42.8), up to 8 % faster only
// for rows of at most 2048 and N >= 12288, and leave the chip idle on narrow layers (K = 8192, N = 1024: 14.7 against 9.6).
template <int V>
using Count = std::integral_constant<int, V>;

template <bool STAGED>
__global__ __launch_bounds__(64 * kWaves) void quant_weight_group_kernel(const uint4* __restrict__ w,
                                                                         int64_t ldw_vec, int nvec, int64_t N,
                                                                         uint32_t* __restrict__ w_nat,
                                                                         uint16_t* __restrict__ s_wc,
                                                                         const GroupOut go) {
  extern __shared__ uint16_t stage[];  // [G][kWaves] s_Wg bits, then [kWaves] s_Wc bits
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t n0 = (int64_t)blockIdx.x * kWaves;
  auto emit = [&](int64_t at, uint16_t wg_bits, float wc) {
    const float sg = half_bits_to_float(wg_bits);
    uint16_t star = 0;
    if (wc != 0.0f) {
      const _Float16 h = (_Float16)(sg / wc);
      star = __builtin_bit_cast(uint16_t, (float)h > kStarCap ? (_Float16)kStarCap : h);
    }
    go.s_star[at] = star;
    if (go.s_wg) go.s_wg[at] = wg_bits;
    if (go.s_int) go.s_int[at] = (int8_t)fminf(fmaxf(__builtin_rintf(half_bits_to_float(star)), 1.0f), 18.0f);
  };
  const int64_t n = n0 + wave;
  const int cells = go.G * kWaves;
  if (n < N) {
    const uint4* row = w + n * ldw_vec;
    uint32_t* out = w_nat + n * (int64_t)nvec;
    uint32_t dmax_bits = 0;  // bits of max |code * s_Wg|, a non-negative float
    // `count` 64s of vectors, the last of them not all there if they are the row's `rest`; all are requested before the first is looked at
    auto vectors = [&](int i0, auto count, auto rest) {
      constexpr int kCount = decltype(count)::value;
      constexpr bool kRest = decltype(rest)::value;
      uint4 v[kCount];
#pragma unroll
      for (int j = 0; j < kCount; ++j) {
        const int idx = i0 + 64 * j + lane;
        v[j] = row[kRest ? min(idx, nvec - 1) : idx];  // (in range and unconditional: a load under its own condition waits for the one before)
      }
      __builtin_amdgcn_sched_barrier(0);
      if (kRest && i0 + 64 * (kCount - 1) + lane >= nvec) v[kCount - 1] = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < kCount; ++j) {
        const int idx = i0 + 64 * j + lane;
        const uint32_t gmax = row16_max_u32(absmax_bits(v[j], 0));
        const uint16_t sgb = weight_scale_bits(half_bits_to_float(gmax));
        const float sg = half_bits_to_float(sgb);
        float cmax = 0.0f;
        uint32_t codes = 0;
        if (sg != 0.0f) codes = quant8<false>(v[j], sg, __builtin_amdgcn_rcpf(sg), &cmax);
        if (!kRest || idx < nvec) out[idx] = codes;
        dmax_bits = max(dmax_bits, __builtin_bit_cast(uint32_t, cmax * sg));
        if constexpr (STAGED)
          if ((lane & 15) == 0 && (!kRest || idx < nvec)) stage[(idx >> 4) * kWaves + wave] = sgb;
      }
    };
    int i0 = 0;
#pragma unroll 1
    for (; i0 + 256 <= nvec; i0 += 256) vectors(i0, Count<4>{}, std::false_type{});
    switch ((nvec - i0 + 63) >> 6) {
      case 1: vectors(i0, Count<1>{}, std::true_type{}); break;
      case 2: vectors(i0, Count<2>{}, std::true_type{}); break;
      case 3: vectors(i0, Count<3>{}, std::true_type{}); break;
      case 4: vectors(i0, Count<4>{}, std::true_type{}); break;
      default: break;
    }
    dmax_bits = wave_max_u32(dmax_bits);
    const uint16_t wcb = scale_bits(__builtin_bit_cast(float, dmax_bits), 127.0f);
    if (lane == 0) s_wc[n] = wcb;
    if constexpr (STAGED) {
      if (lane == 0) stage[cells + wave] = wcb;
    } else {
      const float wc = half_bits_to_float(wcb);
      for (int i0 = 0; i0 < nvec; i0 += 64) {  // the group maxima again, from L2
        const int idx = i0 + lane;
        const uint4 vec = idx < nvec ? row[idx] : make_uint4(0, 0, 0, 0);
        const uint32_t gmax = row16_max_u32(absmax_bits(vec, 0));
        if ((lane & 15) == 0 && idx < nvec)
          emit((int64_t)(idx >> 4) * N + n, weight_scale_bits(half_bits_to_float(gmax)), wc);
      }
    }
  }
  if constexpr (STAGED) {
    __syncthreads();
    for (int c = threadIdx.x; c < cells; c += 64 * kWaves) {
      const int r = c & (kWaves - 1);
      if (n0 + r < N) emit((int64_t)(c / kWaves) * N + n0 + r, stage[c], half_bits_to_float(stage[cells + r]));
    }
  }
}

int launch_quant_weight(const void* w, int64_t N, int64_t K, int64_t ldw, bool grouped, uint32_t* w_nat,
                        uint16_t* s_ch, uint16_t* s_wg, uint16_t* s_star, int8_t* s_int, hipStream_t st) {
  if (N == 0) return QQQ_OK;
  const uint4* wp = (const uint4*)w;
  const int64_t ldw_vec = ldw / 8;
  const int nvec = (int)(K / 8);
  if (!grouped) {
    const dim3 grid((unsigned)N), block(256);
    const int vpt = (nvec + 255) / 256;
#define QQQ_QW(V) \
  hipLaunchKernelGGL((quant_weight_channel_kernel<V>), grid, block, 0, st, wp, ldw_vec, nvec, w_nat, s_ch)
    if (vpt <= 1) QQQ_QW(1);
    else if (vpt <= 2) QQQ_QW(2);
    else if (vpt <= 4) QQQ_QW(4);
    else if (vpt <= 8) QQQ_QW(8);
    else if (vpt <= 16) QQQ_QW(16);
    else QQQ_QW(0);
#undef QQQ_QW
  } else {
    GroupOut go;
    go.s_wg = s_wg;
    go.s_star = s_star;
    go.s_int = s_int;
    go.G = (int)(K / QQQ_GROUP);
    const size_t stage = (size_t)(go.G + 1) * kWaves * 2;
    const dim3 grid((unsigned)((N + kWaves - 1) / kWaves)), block(64 * kWaves);
    if (stage <= 48u * 1024u)
      hipLaunchKernelGGL((quant_weight_group_kernel<true>), grid, block, stage, st, wp, ldw_vec, nvec, N, w_nat, s_ch, go);
    else
      hipLaunchKernelGGL((quant_weight_group_kernel<false>), grid, block, 0, st, wp, ldw_vec, nvec, N, w_nat, s_ch, go);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(QQQ_ERR_HIP, "quant_weight launch: %s", hipGetErrorString(e));
  return QQQ_OK;
}

}  // namespace qqq
