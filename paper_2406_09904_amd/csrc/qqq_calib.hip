// Offline (calibration-time) stage of QQQ on one layer: adaptive smoothing (Sec. 3.1, Eq. 1-2).  Entry points of
// include/qqq_calib.h (the Hessian of Sec. 3.2 is in qqq_hessian.hip, its compensation sweep in qqq_compensate.hip).
//
// Everything that decides an integer code is done in a fixed precision and operation order (stated at
// each kernel) so that the result can be checked bit for bit; floating-point contraction is off in
// this file for that reason.
#include "qqq_calib.h"
#include "qqq_internal.h"

#pragma clang fp contract(off)

namespace qqq {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

static bool aligned16c(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
static size_t align256c(size_t v) { return (v + 255) & ~(size_t)255; }

static int check_launch(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(QQQ_ERR_HIP, "%s launch: %s", what, hipGetErrorString(e));
  return QQQ_OK;
}

// ------------------------------------------------------------------ small helpers

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v, uint32_t* p2, size_t n2) {
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n + n2; i += stride) (i < n ? p[i] : p2[i - n]) = v;
}

// one array, or two
static int fill_u32(void* p, size_t n, uint32_t v, hipStream_t st, void* p2 = nullptr, size_t n2 = 0) {
  const size_t want = (n + n2 + 255) / 256;
  const unsigned blocks = (unsigned)(want < 2048 ? want : 2048);
  hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks ? blocks : 1), dim3(256), 0, st, (uint32_t*)p, n, v, (uint32_t*)p2, n2);
  return check_launch("fill");
}

// ------------------------------------------------------------------ Sec. 3.1: channel maxima

// absmax[t] = max_m |X[m,t]| on the fp16 bit patterns (magnitude order = integer order with the
// sign cleared); a workgroup is 32 column vectors (8 channels, one 128-bit load per row) by 8 row groups of
// rows_per_block / 8 rows, which meet in LDS, and the workgroups through atomicMax on the (non-negative) bit
// patterns.  absmax holds fp16 bit patterns as uint32 until absmax_finish_kernel widens them to fp32 and takes
// the overall maximum.
__global__ __launch_bounds__(256) void channel_absmax_kernel(const uint4* x, int64_t M, int64_t kvec,
                                                             int64_t rows_per_block, uint32_t* absmax_bits) {
  __shared__ uint32_t part[8][32][9];
  const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int64_t v = (int64_t)blockIdx.x * 32 + c;
  int64_t m1 = ((int64_t)blockIdx.y + 1) * rows_per_block;
  if (m1 > M) m1 = M;
  uint32_t mx[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (v < kvec) {
#pragma unroll 4
    for (int64_t m = (int64_t)blockIdx.y * rows_per_block + g; m < m1; m += 8) {
      const uint4 q = x[m * kvec + v];
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mx[2 * i] = max(mx[2 * i], w[i] & 0x7FFFu);
        mx[2 * i + 1] = max(mx[2 * i + 1], (w[i] >> 16) & 0x7FFFu);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) part[g][c][i] = mx[i];
  __syncthreads();
  const int cc = threadIdx.x >> 3, i = threadIdx.x & 7;  // one channel of the 256 per thread
  uint32_t r = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) r = max(r, part[k][cc][i]);
  const int64_t t = ((int64_t)blockIdx.x * 32 + cc) * 8 + i;
  if (t < kvec * 8) atomicMax(&absmax_bits[t], r);
}

// in place: fp16 bit patterns -> fp32 values (one workgroup); with sigmas, from the largest of them
// sigma_g = fp32(max|X| * g / G), the product and the quotient in fp64, g = 1..G
__global__ __launch_bounds__(1024) void absmax_finish_kernel(uint32_t* absmax, int64_t K, float* sigmas, int G) {
  __shared__ uint32_t smax;
  if (threadIdx.x == 0) smax = 0;
  __syncthreads();
  uint32_t mx = 0;
  for (int64_t t = threadIdx.x; t < K; t += 1024) {
    const uint32_t b = absmax[t];
    mx = max(mx, b);
    reinterpret_cast<float*>(absmax)[t] = half_bits_to_float(b);
  }
  atomicMax(&smax, mx);
  __syncthreads();
  if ((int)threadIdx.x < G) sigmas[threadIdx.x] = (float)((double)half_bits_to_float(smax) * (double)(threadIdx.x + 1) / (double)G);
}

// s_t = absmax_t / sigma (one fp32 division) where absmax_t > sigma, else 1; grid.y: several sigmas, their vectors
// stride_bytes apart
__global__ __launch_bounds__(256) void smoothing_vector_kernel(const float* absmax, const float* sigmas,
                                                               int64_t K, float* s, int64_t stride_bytes) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= K) return;
  const float sigma = sigmas[blockIdx.y];
  const float a = absmax[t];
  ((float*)((char*)s + stride_bytes * blockIdx.y))[t] = a > sigma ? a / sigma : 1.0f;
}

// eight channels of X' = fp16_rne(fp32(X) / s) (DIVIDE) or W' = fp16_rne(fp32(W) * s): one fp32 operation, one rounding.
// ANY_ZERO: a product of -0 may come out as 0; it is then a mixed-precision multiply-add with 0, which takes the fp16 weight as
// it is (the same fp32 rounding).
template <bool DIVIDE, bool ANY_ZERO = false>
__device__ __forceinline__ uint4 smooth8(uint4 q, float4 s0, float4 s1) {
  const float sv[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = half_bits_to_float(w[j] & 0xFFFFu), b = half_bits_to_float(w[j] >> 16);
    float ra = DIVIDE ? a / sv[2 * j] : ANY_ZERO ? __builtin_fmaf(a, sv[2 * j], 0.0f) : a * sv[2 * j];
    float rb = DIVIDE ? b / sv[2 * j + 1] : ANY_ZERO ? __builtin_fmaf(b, sv[2 * j + 1], 0.0f) : b * sv[2 * j + 1];
    // the fp32 result is rounded before the conversion sees it: left alone, the compiler turns
    // multiply + convert into one mixed-precision instruction that rounds the exact product once
    asm volatile("" : "+v"(ra), "+v"(rb));
    typedef float v2f __attribute__((ext_vector_type(2)));
    o[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){ra, rb}, h2));
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}
template <bool DIVIDE, bool ANY_ZERO = false>
__device__ __forceinline__ uint4 smooth8(uint4 q, const float* s) {
  return smooth8<DIVIDE, ANY_ZERO>(q, *reinterpret_cast<const float4*>(s), *reinterpret_cast<const float4*>(s + 4));
}

template <bool DIVIDE>
__global__ __launch_bounds__(256) void smooth_apply_kernel(const uint4* in, const float* s, int64_t rows,
                                                           int64_t kvec, uint4* out) {
  const int64_t total = rows * kvec;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride)
    out[i] = smooth8<DIVIDE>(in[i], s + (i % kvec) * 8);
}

// ------------------------------------------------------------------ a grid point's operands

// The smoothed, quantised operands of several grid points (grid.y), each point's buffers point_bytes apart, straight
// from X and W: no smoothed tensor is written.  Arithmetic as in smooth_apply_kernel followed by the hot path's
// quantisers, operation for operation.

// One token per workgroup (qqq_quant_act on X ./ s).  KEEP: the smoothed row stays in registers (K <= 8192); else it
// is computed twice.
template <bool KEEP>
__global__ __launch_bounds__(256) void point_activations_kernel(const uint4* x, const float* s, int64_t s_bytes, int kvec, int64_t point_bytes,
                                                                int8_t* a_q, float* s_a) {
  __shared__ uint32_t part[4];
  const int64_t off = point_bytes * blockIdx.y, m = blockIdx.x;
  const uint4* row = x + m * kvec;
  const float* sv = (const float*)((const char*)s + s_bytes * blockIdx.y);
  uint2* out = (uint2*)(a_q + off) + m * kvec;
  constexpr int kVecs = KEEP ? 4 : 1;
  uint4 v[kVecs];
  uint32_t bits = 0;
  if constexpr (KEEP) {
#pragma unroll
    for (int j = 0; j < kVecs; ++j) {
      const int i = threadIdx.x + 256 * j;
      if (i < kvec) bits = absmax_bits(v[j] = smooth8<true>(row[i], sv + 8 * i), bits);
    }
  } else {
    for (int i = threadIdx.x; i < kvec; i += 256) bits = absmax_bits(smooth8<true>(row[i], sv + 8 * i), bits);
  }
  bits = wave_max_u32(bits);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = bits;
  __syncthreads();
  const float amax = half_bits_to_float(max(max(part[0], part[1]), max(part[2], part[3])));
  const float sc = amax / 127.0f, rs = reciprocal_near(sc);
  if (threadIdx.x == 0) ((float*)((char*)s_a + off))[m] = amax == 0.0f ? 0.0f : sc;
  auto codes = [&](uint4 q) {
    return amax == 0.0f ? make_uint2(0, 0) : quant8_act(q, sc, rs);
  };
  if constexpr (KEEP) {
#pragma unroll
    for (int j = 0; j < kVecs; ++j) {
      const int i = threadIdx.x + 256 * j;
      if (i < kvec) out[i] = codes(v[j]);
    }
  } else {
    for (int i = threadIdx.x; i < kvec; i += 256) out[i] = codes(smooth8<true>(row[i], sv + 8 * i));
  }
}

// 16 output channels per workgroup (qqq_quantize_w4_perchannel on W .* s, then qqq_pack_w4): a wave takes four
// channels one after the other, its lanes hold the row (K <= 4096: in registers, s with it; else the row is smoothed
// twice, 4096 channels at a time), and the codes meet in LDS in the packed layout's order, so whole 1 KiB chunks are
// written.  About 7 instructions per weight and grid point, 3.2 us of the 6.3 that a grid point takes at K = N = 4096 (9.5 with the rounding,
// the clamp and the nibbles in fp32 and converted products); what else bounds it there, where 176 registers leave two waves a SIMD, is open.
// V: 64s of vectors of the row, a body of its own for each up to 8, so that short rows neither work on vectors that are not there nor hold
// registers for them (one body of 8 for all: a search of 17 points at M = 64, K = 128, N = 8192 157 us, 88 now; 12 points at M = 128, K = 2048,
// N = 4096 158, 142 now).  V = 0: any row, 8 at a time, in loops and 108 registers, four workgroups a CU (the channels written out, 142 registers and three
// workgroups: 5 points at M = 100, K = 8192, N = 3088 277 us, 244 now).
template <int V>
__global__ __launch_bounds__(256, V ? 1 : 4) void point_weights_kernel(const uint4* w, const float* s, int64_t s_bytes, int64_t N, int kvec,
                                                            int64_t point_bytes, uint8_t* packed, uint16_t* s_w) {
  constexpr bool ONE = V > 0;
  constexpr int kV = ONE ? V : 8;
  __shared__ uint32_t stage[4 * kV * 256];  // 1 KiB a k-step
  // the points of one group of channels run one after the other on the same XCD (workgroup ids go round the
  // eight of them), so its rows come from that XCD's L2 after the first
  const int64_t groups = N / 16;
  const int points = gridDim.y;
  const int64_t lin = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  int64_t nt;
  int pt;
  if (groups % 8 == 0) {
    const int64_t blk = lin / (8 * points), in = lin % (8 * points);
    nt = blk * 8 + in % 8;
    pt = (int)(in / 8);
  } else {
    nt = lin % groups;
    pt = (int)(lin / groups);
  }
  const int64_t off = point_bytes * pt;
  const float* sv = (const float*)((const char*)s + s_bytes * pt);
  uint32_t* out = (uint32_t*)(packed + off);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ float scales[ONE ? 1 : 16];
  uint4 v[kV];
  auto smooth_row = [&](const uint4* row, int i0) {
#pragma unroll
    for (int j = 0; j < kV; ++j) {
      const int i = i0 + lane + 64 * j;
      v[j] = i < kvec ? smooth8<false, true>(row[i], sv + 8 * i) : make_uint4(0, 0, 0, 0);
    }
  };
  auto scale_of_row = [&](int64_t n, const uint4* row) {
    uint32_t bits = 0;
    for (int i0 = 0; i0 < kvec; i0 += 512) {
      smooth_row(row, i0);
#pragma unroll
      for (int j = 0; j < kV; ++j) bits = absmax_bits(v[j], bits);
    }
    const uint16_t sb = weight_scale_bits(half_bits_to_float(wave_max_u32(bits)));
    if (lane == 0) ((uint16_t*)((char*)s_w + off))[n] = sb;
    return half_bits_to_float(sb);
  };
  // natural word i of channel nl = 16 nt + c: word (k-step i / 16, lane c + 16 kc, dword d) of the packed layout.  A wave writes
  // words of one c: the sixteen vectors of a kc are turned so that its four k-steps and four kc take all banks
  auto slot = [](int step, int kc, int c) { return 16 * kc + ((c + 4 * (step & 3) + kc) & 15); };
  auto put = [&](int c, float scale, int i0) {
    const float rs = __builtin_amdgcn_rcpf(scale);
    float cmax;
#pragma unroll
    for (int j = 0; j < kV; ++j) {
      const int i = lane + 64 * j;
      if (i0 + i >= kvec) continue;
      const uint32_t word = scale != 0.0f ? quant8<true>(v[j], scale, rs, &cmax) : 0u;
      const int o = i & 15, kc = (o & 7) >> 1, d = 2 * (o >> 3) + (o & 1);
      stage[(i >> 4) * 256 + slot(i >> 4, kc, c) * 4 + d] = word;
    }
  };
  auto flush = [&](int i0) {  // whole chunks of up to 32 k-steps
    __syncthreads();
    const int steps = min(32, (kvec - i0) >> 4);
    for (int e = threadIdx.x; e < steps * 64; e += 256)
      *reinterpret_cast<uint4*>(out + (((int64_t)(i0 >> 4) + (e >> 6)) * groups + nt) * 256 + (e & 63) * 4) =
          *reinterpret_cast<const uint4*>(&stage[(e & ~63) * 4 + slot(e >> 6, (e >> 4) & 3, e & 15) * 4]);
    __syncthreads();
  };
  if constexpr (ONE) {
    // the lanes keep their part of s for the four channels, and request the next channel's weights before they work on one
    float4 s0[kV], s1[kV];
    uint4 next[kV];
    auto request = [&](int q) {
      const uint4* row = w + (nt * 16 + 4 * wave + q) * kvec;
#pragma unroll
      for (int j = 0; j < kV; ++j) next[j] = row[min(lane + 64 * j, kvec - 1)];
    };
    request(0);
#pragma unroll
    for (int j = 0; j < kV; ++j) {
      const float4* from = reinterpret_cast<const float4*>(sv) + 2 * min(lane + 64 * j, kvec - 1);
      s0[j] = from[0];
      s1[j] = from[1];
    }
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      uint32_t bits = 0;
#pragma unroll
      for (int j = 0; j < kV; ++j) v[j] = smooth8<false, true>(next[j], s0[j], s1[j]);
      request(min(q + 1, 3));
#pragma unroll
      for (int j = 0; j < kV; ++j) bits = absmax_bits(v[j], bits);  // (past the row's end its last vector again)
      const uint16_t sb = weight_scale_bits(half_bits_to_float(wave_max_u32(bits)));
      if (lane == 0) ((uint16_t*)((char*)s_w + off))[nt * 16 + 4 * wave + q] = sb;
      put(4 * wave + q, half_bits_to_float(sb), 0);
    }
    flush(0);
  } else {
#pragma unroll 1
    for (int q = 0; q < 4; ++q) scales[4 * wave + q] = scale_of_row((nt * 16 + 4 * wave + q), w + (nt * 16 + 4 * wave + q) * kvec);
    for (int i0 = 0; i0 < kvec; i0 += 512) {
#pragma unroll 1
      for (int q = 0; q < 4; ++q) {
        const int c = 4 * wave + q;
        smooth_row(w + (nt * 16 + c) * kvec, i0);
        put(c, scales[c], i0);
      }
      flush(i0);
    }
  }
}

// ------------------------------------------------------------------ X W^T in fp32 (reference product of Eq. 2)

// 64 x 128 output tile per workgroup, a wave per 32 x 64 part of it (v_mfma_f32_32x32x16_f16, fp32 accumulation), 64 of
// K at a time through two LDS stages with the next four times 64 already requested (a workgroup is alone on its CU,
// so nothing else covers the latency: 62 us with the next 64 only).  Lane l holds row (A) / column (B) l % 32 and
// the 8 consecutive k of half l / 32; register v of the result is row 8*(v/4) + 4*(l/32) + v%4, column l % 32.  The
// 16-byte slots of a stage's row r are XOR-swizzled by (r/2)%8, which spreads both the writes and the 16 rows that a
// fragment read takes at a time over the banks.  Bound by the LDS reads (three fragments for two MFMAs); the tile is
// small so that a calibration batch fills the chip: M = 512, K = N = 4096 39 us (123 with one wave per 32 x 32 tile
// reading its fragments straight from memory).
__global__ __launch_bounds__(256) void fp16_gemm_nt_kernel(const uint4* x, const uint4* w, int M, int N, int kvec,
                                                           float* y) {
  __shared__ uint4 stage[2][192 * 8];  // 64 rows of X, then 128 of W, 8 vectors of 8 k each
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r32 = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 128;
  const int wm = (wave & 1) * 32, wn = 64 + (wave >> 1) * 64;  // the wave's first row of X and of W in a stage
  const uint4* src[6];
  int slot[6], col[6];
#pragma unroll
  for (int j = 0; j < 6; ++j) {  // (rows past M and N repeat the last one; their products are not stored)
    const int e = tid + 256 * j, r = e >> 3;
    col[j] = e & 7;
    slot[j] = r * 8 + (col[j] ^ ((r >> 1) & 7));
    src[j] = r < 64 ? x + (int64_t)min(m0 + r, M - 1) * kvec : w + (int64_t)min(n0 + r - 64, N - 1) * kvec;
  }
  uint4 next[4][6];  // (requested unconditionally, vectors past K clamped and zeroed on their way to LDS)
  auto fetch = [&](uint4 (&q)[6], int v0) {
#pragma unroll
    for (int j = 0; j < 6; ++j) q[j] = src[j][min(v0 + col[j], kvec - 1)];
  };
  v16f acc[2];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.0f;
  auto frag = [&](const uint4* st, int row, int s) {
    return __builtin_bit_cast(v8h, st[row * 8 + ((2 * s + h) ^ ((row >> 1) & 7))]);
  };
#pragma unroll
  for (int u = 0; u < 4; ++u) fetch(next[u], 8 * u);
  for (int v0 = 0; v0 < kvec; v0 += 32) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // (stages past K hold zeros)
      uint4* st = stage[u & 1];
#pragma unroll
      for (int j = 0; j < 6; ++j) st[slot[j]] = v0 + 8 * u + col[j] < kvec ? next[u][j] : make_uint4(0, 0, 0, 0);
      fetch(next[u], v0 + 8 * u + 32);
      lds_barrier();  // (the other stage is not written before everyone is past its reads)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const v8h a = frag(st, wm + r32, s), b0 = frag(st, wn + r32, s), b1 = frag(st, wn + 32 + r32, s);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b0, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b1, acc[1], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int n = n0 + wn - 64 + 32 * c + r32;
    if (n >= N) continue;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int m = m0 + wm + 8 * (v >> 2) + 4 * h + (v & 3);
      if (m < M) y[(int64_t)m * N + n] = acc[c][v];
    }
  }
}

// The same product for small problems: one wave per 32 x 32 tile, no LDS.  Lane l holds row (A) / column (B) l % 32 and the 8
// consecutive k of half l / 32 straight from memory (each lane walks its own row 16 bytes at a time); register v of the result
// as above.
__global__ __launch_bounds__(64) void fp16_gemm_nt_wave_kernel(const uint4* x, const uint4* w, int M, int N, int kvec, float* y) {
  const int lane = threadIdx.x, r32 = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  const uint4* xa = x + (int64_t)min(m0 + r32, M - 1) * kvec + h;
  const uint4* wb = w + (int64_t)min(n0 + r32, N - 1) * kvec + h;
  v16f acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  for (int i = 0; i < kvec; i += 2)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, xa[i]), __builtin_bit_cast(v8h, wb[i]), acc, 0, 0, 0);
  const int n = n0 + r32;
  if (n >= N) return;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int m = m0 + 8 * (v >> 2) + 4 * h + (v & 3);
    if (m < M) y[(int64_t)m * N + n] = acc[v];
  }
}

// ------------------------------------------------------------------ the grid's minimum

// The first minimum of the losses and, with its sigma, the smoothing vector and both smoothed matrices, in one launch (four of a few microseconds
// otherwise): every workgroup looks for the minimum itself.  A thread keeps eight channels' s and walks down the rows of X, then of W.
__global__ __launch_bounds__(256) void best_point_kernel(const double* losses, int G, const float* absmax, const float* sigmas, const uint4* x,
                                                         const uint4* w, int64_t M, int64_t N, int64_t kvec, uint4* xs, uint4* ws, float* s,
                                                         int32_t* best) {
  __shared__ double loss[256];
  if ((int)threadIdx.x < G) loss[threadIdx.x] = losses[threadIdx.x];
  __syncthreads();
  int b = 0;
  for (int g = 1; g < G; ++g)
    if (loss[g] < loss[b]) b = g;  // first minimum
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) best[0] = b;
  if (v >= kvec) return;
  const float sigma = sigmas[b];
  float4 a[2] = {reinterpret_cast<const float4*>(absmax)[2 * v], reinterpret_cast<const float4*>(absmax)[2 * v + 1]};
  float* e = reinterpret_cast<float*>(a);
#pragma unroll
  for (int i = 0; i < 8; ++i) e[i] = e[i] > sigma ? e[i] / sigma : 1.0f;
  if (blockIdx.y == 0) {
    reinterpret_cast<float4*>(s)[2 * v] = a[0];
    reinterpret_cast<float4*>(s)[2 * v + 1] = a[1];
  }
  int64_t r = blockIdx.y;
  for (; r < M; r += gridDim.y) xs[r * kvec + v] = smooth8<true>(x[r * kvec + v], a[0], a[1]);
#pragma unroll 4
  for (r -= M; r < N; r += gridDim.y) ws[r * kvec + v] = smooth8<false>(w[r * kvec + v], a[0], a[1]);
}

// loss += sum ( fp64(acc) * fp64(s_a[m]) * fp64(s_w[n]) - fp64(y_ref) )^2, fp64 throughout
__global__ __launch_bounds__(256) void smooth_loss_kernel(const int32_t* acc, const float* s_a, const uint16_t* s_w,
                                                          const float* y_ref, int64_t M, int64_t N, double* loss) {
  __shared__ double part[256];
  const int64_t total = M * N;
  const int64_t stride = (int64_t)gridDim.x * 256;
  double sum = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
    const int64_t m = i / N, n = i - m * N;
    const double d = (double)acc[i] * (double)s_a[m] * (double)half_bits_to_float(s_w[n]) - (double)y_ref[i];
    sum += d * d;
  }
  part[threadIdx.x] = sum;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(loss, part[0]);
}


static bool calib_shape_ok(int64_t M, int64_t N, int64_t K) {
  return M >= 1 && M <= 0x7FFFFFFF && N >= 16 && N % 16 == 0 && N <= 0x7FFFFFF0 && K >= 128 && K % 128 == 0 &&
         K <= 131072;
}

// Workspace of qqq_adaptive_smoothing: the channel maxima, X W^T, and room for the smoothing vectors and quantised
// operands of some grid points (M K + N K / 2 bytes and a little each; the terms below hold at least two)
static size_t smooth_workspace_bytes(int64_t M, int64_t N, int64_t K) {
  const size_t mk = (size_t)M * K, nk = (size_t)N * K, mn = (size_t)M * N;
  size_t total = 2 * align256c((size_t)K * 4) + 256 + align256c((size_t)M * 4) + align256c((size_t)N * 2);
  for (size_t bytes : {mn * 4, mk * 2, nk * 2, mk, nk / 2, nk / 2, mn * 4, mn * 2, qqq_gemm_workspace_bytes(M, N, K)})
    total += align256c(bytes);
  return total;
}

// sigmas: optional, the grid's G thresholds; losses, then, are set to 0 too
static int launch_absmax(const void* x, int64_t M, int64_t K, float* absmax, float* sigmas, int G, double* losses, hipStream_t st) {
  int rc = fill_u32(absmax, (size_t)K, 0u, st, losses, (size_t)G * 2);
  if (rc != QQQ_OK) return rc;
  const int64_t kvec = K / 8;
  int64_t row_blocks = (M + 31) / 32;
  if (row_blocks > 1024) row_blocks = 1024;
  const int64_t rows_per_block = (M + row_blocks - 1) / row_blocks;
  hipLaunchKernelGGL(channel_absmax_kernel, dim3((unsigned)((kvec + 31) / 32), (unsigned)row_blocks), dim3(256), 0,
                     st, (const uint4*)x, M, kvec, rows_per_block, (uint32_t*)absmax);
  rc = check_launch("channel_absmax");
  if (rc != QQQ_OK) return rc;
  hipLaunchKernelGGL(absmax_finish_kernel, dim3(1), dim3(1024), 0, st, (uint32_t*)absmax, K, sigmas, G);
  return check_launch("channel_absmax (finish)");
}

static int launch_smooth(const void* x, const void* w, const float* absmax, const float* sigmas, int64_t M, int64_t N, int64_t K, void* xs, void* ws, float* s, hipStream_t st) {
  hipLaunchKernelGGL(smoothing_vector_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, absmax, sigmas, K, s, (int64_t)0);
  int rc = check_launch("smoothing_vector");
  if (rc != QQQ_OK) return rc;
  const int64_t kvec = K / 8;
  auto blocks = [](int64_t total) { return (unsigned)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096); };
  hipLaunchKernelGGL((smooth_apply_kernel<true>), dim3(blocks(M * kvec)), dim3(256), 0, st, (const uint4*)x, s, M, kvec,
                     (uint4*)xs);
  rc = check_launch("smooth_apply (activations)");
  if (rc != QQQ_OK) return rc;
  hipLaunchKernelGGL((smooth_apply_kernel<false>), dim3(blocks(N * kvec)), dim3(256), 0, st, (const uint4*)w, s, N, kvec,
                     (uint4*)ws);
  return check_launch("smooth_apply (weights)");
}

// Which of the two: the tiles pay a fill of four stages of 64 k and a barrier each, the waves a memory latency per 16 k.  With
// operands that come from memory, as a layer's do, the waves are ahead up to K = 256 while they are few (M = 1, N = 300: K = 128 3.4 us
// against 5.4, K = 256 level to 9 % ahead) and where K is tiny at any size (M = 2048, N = 11008, K = 16: 16.6 us, bound by the output, against 35).
// From K = 512 on they are behind, 10 % there and up to 2.4 times beyond, although on operands that an L2 holds already they
// would still lead by up to 17 % at K = 512 .. 1040.
static bool waves_ahead(int64_t M, int64_t N, int64_t K) {
  return K <= 48 || (K <= 256 && ((M + 31) / 32) * ((N + 31) / 32) * K <= 180000);
}
static int launch_fp16_gemm(const void* x, const void* w, int64_t M, int64_t N, int64_t K, float* y, hipStream_t st) {
  if (waves_ahead(M, N, K)) {
    hipLaunchKernelGGL(fp16_gemm_nt_wave_kernel, dim3((unsigned)((N + 31) / 32), (unsigned)((M + 31) / 32)), dim3(64), 0, st,
                       (const uint4*)x, (const uint4*)w, (int)M, (int)N, (int)(K / 8), y);
    route_note("fp16 tile=32x32");
    return check_launch("fp16_gemm_nt (waves)");
  }
  hipLaunchKernelGGL(fp16_gemm_nt_kernel, dim3((unsigned)((N + 127) / 128), (unsigned)((M + 63) / 64)), dim3(256), 0, st,
                     (const uint4*)x, (const uint4*)w, (int)M, (int)N, (int)(K / 8), y);
  route_note("fp16 tile=64x128");
  return check_launch("fp16_gemm_nt");
}

// Several grid points per launch, or one point after the other through the hot path's own calls?  A launch for several has workgroups
// that walk all of K alone (16 channels' weights, a tile of the product), a point by itself costs its launches and the smoothed
// layer's way through memory.  Fitted to both on 4836 calls (M = 1 .. 1024, K = 128 .. 131072, N = 16 .. 8192, 1 to 20 points), in
// microseconds; the pick is 0.2 % behind the better one on average, the batches alone 12 % (M = 16, K = 131072, N = 16, 20 points 10.2 ms against
// 3.5; M = 16, K = 16384, N = 16, 20 points 1.06 against 0.63; M = 1, K = 8192, N = 256, one point 172 us against 119).
static bool steps_ahead(int64_t M, int64_t N, int64_t K, int grid_points, int at_once) {
  const double k = 1e-3 * (double)K, weights = k * 1e-3 * (double)N, activations = k * 1e-3 * (double)M;
  const int batches = (grid_points + at_once - 1) / at_once;
  return batches * (27.1 + (K > 4096 ? 8.0 : 4.6) * k) > grid_points * (25.0 + 1.2 * weights + 6.9 * activations) + 10.0;
}

}  // namespace qqq

using namespace qqq;

extern "C" {

int qqq_channel_absmax(const void* x_fp16, int64_t M, int64_t K, float* absmax, void* stream) {
  if (M < 1 || M > 0x7FFFFFFF || K < 8 || K % 8 != 0 || K > (1 << 24))
    return set_error(QQQ_ERR_SHAPE, "channel_absmax: unsupported M=%lld K=%lld (need K%%8==0)", (long long)M, (long long)K);
  if (!x_fp16 || !absmax) return set_error(QQQ_ERR_NULL, "channel_absmax: null pointer argument");
  if (!aligned16c(x_fp16) || (reinterpret_cast<uintptr_t>(absmax) & 3u))
    return set_error(QQQ_ERR_SHAPE, "channel_absmax: x must be 16-byte, absmax 4-byte aligned");
  return launch_absmax(x_fp16, M, K, absmax, nullptr, 0, nullptr, (hipStream_t)stream);
}

int qqq_smooth_apply(const void* x_fp16, const void* w_fp16, const float* absmax, const float* sigma, int64_t M,
                     int64_t N, int64_t K, void* xs_fp16, void* ws_fp16, float* s, void* stream) {
  if (M < 1 || N < 1 || M > 0x7FFFFFFF || N > 0x7FFFFFFF || K < 8 || K % 8 != 0 || K > (1 << 24))
    return set_error(QQQ_ERR_SHAPE, "smooth_apply: unsupported M=%lld N=%lld K=%lld (need K%%8==0)", (long long)M,
                     (long long)N, (long long)K);
  if (!x_fp16 || !w_fp16 || !absmax || !sigma || !xs_fp16 || !ws_fp16 || !s)
    return set_error(QQQ_ERR_NULL, "smooth_apply: null pointer argument");
  if (!aligned16c(x_fp16) || !aligned16c(w_fp16) || !aligned16c(xs_fp16) || !aligned16c(ws_fp16) || !aligned16c(s) ||
      (reinterpret_cast<uintptr_t>(absmax) & 3u) || (reinterpret_cast<uintptr_t>(sigma) & 3u))
    return set_error(QQQ_ERR_SHAPE, "smooth_apply: matrices and s must be 16-byte, absmax and sigma 4-byte aligned");
  return launch_smooth(x_fp16, w_fp16, absmax, sigma, M, N, K, xs_fp16, ws_fp16, s, (hipStream_t)stream);
}

int qqq_fp16_gemm_nt(const void* x_fp16, const void* w_fp16, int64_t M, int64_t N, int64_t K, float* y, void* stream) {
  route_reset();
  if (M < 1 || N < 1 || M > 0x7FFFFFF0 || N > 0x7FFFFFF0 || K < 16 || K % 16 != 0 || K > (1 << 24) ||
      (M + 31) / 32 > 65535)
    return set_error(QQQ_ERR_SHAPE, "fp16_gemm_nt: unsupported M=%lld N=%lld K=%lld (need K%%16==0, M <= 2097120)",
                     (long long)M, (long long)N, (long long)K);
  if (!x_fp16 || !w_fp16 || !y) return set_error(QQQ_ERR_NULL, "fp16_gemm_nt: null pointer argument");
  if (!aligned16c(x_fp16) || !aligned16c(w_fp16) || (reinterpret_cast<uintptr_t>(y) & 3u))
    return set_error(QQQ_ERR_SHAPE, "fp16_gemm_nt: x and w must be 16-byte, y 4-byte aligned");
  return launch_fp16_gemm(x_fp16, w_fp16, M, N, K, y, (hipStream_t)stream);
}

size_t qqq_smoothing_workspace_bytes(int64_t M, int64_t N, int64_t K) {
  if (!calib_shape_ok(M, N, K)) return 0;
  return smooth_workspace_bytes(M, N, K);
}

int qqq_adaptive_smoothing(const void* x_fp16, const void* w_fp16, int64_t M, int64_t N, int64_t K, int grid_points,
                           void* xs_fp16, void* ws_fp16, float* s, float* sigmas, double* losses, int32_t* best,
                           void* workspace, size_t workspace_bytes, void* stream) {
  route_reset();
  if (!calib_shape_ok(M, N, K) || (M + 31) / 32 > 65535)
    return set_error(QQQ_ERR_SHAPE, "adaptive_smoothing: unsupported M=%lld N=%lld K=%lld (need N%%16==0, K%%128==0, "
                     "128<=K<=131072, M <= 2097120)", (long long)M, (long long)N, (long long)K);
  if (grid_points < 1 || grid_points > 256)
    return set_error(QQQ_ERR_SHAPE, "adaptive_smoothing: grid_points must be in 1..256, got %d", grid_points);
  if (!x_fp16 || !w_fp16 || !xs_fp16 || !ws_fp16 || !s || !sigmas || !losses || !best || !workspace)
    return set_error(QQQ_ERR_NULL, "adaptive_smoothing: null pointer argument");
  if (!aligned16c(x_fp16) || !aligned16c(w_fp16) || !aligned16c(xs_fp16) || !aligned16c(ws_fp16) || !aligned16c(s) ||
      !aligned16c(workspace) || (reinterpret_cast<uintptr_t>(sigmas) & 3u) || (reinterpret_cast<uintptr_t>(losses) & 7u) ||
      (reinterpret_cast<uintptr_t>(best) & 3u))
    return set_error(QQQ_ERR_SHAPE, "adaptive_smoothing: matrices, s and workspace must be 16-byte aligned, sigmas and "
                     "best 4-byte, losses 8-byte");
  const size_t total = qqq_smoothing_workspace_bytes(M, N, K);
  if (workspace_bytes < total)
    return set_error(QQQ_ERR_WORKSPACE, "adaptive_smoothing: workspace %zu bytes < %zu needed", workspace_bytes, total);
  hipStream_t st = (hipStream_t)stream;
  char* base = (char*)workspace;
  size_t at = 0;
  auto take = [&](size_t bytes) { char* p = base + at; at += align256c(bytes); return p; };
  float* absmax = (float*)take((size_t)K * 4);
  float* y_ref = (float*)take((size_t)M * N * 4);
  // a grid point's smoothing vector and quantised operands; as many points at a time as the workspace holds
  const size_t first = at;
  float* s_point = (float*)take((size_t)K * 4);
  int8_t* a_q = (int8_t*)take((size_t)M * K);
  float* s_a = (float*)take((size_t)M * 4);
  uint8_t* packed = (uint8_t*)take((size_t)N * K / 2);
  uint16_t* s_w = (uint16_t*)take((size_t)N * 2);
  const int64_t point_bytes = (int64_t)(at - first);
  const int64_t room = (int64_t)(total - first) / point_bytes;  // at least two: see smooth_workspace_bytes
  const int at_once = room < grid_points ? (int)room : grid_points;

  int rc = launch_absmax(x_fp16, M, K, absmax, sigmas, grid_points, losses, st);
  if (rc != QQQ_OK) return rc;
  if ((rc = launch_fp16_gemm(x_fp16, w_fp16, M, N, K, y_ref, st)) != QQQ_OK) return rc;
  const int64_t column_blocks = (K / 8 + 255) / 256;
  // an input lies in the smoothed weights' place (a layer may be smoothed in place)
  const auto holds = [&](const void* in, int64_t rows) {
    const uintptr_t at_in = reinterpret_cast<uintptr_t>(in), at_ws = reinterpret_cast<uintptr_t>(ws_fp16);
    return at_in < at_ws + (uintptr_t)N * K * 2 && at_ws < at_in + (uintptr_t)rows * K * 2;
  };
  auto apply_best = [&](int64_t m, int64_t n) {  // (two rounds of workgroups: a thread's rows are requested four at a time)
    const int64_t rows = 8 * num_cus() / column_blocks;
    hipLaunchKernelGGL(best_point_kernel, dim3((unsigned)column_blocks, (unsigned)(rows < 1 ? 1 : rows < m + n ? rows : m + n)), dim3(256), 0, st, losses,
                       grid_points, absmax, sigmas, (const uint4*)x_fp16, (const uint4*)w_fp16, m, n, K / 8, (uint4*)xs_fp16, (uint4*)ws_fp16, s, best);
    return check_launch("best point");
  };
  auto finish = [&]() {
    if (!holds(x_fp16, M)) return apply_best(M, N);
    const int done = apply_best(M, 0);  // the smoothed weights go where X is read: X first
    return done != QQQ_OK ? done : apply_best(0, N);
  };
  if (steps_ahead(M, N, K, grid_points, at_once)) {
    // a point at a time through the hot path's own calls, the smoothed layer, its codes and their product in the workspace
    at = first;
    char* xs = take((size_t)M * K * 2);
    char* ws = take((size_t)N * K * 2);
    s_point = (float*)take((size_t)K * 4);
    a_q = (int8_t*)take((size_t)M * K);
    s_a = (float*)take((size_t)M * 4);
    uint32_t* w_nat = (uint32_t*)take((size_t)N * K / 2);
    s_w = (uint16_t*)take((size_t)N * 2);
    packed = (uint8_t*)take((size_t)N * K / 2);
    int32_t* acc = (int32_t*)take((size_t)M * N * 4);
    char* y = take((size_t)M * N * 2);
    const size_t gemm_bytes = qqq_gemm_workspace_bytes(M, N, K);
    char* gemm_ws = take(gemm_bytes);
    if ((rc = fill_u32(gemm_ws, (gemm_bytes + 3) / 4, 0u, st)) != QQQ_OK) return rc;
    const int64_t elements = M * N;
    const unsigned blocks = (unsigned)((elements + 255) / 256 < 2048 ? (elements + 255) / 256 : 2048);
    for (int g = 0; g < grid_points; ++g) {
      if ((rc = launch_smooth(x_fp16, w_fp16, absmax, sigmas + g, M, N, K, xs, ws, s_point, st)) != QQQ_OK) return rc;
      if ((rc = qqq_quant_act(xs, M, K, K, a_q, s_a, stream)) != QQQ_OK) return rc;
      if ((rc = qqq_quantize_w4_perchannel(ws, N, K, K, w_nat, s_w, stream)) != QQQ_OK) return rc;
      if ((rc = qqq_pack_w4(w_nat, N, K, packed, stream)) != QQQ_OK) return rc;
      if ((rc = qqq_gemm_w4a8_perchannel(a_q, s_a, packed, s_w, y, acc, M, N, K, gemm_ws, gemm_bytes, stream)) != QQQ_OK) return rc;
      hipLaunchKernelGGL(smooth_loss_kernel, dim3(blocks), dim3(256), 0, st, acc, s_a, s_w, y_ref, M, N, losses + g);
      if ((rc = check_launch("smooth_loss")) != QQQ_OK) return rc;
    }
    route_note("loss");
    return finish();
  }
  GemmParams p = {};
  p.a_q = a_q;
  p.s_a = s_a;
  p.w = (const uint4*)packed;
  p.s_w = (const _Float16*)s_w;
  p.M = (int)M;
  p.N = (int)N;
  p.K = (int)K;
  p.T = (int)(K / 128);
  p.k_splits = 1;
  p.y_ref = y_ref;
  p.point_bytes = point_bytes;
  const int kvec = (int)(K / 8);
  // all points' smoothing vectors at once where the smoothed weights' place, which is written last, holds them and no input
  float* vectors = 2 * grid_points <= N && !holds(w_fp16, N) && !holds(x_fp16, M) ? (float*)ws_fp16 : nullptr;
  if (vectors)
    hipLaunchKernelGGL(smoothing_vector_kernel, dim3((unsigned)((K + 255) / 256), (unsigned)grid_points), dim3(256), 0, st, absmax,
                       sigmas, K, vectors, K * 4);
  for (int g = 0; g < grid_points; g += at_once) {
    // the candidates' smoothed layers, quantised as the hot path quantises them, and their losses
    const unsigned points = (unsigned)(grid_points - g < at_once ? grid_points - g : at_once);
    if (vectors == nullptr)
      hipLaunchKernelGGL(smoothing_vector_kernel, dim3((unsigned)((K + 255) / 256), points), dim3(256), 0, st, absmax,
                         sigmas + g, K, s_point, point_bytes);
    const float* s_of = vectors ? vectors + g * K : s_point;
    const int64_t s_bytes = vectors ? K * 4 : point_bytes;
    auto activations = K <= 8192 ? point_activations_kernel<true> : point_activations_kernel<false>;
    hipLaunchKernelGGL(activations, dim3((unsigned)M, points), dim3(256), 0, st, (const uint4*)x_fp16, s_of, s_bytes, kvec,
                       point_bytes, a_q, s_a);
    static constexpr decltype(&point_weights_kernel<0>) kWeights[9] = {
        point_weights_kernel<0>, point_weights_kernel<1>, point_weights_kernel<2>, point_weights_kernel<3>, point_weights_kernel<4>,
        point_weights_kernel<5>, point_weights_kernel<6>, point_weights_kernel<7>, point_weights_kernel<8>};
    const auto weights = kWeights[K <= 4096 ? (K + 511) / 512 : 0];
    hipLaunchKernelGGL(weights, dim3((unsigned)(N / 16), points), dim3(256), 0, st, (const uint4*)w_fp16, s_of, s_bytes, N, kvec,
                       point_bytes, packed, s_w);
    if ((rc = check_launch("smoothing grid point")) != QQQ_OK) return rc;
    p.loss = losses + g;
    if ((rc = launch_gemm_loss(p, (int)points, st)) != QQQ_OK) return rc;
  }
  return finish();
}

}  // extern "C"
