// Hessian of Sec. 3.2 (H = 2 X^T X over the calibration tokens), entry point qqq_hessian of include/qqq_calib.h.
#include "qqq_calib.h"
#include "qqq_internal.h"

#include <type_traits>

#pragma clang fp contract(off)

namespace qqq {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

// pair (p <= q) number u of a triangle, column by column
struct Pair { int p, q; };
__device__ __forceinline__ Pair triangle_pair(int64_t u) {
  int q = (int)((__builtin_sqrtf(8.0f * (float)u + 1.0f) - 1.0f) * 0.5f);
  while ((int64_t)(q + 1) * (q + 2) / 2 <= u) ++q;
  while ((int64_t)q * (q + 1) / 2 > u) --q;
  return {(int)(u - (int64_t)q * (q + 1) / 2), q};
}

template <int TE>
struct TileStage {
  static constexpr int kTok = 2048 / TE, kStride = TE == 64 ? 72 : 48;
  static constexpr int kTr = TE / 2 + 1;  // row stride of a quarter on its way to the mirrored place
  union {
    uint16_t x[2][kTok * kStride];
    double t[4][TE / 2 * kTr];
  };
};

// H = 2 X^T X in fp64 on the fp64 matrix cores.  H is symmetric: 256 threads per TE x TE tile on or above
// the diagonal, written to both places.  Both operands are columns of X, kept in LDS as the fp16 they are
// (2048 / TE tokens at a time, the next ones already requested) and widened when a fragment is read:
// v_mfma_f64_16x16x4_f64 takes 64 clocks, so the widening and the LDS reads are free next to it.  Lane l holds
// column l % 16 and token l / 16 of both operands; register v of the result is row 4 v + l / 16, column l % 16.
// Row strides of the stages (72 and 48 halves) keep the four token rows of a fragment on different banks.
// A wave holds a (TE/2) x (TE/2) quarter.  TE = 64 reads each fragment for two MFMAs; TE = 32 is for narrow layers,
// where 64 x 64 tiles leave CUs idle.
// Bound: the fp64 matrix rate (78.6 TFLOP/s nominal).  K = 4096, 2048 tokens: 0.68 ms, 51 TFLOP/s of the one
// triangle (3.66 ms with both triangles on vector multiply-adds); K = 2048, 1111 tokens: 0.136 ms (0.55).
// VEC: rows of X are 16-byte aligned (K % 8 == 0 and an aligned base); else element by element.
template <int TE, bool VEC>
__device__ __forceinline__ void hessian_tile(const _Float16* x, int64_t M, int64_t K, double* H, int ti, int tj, TileStage<TE>& sm) {
  constexpr int kTok = TileStage<TE>::kTok, kStride = TileStage<TE>::kStride, kTr = TileStage<TE>::kTr, kW = TE / 32, kVecs = TE / 8;
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, q = lane >> 4;
  const int wr = (wave >> 1) * (TE / 2), wc = (wave & 1) * (TE / 2);
  const int64_t c0[2] = {(int64_t)ti * TE, (int64_t)tj * TE};
  const int srow = tid / kVecs, scol = 8 * (tid % kVecs);  // this thread's 8 elements of a stage

  uint4 next[2];
  auto fetch = [&](int64_t m0) {  // tokens past M and channels past K feed zeros
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int64_t m = m0 + srow, c = c0[o] + scol;
      if constexpr (VEC) {
        next[o] = (m < M && c < K) ? *reinterpret_cast<const uint4*>(x + m * K + c) : make_uint4(0, 0, 0, 0);
      } else {
        uint32_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          e[i] = (m < M && c + i < K) ? (uint32_t)reinterpret_cast<const uint16_t*>(x)[m * K + c + i] : 0u;
        next[o] = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
      }
    }
  };
  v4d acc[kW][kW];
#pragma unroll
  for (int i = 0; i < kW; ++i)
#pragma unroll
    for (int j = 0; j < kW; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};
  fetch(0);
  for (int64_t m0 = 0; m0 < M; m0 += kTok) {
#pragma unroll
    for (int o = 0; o < 2; ++o) *reinterpret_cast<uint4*>(&sm.x[o][srow * kStride + scol]) = next[o];
    __syncthreads();
    if (m0 + kTok < M) fetch(m0 + kTok);
#pragma unroll
    for (int s = 0; s < kTok / 4; ++s) {
      double a[kW], b[kW];
#pragma unroll
      for (int i = 0; i < kW; ++i) {
        a[i] = (double)half_bits_to_float(sm.x[0][(4 * s + q) * kStride + wr + 16 * i + l16]);
        b[i] = (double)half_bits_to_float(sm.x[1][(4 * s + q) * kStride + wc + 16 * i + l16]);
      }
#pragma unroll
      for (int i = 0; i < kW; ++i)
#pragma unroll
        for (int j = 0; j < kW; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  double* const tr = sm.t[wave];
#pragma unroll
  for (int i = 0; i < kW; ++i)
#pragma unroll
    for (int j = 0; j < kW; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * i + 4 * v + q, c = 16 * j + l16;
        const double h = 2.0 * acc[i][j][v];
        const int64_t gi = c0[0] + wr + r, gj = c0[1] + wc + c;
        if (gi < K && gj < K) H[gi * K + gj] = h;
        tr[c * kTr + r] = h;
      }
  if (ti == tj) return;  // the whole diagonal tile was computed, both halves bit for bit alike
  // mirrored: rows of the quarter's transpose, from the wave's own patch (one wave's LDS accesses stay in order)
  constexpr int kE = TE / 2;
  for (int e = lane; e < kE * kE; e += 64) {
    const int c = e / kE, r = e % kE;
    const int64_t gi = c0[1] + wc + c, gj = c0[0] + wr + r;
    if (gi < K && gj < K) H[gi * K + gj] = tr[c * kTr + r];
  }
}

template <int TE, bool VEC>
__global__ __launch_bounds__(256, 4) void hessian_kernel(const _Float16* x, int64_t M, int64_t K, double* H) {
  __shared__ __attribute__((aligned(16))) TileStage<TE> sm;
  const Pair t = triangle_pair(blockIdx.x);
  hessian_tile<TE, VEC>(x, M, K, H, t.p, t.q, sm);
}

// The same sums on the int8 matrix cores, exactly.  An fp16 value is an integer multiple of 2^-24; below 127.5 in magnitude that
// integer is four digits d_p of base 256, each in [-128, 127], so that
//     sum x y = 2^-48 sum_L 256^L T_L,   T_L = sum over tokens and p + q = L of d_p(x) d_q(y),  L = 0 .. 6:
// sixteen int8 products whose int32 sums are exact (|T_L| <= 5 * 2^14 M, M <= kMaxTokens), put together in 64-bit integers and rounded to
// fp64 once.  (The fp64 products round whenever the running sum outgrows 53 bits.)  Sixteen of 5 POP/s nominal are four times
// the fp64 matrix cores' 78.6 TFLOP/s.
// Larger values: from the stage on that shows one, a tile takes five digits (enough below 32640; twenty-five products, L = 0 .. 8), on top
// of the sums that it has, so nothing is done twice, wherever in the tokens they stand.  Only a value from 32640 on, an infinity or a NaN has
// its tiles done by hessian_tile, from the first token.
// Tile: 64 x 64 of H by 4 waves, 32 x 32 each: seven levels of a 32 x 32 accumulator are 112 registers, so a CU takes two
// workgroups, one splitting while the other multiplies.  A stage is 64 tokens: every thread takes 4 tokens of 4 channels twice, splits
// them (an fp16 value times 2^24 is exact in fp32; adding 0x808080 makes the bytes of the integer the digits plus 128) and stores the
// digits of 4 tokens as a word in [digit][channel][token] order, the operand order of v_mfma_i32_32x32x32_i8, 16-byte slots of a channel
// XOR-swizzled by (channel / 4) % 4 and 64 bytes left free after 16 channels (fragment reads and stores take all banks once).  The next
// stage is split between this one's products, twelve vector instructions to a product (the split ends early: 4 and 8 took 6 % longer, 20
// and 30 1-3 %), and what it splits was requested half a stage before, through the buffer's range check: with a branch for the tokens
// past M the compiler waited for all requests at once.
// Bound: 32 MFMAs of 32 clocks and 242 vector instructions of 4 a wave and stage, two waves on a SIMD; without the split a launch takes
// 174 us of the 270, so products and split overlap little.  [M, K] = [2048, 4096]: 271 us (hessian_kernel 680), [1111, 2048]: 58 (134),
// [2048, 1024]: 41 (74), [300, 1024]: 13.4 (16.5).  With large values, [2048, 4096], hessian_kernel 680: in 0.2, 1 and 5 % of the channels 314, 366
// and 410 us, everywhere 406, in the last token of every channel 299; [2048, 1024], hessian_kernel 75: 62 and in the last token 46.
// (hessian_tile from the stage on that shows one, as for infinities: 442, 606, 706, 706, 932; 101 and 132.)
constexpr int kMaxTokens = 16384;
constexpr int kFour = 0x57F8, kFive = 0x77F8;  // fp16 bits of 127.5 and 32640: what four and five digits hold lies below

__global__ __launch_bounds__(256, 2) void hessian_digits_kernel(const _Float16* x, int M, int K, double* H) {
  constexpr int kPlane = 128 * 64 + 8 * 64, kStage = 4 * kPlane;  // channel c at 64 (c + c / 16)
  __shared__ __attribute__((aligned(16))) union {
    int8_t d[2 * kStage];
    TileStage<64> tile;
  } sm;
  __shared__ int s_large[2], s_over[2];  // the stage in buffer 0 / 1 of sm.d holds a value from 127.5 on, from 32640 on
  const Pair t = triangle_pair(blockIdx.x);
  const int r0 = t.p * 64, c0 = t.q * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kb = lane >> 4, wr = wave >> 1, wc = wave & 1;
  if (tid < 2) s_large[tid] = s_over[tid] = 0;

  // what this thread splits: for two of a stage's four 16-byte slots (16 tokens) 4 tokens, 4 kb .., of channels 4 l16 .. of the tile's
  // rows (waves 0, 1) or columns (2, 3)
  const int panel = wave >> 1, slot0 = 2 * (wave & 1);
  const int channel = min((panel ? c0 : r0) + 4 * l16, K - 4);  // (K % 8 == 0; channels past it are not stored)
  const int row0 = 64 * panel + 4 * l16, store0 = (row0 + row0 / 16) * 64 + 4 * kb, turn = l16 & 3;
  // (tokens past M: the buffer's range check makes them 0)
  const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(x), 0, M * K * 2, 0x00020000);
  const uint32_t row_bytes = 2u * K;
  uint32_t at0 = (uint32_t)(16 * slot0 + 4 * kb) * row_bytes + 2u * channel;  // of the next stage to request
  u2 raw[2][4];
  auto request = [&](int i) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      raw[i][j] = __builtin_amdgcn_raw_buffer_load_b64(rows, at0 + (16 * i + j) * row_bytes, 0, 0);
    if (i) at0 += 64 * row_bytes;
  };
  typedef unsigned short us2 __attribute__((ext_vector_type(2)));
  us2 top = {0, 0};  // largest magnitude seen, as bits
  // Channels 2 pair, 2 pair + 1 of the four.  From 128 on, and for infinities and NaN, the conversion leaves the range of int (in five digits:
  // infinities and NaN); this relies on v_cvt_i32_f32 giving some integer there.  Which does not matter: its products are taken off
  // again or thrown away
  auto split = [&](int i, int pair, int8_t* to) {
    uint32_t m[2][4];  // the integers + 0x808080
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t two = pair ? raw[i][j][1] : raw[i][j][0];
      top = __builtin_elementwise_max(top, __builtin_bit_cast(us2, two & 0x7FFF7FFFu));
      m[0][j] = (uint32_t)(int)__builtin_fmaf(half_bits_to_float(two & 0xFFFFu), 16777216.0f, 0.0f) + 0x808080u;
      m[1][j] = (uint32_t)(int)__builtin_fmaf(half_bits_to_float(two >> 16), 16777216.0f, 0.0f) + 0x808080u;
    }
    int8_t* at = to + store0 + (((slot0 + i) ^ turn) << 4);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      // 4 x 4 bytes transposed; v_perm_b32: selector bytes 0-3 pick from the second source, 4-7 from the first
      const uint32_t a = __builtin_amdgcn_perm(m[e][1], m[e][0], 0x05010400u), b = __builtin_amdgcn_perm(m[e][3], m[e][2], 0x05010400u);
      const uint32_t c = __builtin_amdgcn_perm(m[e][1], m[e][0], 0x07030602u), d = __builtin_amdgcn_perm(m[e][3], m[e][2], 0x07030602u);
      const uint32_t digit[4] = {__builtin_amdgcn_perm(b, a, 0x05040100u) ^ 0x80808080u, __builtin_amdgcn_perm(b, a, 0x07060302u) ^ 0x80808080u,
                                 __builtin_amdgcn_perm(d, c, 0x05040100u) ^ 0x80808080u, __builtin_amdgcn_perm(d, c, 0x07060302u)};
#pragma unroll
      for (int p = 0; p < 4; ++p) *reinterpret_cast<uint32_t*>(at + p * kPlane + 64 * (2 * pair + e)) = digit[p];
    }
  };

  // Five digits, in stages of 32 tokens (two stages of five planes fit where two of 64 tokens and four do): 4 tokens, 4 kb .., of slot wave % 2.
  // Adding 1.5 * 2^23 rounds x to a whole number, which then stands in the sum's low bits: the upper two digits come from it (128 added) and the carry
  // of the lower three, those from 2^24 times what is left of x (at most 2^23; kMagic's part taken out by one multiply-add), all exact.
  // 32 bytes left free after 16 channels, slots XOR-swizzled by (channel / 8) % 2: all banks once, as above
  constexpr int kPlane5 = kPlane / 2, kStage5 = 5 * kPlane5;
  const int store5 = (row0 + row0 / 16) * 32 + 4 * kb + (((wave & 1) ^ ((l16 >> 1) & 1)) << 4);
  auto request5 = [&](int i) {
#pragma unroll
    for (int j = 0; j < 4; ++j) raw[i][j] = __builtin_amdgcn_raw_buffer_load_b64(rows, at0 + j * row_bytes, 0, 0);
    at0 += 32 * row_bytes;
  };
  auto split5 = [&](int i, int pair, int8_t* to) {
    uint32_t lo[2][4], hi[2][4];  // the lower integer + 0x808080; the upper + 0x80 in the low half
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t two = pair ? raw[i][j][1] : raw[i][j][0];
      top = __builtin_elementwise_max(top, __builtin_bit_cast(us2, two & 0x7FFF7FFFu));
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        constexpr float kMagic = 12582912.0f + 128.0f;
        const float v = half_bits_to_float(e ? two >> 16 : two & 0xFFFFu), t = __builtin_fmaf(v, 1.0f, kMagic);
        const float left = __builtin_fmaf(v, 16777216.0f, __builtin_fmaf(t, -16777216.0f, kMagic * 16777216.0f));
        lo[e][j] = (uint32_t)(int)left + 0x808080u;
        hi[e][j] = __builtin_bit_cast(uint32_t, t) + (lo[e][j] >> 24);
      }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      auto bytes = [](const uint32_t (&w)[4], uint32_t select) {  // two bytes of each of the four words, byte by byte
        return make_uint2(__builtin_amdgcn_perm(w[1], w[0], select), __builtin_amdgcn_perm(w[3], w[2], select));
      };
      const uint2 l01 = bytes(lo[e], 0x05010400u), l2 = bytes(lo[e], 0x07030602u), h = bytes(hi[e], 0x05010400u);
      const uint32_t digit[5] = {__builtin_amdgcn_perm(l01.y, l01.x, 0x05040100u) ^ 0x80808080u, __builtin_amdgcn_perm(l01.y, l01.x, 0x07060302u) ^ 0x80808080u,
                                 __builtin_amdgcn_perm(l2.y, l2.x, 0x05040100u) ^ 0x80808080u, __builtin_amdgcn_perm(h.y, h.x, 0x05040100u) ^ 0x80808080u,
                                 __builtin_amdgcn_perm(h.y, h.x, 0x07060302u)};
#pragma unroll
      for (int p = 0; p < 5; ++p) *reinterpret_cast<uint32_t*>(to + store5 + p * kPlane5 + 32 * (2 * pair + e)) = digit[p];
    }
  };

  v16i acc[9];
#pragma unroll
  for (int l = 0; l < 7; ++l)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[l][v] = 0;
  // this lane's fragments: channel lane % 32 of the wave's rows / columns, tokens 32 k + 16 (lane / 32) .. of k-step k
  const int l32 = lane & 31, at32 = (l32 + l32 / 16) * 64, half = lane >> 5, turn32 = (l32 >> 2) & 3;
  const int fk[2] = {at32 + ((half ^ turn32) << 4), at32 + (((2 + half) ^ turn32) << 4)};
  const int fa = 34 * wr * 64, fb = (68 + 34 * wc) * 64;  // (17 rows of 64 bytes for 16 channels)

  request(0);
  request(1);
  __syncthreads();  // (s_large and s_over are zero)
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    split(i, 0, sm.d);
    split(i, 1, sm.d);
    __builtin_amdgcn_sched_barrier(0);
    request(i);
    __builtin_amdgcn_sched_barrier(0);
  }
  auto shown = [&](int limit) { return max((int)top[0], (int)top[1]) >= limit; };
  if (shown(kFour)) s_large[0] = 1;
  __syncthreads();
  int stage = 0, m0 = 0;
  const int at_once = __builtin_amdgcn_readfirstlane(s_large[0]);
  int large = at_once;
  for (; (m0 < M) & !large; m0 += 64) {
    const int8_t* s = sm.d + stage * kStage;
    int8_t* next = sm.d + (stage ^ 1) * kStage;  // (behind the last stage: zeros, not used)
    const int flag = s_large[stage];  // (set before the last barrier, and not again in this stage: all waves read alike)
    v4i a[2], b[2][4];
    auto read_a = [&](int g) { a[g & 1] = *reinterpret_cast<const v4i*>(s + (g & 3) * kPlane + fa + fk[g >> 2]); };
    auto read_b = [&](int k, int q) { b[k][q] = *reinterpret_cast<const v4i*>(s + q * kPlane + fb + fk[k]); };
    read_a(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) read_b(0, q);
#pragma unroll
    for (int g = 0; g < 8; ++g) {  // digit g % 4 of the rows, k-step g / 4
      if (g < 7) read_a(g + 1);
      if (g < 4) read_b(1, g);
      if (!(g & 1)) split(g >> 2, (g >> 1) & 1, next);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[(g & 3) + q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[g & 1], b[g >> 2][q], acc[(g & 3) + q], 0, 0, 0);
      if (g & 1) {
#pragma unroll
        for (int n = 0; n < 8; ++n) {  // a product, then vector instructions that fit in its 32 clocks
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
        }
        if (g & 2) request(g >> 2);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (shown(kFour)) s_large[stage ^ 1] = 1;
    large = __builtin_amdgcn_readfirstlane(flag);
    __syncthreads();
    stage ^= 1;
  }
  const bool five = large;  // (uniform)
  if (five) {
    if (!at_once) m0 -= 64, stage ^= 1;
#pragma unroll
    for (int l = 7; l < 9; ++l)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[l][v] = 0;
    // That stage's digits are none of its values', and it was multiplied before the flag had come (waiting for the flag took 1 to 5 % longer
    // where nothing is large): its products off again, as -a b = ~a b + b
    const int8_t* s = sm.d + stage * kStage;
    if (!at_once)
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const v4i a = ~*reinterpret_cast<const v4i*>(s + (g & 3) * kPlane + fa + fk[g >> 2]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const v4i b = *reinterpret_cast<const v4i*>(s + q * kPlane + fb + fk[g >> 2]);
        acc[(g & 3) + q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc[(g & 3) + q], 0, 0, 0);
        acc[(g & 3) + q] = __builtin_amdgcn_mfma_i32_32x32x32_i8((v4i)0x01010101, b, acc[(g & 3) + q], 0, 0, 0);
      }
    }
    const int fk5 = (l32 + l32 / 16) * 32 + ((half ^ ((l32 >> 3) & 1)) << 4);
    int over = 0;
    auto multiply = [&](auto buffer) {  // the stage in it, while the next is split into the other
      constexpr int kThis = decltype(buffer)::value, kNext = kThis ^ 1;
      const int8_t* s = sm.d + kThis * kStage5 + fk5;
      over |= s_over[kThis];  // (set before the last barrier, and not again in this stage)
      v4i a[2], b[5];
      auto read_a = [&](int p) { a[p & 1] = *reinterpret_cast<const v4i*>(s + p * kPlane5 + fa / 2); };
      read_a(0);
#pragma unroll
      for (int q = 0; q < 5; ++q) b[q] = *reinterpret_cast<const v4i*>(s + q * kPlane5 + fb / 2);
#pragma unroll
      for (int p = 0; p < 5; ++p) {
        if (p < 4) read_a(p + 1);
        if (p == 0 || p == 2) split5(kNext, p / 2, sm.d + kNext * kStage5);
#pragma unroll
        for (int q = 0; q < 5; ++q) acc[p + q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[p & 1], b[q], acc[p + q], 0, 0, 0);
        if (p & 1) {
#pragma unroll
          for (int n = 0; n < 10; ++n) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
          }
          if (p == 3) request5(kNext);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (shown(kFive)) s_over[kNext] = 1;
      __syncthreads();
    };
    at0 = (uint32_t)(m0 + 16 * (wave & 1) + 4 * kb) * row_bytes + 2u * channel;
    request5(0);
    request5(1);
    __syncthreads();  // (every wave has read the buffers)
    split5(0, 0, sm.d);
    split5(0, 1, sm.d);
    request5(0);
    if (shown(kFive)) s_over[0] = 1;
    __syncthreads();
#pragma nounroll
    for (; m0 < M && !__builtin_amdgcn_readfirstlane(over); m0 += 64) {  // (a way out between the two makes the compiler hold the sums twice)
      multiply(std::integral_constant<int, 0>{});
      multiply(std::integral_constant<int, 1>{});
    }
    if (__builtin_amdgcn_readfirstlane(over)) {  // (behind a barrier)
      hessian_tile<64, true>(x, M, K, H, t.p, t.q, sm.tile);
      return;
    }
  }
  // register v of a 32 x 32 tile is row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32; the factor 2 * 2^-48 is exact
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    int64_t lo = (int64_t)acc[0][v] + ((int64_t)acc[1][v] << 8) + ((int64_t)acc[2][v] << 16);
    double h;
    if (!five) {
      const int64_t hi = (int64_t)acc[3][v] + ((int64_t)acc[4][v] << 8) + ((int64_t)acc[5][v] << 16) + ((int64_t)acc[6][v] << 24) + (lo >> 24);
      lo &= 0xFFFFFF;
      h = __builtin_fma((double)hi, 16777216.0, (double)lo) * 0x1p-47;  // |hi| < 2^53: both are exact, so this rounds the sum once
    } else {
      lo += (int64_t)acc[3][v] << 24;
      const int64_t hi = (int64_t)acc[4][v] + ((int64_t)acc[5][v] << 8) + ((int64_t)acc[6][v] << 16) + ((int64_t)acc[7][v] << 24) +
                         ((int64_t)acc[8][v] << 32) + (lo >> 32);
      const uint64_t low = (uint32_t)lo;
      // The sum is hi 2^32 + low, |hi| < 2^61.  Its 62 leading bits as an integer, the lowest of them set if anything below is: the
      // conversion rounds that as it would the whole
      const int shift = min(32, __builtin_clzll((uint64_t)(hi < 0 ? ~hi : hi) | 1) - 1);
      const uint64_t rest = low << shift;
      const int64_t lead = (int64_t)(((uint64_t)hi << shift) + (rest >> 32)) | ((uint32_t)rest != 0);
      h = __builtin_ldexp((double)lead, -15 - shift);
    }
    const int64_t gi = r0 + 32 * wr + 8 * (v >> 2) + 4 * half + (v & 3), gj = c0 + 32 * wc + l32;
    if (gi < K && gj < K) {
      H[gi * K + gj] = h;
      H[gj * K + gi] = h;
    }
  }
}

}  // namespace

}  // namespace qqq

using namespace qqq;

extern "C" {

int qqq_hessian(const void* x_fp16, int64_t M, int64_t K, double* H, void* stream) {
  if (M < 1 || M > 0x7FFFFFFF || K < 1 || K > 16384)
    return set_error(QQQ_ERR_SHAPE, "hessian: unsupported M=%lld K=%lld (need 1 <= K <= 16384)", (long long)M, (long long)K);
  if (!x_fp16 || !H) return set_error(QQQ_ERR_NULL, "hessian: null pointer argument");
  if ((reinterpret_cast<uintptr_t>(x_fp16) & 1u) || (reinterpret_cast<uintptr_t>(H) & 7u))
    return set_error(QQQ_ERR_SHAPE, "hessian: x must be 2-byte, H 8-byte aligned");
  auto tiles = [&](int64_t te) { const int64_t t = (K + te - 1) / te; return t * (t + 1) / 2; };
  // 64 x 64 tiles where they give every CU at least two, else 32 x 32
  const int64_t cus = num_cus();
  const bool wide = tiles(64) >= 2 * cus;
  const bool vec = K % 8 == 0 && (reinterpret_cast<uintptr_t>(x_fp16) & 15u) == 0;
  // Digits where a CU in two has a 64 x 64 tile, from so many stages of 64 tokens on that they gain at least about what large values in every
  // channel can make them lose: more stages the fewer rounds of 32 x 32 tiles the fp64 products take.  us, fp64 / digits / digits with
  // large values everywhere: K = 968 M = 640 20.8 17.5 25.2, M = 1024 30.0 23.3 34.4; K = 1024 M = 192 11.0 10.3 13.6, M = 256 13.1 11.2 15.3; K = 1280
  // M = 128 11.0 10.6 12.9, M = 192 13.8 11.7 14.5; K = 1536 M = 256 19.2 17.3 21.8, M = 320 22.6 18.8 24.4; K = 2048 M = 96 18.9 19.3 24.2, M = 128
  // 22.6 19.5 24.4; K = 4096 M = 128 53.6 44.4 57.6.
  const int64_t rounds = (tiles(32) + cus - 1) / cus;
  const int64_t stages = wide ? 2 : tiles(64) > cus ? 5 : rounds >= 4 ? 3 : rounds == 3 ? 4 : 16;
  if (vec && M <= kMaxTokens && M >= 128 && (M + 63) / 64 >= stages && tiles(64) >= cus / 2) {
    hipLaunchKernelGGL(hessian_digits_kernel, dim3((unsigned)tiles(64)), dim3(256), 0, (hipStream_t)stream, (const _Float16*)x_fp16,
                       (int)M, (int)K, H);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? QQQ_OK : set_error(QQQ_ERR_HIP, "hessian launch: %s", hipGetErrorString(e));
  }
  const dim3 grid((unsigned)tiles(wide ? 64 : 32));
#define QQQ_HESSIAN(TE, VEC) \
  hipLaunchKernelGGL((hessian_kernel<TE, VEC>), grid, dim3(256), 0, (hipStream_t)stream, (const _Float16*)x_fp16, M, K, H)
  if (wide) { if (vec) QQQ_HESSIAN(64, true); else QQQ_HESSIAN(64, false); }
  else { if (vec) QQQ_HESSIAN(32, true); else QQQ_HESSIAN(32, false); }
#undef QQQ_HESSIAN
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? QQQ_OK : set_error(QQQ_ERR_HIP, "hessian launch: %s", hipGetErrorString(e));
}

}  // extern "C"
