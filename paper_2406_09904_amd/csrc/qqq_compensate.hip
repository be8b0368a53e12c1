// Hessian-based quantisation compensation (Sec. 3.2, Eq. 3-4) on one layer: entry points
// qqq_gptq_quantize_w4_perchannel / _pergroup of include/qqq_calib.h.
//
// Eq. 4 needs, for each channel i, row i of the inverse Hessian of the channels not yet quantised.  Those
// rows never have to be formed.  With H = R D R^T, R unit upper triangular and D diagonal (the Cholesky
// factorisation taken from the last channel to the first), row i of [H_F^-1] over its diagonal entry
// is row i of R^-1, so the running weight of channel j obeys
//     w_j = W_j + sum_{i < j} (W_i - Q_i) R[i,j]
// when its turn comes, W the original weights and Q the dequantised codes: the moves of Eq. 4, summed.  One factorisation of
// K^3/6 multiply-adds and a triangular product of N K^2 / 2 replace an explicit inverse and a rank-1
// update of both matrices per channel, and W_i - Q_i is exact in fp64 (fp16 minus int4 x fp16).
//
// Both parts are blocked so that almost all of their arithmetic is fp64 MFMA (f64_update_kernel, factor_update):
//   factorisation  factor_kernel: 64 channels at a time, from the last
//   sweep          per 512 channels, from the first: sweep_kernel, then the update of the channels after
// What is left serial is one dependent step per channel, in registers.
// Bound, without the Hessian: K = N = 4096 holds 2.3e10 + 6.9e10 fp64 operations, 1.2 ms at the nominal 78.6 TFLOP/s of the
// fp64 matrix cores (1.7 ms at the 54 that f64_update_kernel reaches).  Measured, K = N = 4096: 2.9 ms, and 3.2 ms with the
// Hessian of 2048 tokens (an inverse by K rank-1 sweeps and a rank-1 update of both matrices per channel: 360 ms); K = 2048,
// N = 5632 with group scales: 1.4 ms, 1.47 ms with the Hessian of 1111 tokens (81 ms).
#include "qqq_calib.h"
#include "qqq_factor_schedule.h"
#include "qqq_internal.h"
#include "qqq_tuning.h"

#include <type_traits>

namespace qqq {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kFB = 64;    // channels per factorisation block
constexpr int kSB = 128;   // channels per sweep block (= a group of the per-group quantiser)
constexpr int kCarried = 4;  // update tiles that go with a sweep, for each workgroup that fits beside it
constexpr int kSO = 512;  // channels after which the rest of the weights is updated
static_assert(kSB == QQQ_GROUP && kSB == 128, "a sweep block is one group");

template <int V>
using Width = std::integral_constant<int, V>;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int check_launch(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(QQQ_ERR_HIP, "%s launch: %s", what, hipGetErrorString(e));
  return QQQ_OK;
}

// One 64-bit value of lane SRC of every sixteen lanes, in all sixteen.
template <int SRC>
__device__ __forceinline__ double row_broadcast(double x) {
  const long u = __builtin_bit_cast(long, x);
  const long v = __builtin_amdgcn_update_dpp(0L, u, 0x150 + SRC, 0xF, 0xF, true);  // row_newbcast
  return __builtin_bit_cast(double, v);
}
// Multiply-adds whose first factor is such a broadcast, x of lane L of every sixteen lanes: the data-parallel move is part of
// v_fmac_f64, which costs what a multiply-add costs (5 clocks); a move of its own takes 6 and 8 of latency, two 32-bit
// ones 12.  The compiler does not form it.  It has to stand two instructions behind the one that wrote x, which the compiler
// does not see to inside an asm statement: the s_nop does, once for up to eight of them.
#define QQQ_FMAC_DPP(ACC, X, M, L) "v_fmac_f64_dpp %" #ACC ", " X ", %" #M " row_newbcast:%" #L " row_mask:0xf bank_mask:0xf\n\t"
// acc[k] += x * m[k]  (SUB: -=, acc[0] last, so that x may be acc[0] itself, in the same registers), k < N
template <int L, bool SUB, int N, int A, int B>
__device__ __forceinline__ void fmac_row(double (&acc)[A], double x, const double (&m)[B]) {
  static_assert(N == 4 || N == 8, "");
  if constexpr (N == 4) {
    if constexpr (SUB)
      asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(1, "-%4", 6, 9) QQQ_FMAC_DPP(2, "-%4", 7, 9) QQQ_FMAC_DPP(3, "-%4", 8, 9) QQQ_FMAC_DPP(0, "-%4", 5, 9)
                   : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]) : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "n"(L));
    else
      asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(0, "%4", 5, 9) QQQ_FMAC_DPP(1, "%4", 6, 9) QQQ_FMAC_DPP(2, "%4", 7, 9) QQQ_FMAC_DPP(3, "%4", 8, 9)
                   : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]) : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "n"(L));
  } else {
    if constexpr (SUB)
      asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(1, "-%8", 10, 17) QQQ_FMAC_DPP(2, "-%8", 11, 17) QQQ_FMAC_DPP(3, "-%8", 12, 17) QQQ_FMAC_DPP(4, "-%8", 13, 17)
                   QQQ_FMAC_DPP(5, "-%8", 14, 17) QQQ_FMAC_DPP(6, "-%8", 15, 17) QQQ_FMAC_DPP(7, "-%8", 16, 17) QQQ_FMAC_DPP(0, "-%8", 9, 17)
                   : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7])
                   : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]), "v"(m[6]), "v"(m[7]), "n"(L));
    else
      asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(0, "%8", 9, 17) QQQ_FMAC_DPP(1, "%8", 10, 17) QQQ_FMAC_DPP(2, "%8", 11, 17) QQQ_FMAC_DPP(3, "%8", 12, 17)
                   QQQ_FMAC_DPP(4, "%8", 13, 17) QQQ_FMAC_DPP(5, "%8", 14, 17) QQQ_FMAC_DPP(6, "%8", 15, 17) QQQ_FMAC_DPP(7, "%8", 16, 17)
                   : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7])
                   : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]), "v"(m[6]), "v"(m[7]), "n"(L));
  }
}
// acc[k] -= (x of lane k) * m, k = FROM down to FROM - N + 1
template <int FROM, int N, int A>
__device__ __forceinline__ void fmac_lanes(double (&acc)[A], double x, double m) {
  static_assert(N >= 0 && N <= 4 && FROM - N + 1 >= 0, "");
  if constexpr (N == 1)
    asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(0, "-%1", 2, 3) : "+v"(acc[FROM]) : "v"(x), "v"(m), "n"(FROM));
  if constexpr (N == 2)
    asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(0, "-%2", 3, 4) QQQ_FMAC_DPP(1, "-%2", 3, 5)
                 : "+v"(acc[FROM]), "+v"(acc[FROM - 1]) : "v"(x), "v"(m), "n"(FROM), "n"(FROM - 1));
  if constexpr (N == 3)
    asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(0, "-%3", 4, 5) QQQ_FMAC_DPP(1, "-%3", 4, 6) QQQ_FMAC_DPP(2, "-%3", 4, 7)
                 : "+v"(acc[FROM]), "+v"(acc[FROM - 1]), "+v"(acc[FROM - 2]) : "v"(x), "v"(m), "n"(FROM), "n"(FROM - 1), "n"(FROM - 2));
  if constexpr (N == 4)
    asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(0, "-%4", 5, 6) QQQ_FMAC_DPP(1, "-%4", 5, 7) QQQ_FMAC_DPP(2, "-%4", 5, 8) QQQ_FMAC_DPP(3, "-%4", 5, 9)
                 : "+v"(acc[FROM]), "+v"(acc[FROM - 1]), "+v"(acc[FROM - 2]), "+v"(acc[FROM - 3])
                 : "v"(x), "v"(m), "n"(FROM), "n"(FROM - 1), "n"(FROM - 2), "n"(FROM - 3));
}
// acc[k] -= (its own lane L) * m, k < 4
template <int L>
__device__ __forceinline__ void fmac_own(double (&acc)[4], double m) {
  asm volatile("s_nop 1\n\t" QQQ_FMAC_DPP(0, "-%0", 4, 5) QQQ_FMAC_DPP(1, "-%1", 4, 5) QQQ_FMAC_DPP(2, "-%2", 4, 5) QQQ_FMAC_DPP(3, "-%3", 4, 5)
               : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]) : "v"(m), "n"(L));
}
#undef QQQ_FMAC_DPP
// what an asm statement above has written, fit for the compiler's own data-parallel moves (which would not wait for it)
__device__ __forceinline__ double fmac_settled(double x) {
  asm volatile("s_nop 1" : "+v"(x));
  return x;
}
template <int XOR>  // value of lane ^ XOR within four lanes
__device__ __forceinline__ uint32_t quad_swap(uint32_t x) {
  constexpr int sel = XOR == 1 ? 0xB1 : 0x4E;
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, sel, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t half_row_mirror(uint32_t x) {  // value of lane 7 - i of every eight lanes
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true);
}
__device__ __forceinline__ float row_max(float x) {  // largest of every sixteen lanes, in all sixteen
  auto rotated = [&](auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  x = fmaxf(x, rotated(Width<0x128>{}));  // row_ror by 8, 4, 2, 1
  x = fmaxf(x, rotated(Width<0x124>{}));
  x = fmaxf(x, rotated(Width<0x122>{}));
  return fmaxf(x, rotated(Width<0x121>{}));
}

// x clamped to [-limit, limit], a NaN left as it is
__device__ __forceinline__ float keep_nan_clamp(float x, float limit) {
  return __builtin_elementwise_minimum(__builtin_elementwise_maximum(x, -limit), limit);
}

// keep[i] = 0 for a channel that never fired (H_ii == 0: its weight counts as 0), else 1;
// damp[0] = percdamp * mean of the diagonal, a never-firing channel counting 1
__global__ __launch_bounds__(1024) void diagonal_kernel(const double* H, int64_t K, double percdamp, double* keep,
                                                        double* damp) {
  __shared__ double part[1024];
  double sum = 0.0;
  for (int64_t i = threadIdx.x; i < K; i += 1024) {
    const double d = H[i * K + i];
    keep[i] = d == 0.0 ? 0.0 : 1.0;
    sum += d == 0.0 ? 1.0 : d;
  }
  part[threadIdx.x] = sum;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) damp[0] = percdamp * (part[0] / (double)K);
}

// Working copies: the upper triangle of the damped Hessian (the factorisation reads nothing below the
// diagonal) and the running weights in fp64, 0 in the place of an infinity or NaN (the sweep puts those back: here only
// the moves are added up).  K % 8 == 0.  grid.x: rows of H, then rows of W.
__global__ __launch_bounds__(256) void prepare_kernel(const double* H, const _Float16* w, const double* keep,
                                                      const double* damp, int64_t N, int64_t K, double* A, int64_t ld, double* W64,
                                                      uint32_t* flags, int n_flags) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n_flags; i += gridDim.x * 256) flags[i] = 0;
  for (int64_t r = blockIdx.x; r < K + N; r += gridDim.x) {
    if (r < K) {
      for (int64_t j = (r & ~(int64_t)1) + 2 * threadIdx.x; j < K; j += 512) {
        double h0 = H[r * K + j], h1 = H[r * K + j + 1];  // (H is 8-byte aligned)
        if (j == r) h0 = (h0 == 0.0 ? 1.0 : h0) + damp[0];
        if (j + 1 == r) h1 = (h1 == 0.0 ? 1.0 : h1) + damp[0];
        *reinterpret_cast<double2*>(A + r * ld + j) = make_double2(h0, h1);
      }
    } else {
      const int64_t at0 = (r - K) * K;
      for (int64_t k = 2 * threadIdx.x; k < K; k += 512) {
        const uint32_t two = *reinterpret_cast<const uint32_t*>(w + at0 + k);
        const bool in0 = keep[k] != 0.0 && (two & 0x7C00u) != 0x7C00u;
        const bool in1 = keep[k + 1] != 0.0 && (two & 0x7C000000u) != 0x7C000000u;
        const double w0 = in0 ? (double)half_bits_to_float(two & 0xFFFFu) : 0.0;
        const double w1 = in1 ? (double)half_bits_to_float(two >> 16) : 0.0;
        *reinterpret_cast<double2*>(W64 + at0 + k) = make_double2(w0, w1);
      }
    }
  }
}

// C += A B in fp64: C [M,N], A [M,kd], B [kd,N], all row-major and 16-byte aligned, N, kd and the strides even.
// 64 x 64 tile per workgroup, a wave per 32 x 32 quarter, 32 of kd at a time through LDS with the next
// 32 already requested.  v_mfma_f64_16x16x4_f64 (64 clocks): lane l holds row (column) l % 16 and k = l / 16
// of the operands, register v of the result is row 4 v + l / 16, column l % 16.  Row strides of the LDS tiles
// (34 and 80 doubles) put the 32 lanes of half a wave on all 64 banks; each fragment read feeds two MFMAs.  M = 4096,
// N = 3584, kd = 512: 280 us, 54 TFLOP/s (MFMAs alone, operands in registers, reach 70 at the 2.15 GHz they then leave); 128 x 64
// tiles and fragments read four k ahead measured the same.  The second launch bound keeps the accumulators in the vector
// registers: left alone the compiler moves them to the accumulation registers and back every 32 of kd (303 us).
constexpr int kAs = 34, kBs = 80;  // row strides of the LDS tiles: 64 rows of A, 32 of B
__device__ __forceinline__ void update_tile(const double* A, int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc,
                                            int M, int N, int kd, int tm, int tn, double* sa, double* sb) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = tm * 64, n0 = tn * 64;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  const int l16 = lane & 15, q = lane >> 4;

  // Every load is in range and unconditional: rows past M and columns past N repeat the last ones (they only reach results
  // that are not stored), k past kd is replaced by zeros on the way to LDS, a k-step later.  (A conditional load of the
  // struct becomes a choice between its address and one in scratch memory, which makes every load a flat one.)
  const double2* pa[4];
  const double2* pb[4];
  double2 ra[4], rb[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = tid + 256 * j;
    pa[j] = reinterpret_cast<const double2*>(A + (int64_t)min(m0 + (e >> 4), M - 1) * lda);
    pb[j] = reinterpret_cast<const double2*>(B + min(n0 + 2 * (e & 31), N - 2));
  }
  auto fetch = [&](int k0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = tid + 256 * j;
      ra[j] = pa[j][min(k0 + 2 * (e & 15), kd - 2) >> 1];
      rb[j] = pb[j][min(k0 + (e >> 5), kd - 1) * (ldb >> 1)];
    }
  };
  fetch(0);
  v4d acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + wr + 16 * i + 4 * v + q, col = n0 + wc + 16 * j + l16;
        acc[i][j][v] = C[(int64_t)min(row, M - 1) * ldc + min(col, N - 1)];
      }
  for (int k0 = 0; k0 < kd; k0 += 32) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = tid + 256 * j;
      double2 a = ra[j];
      double2 b = rb[j];
      if (k0 + 2 * (e & 15) >= kd) a.x = a.y = 0.0;
      if (k0 + (e >> 5) >= kd) b.x = b.y = 0.0;
      *reinterpret_cast<double2*>(&sa[(e >> 4) * kAs + 2 * (e & 15)]) = a;
      *reinterpret_cast<double2*>(&sb[(e >> 5) * kBs + 2 * (e & 31)]) = b;
    }
    __syncthreads();
    if (k0 + 32 < kd) fetch(k0 + 32);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = sa[(wr + 16 * i + l16) * kAs + 4 * s + q];
        b[i] = sb[(4 * s + q) * kBs + wc + 16 * i + l16];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + wr + 16 * i + 4 * v + q, col = n0 + wc + 16 * j + l16;
        if (row < M && col < N) C[(int64_t)row * ldc + col] = acc[i][j][v];
      }
}

__global__ __launch_bounds__(256, 3) void f64_update_kernel(const double* A, int64_t lda, const double* B, int64_t ldb,
                                                         double* C, int64_t ldc, int M, int N, int kd) {
  __shared__ __attribute__((aligned(16))) double sa[64 * kAs];
  __shared__ __attribute__((aligned(16))) double sb[32 * kBs];
  update_tile(A, lda, B, ldb, C, ldc, M, N, kd, blockIdx.y, blockIdx.x, sa, sb);
}

// ---- H = R D R^T, all of it in one launch.
// Blocks of 64 channels from the last: block k's diagonal tile is factored (64 dependent pivots), the row tiles i < k above it are solved
// (y_j = a_j - sum_{k' > j} y_k' R[j,k'], x_j = y_j / d_j: R = x and R D = y there), and every tile (i, j), i <= j < k, gets A -= R[i,k] (R D)[j,k]^T.
// What bounds it is the chain of all pivots, so one workgroup does nothing else: block after block it factors the tile, solves the row tile
// next to it and takes that off the next tile, without leaving its CU.  All other workgroups draw tickets for the rest (qqq_factor_schedule.h), in a fixed order in
// which a task needs only earlier ones and the chain's earlier blocks.  There are two queues, a workgroup in three on the one that the chain waits for (solves,
// updates by one panel), the others on the updates by four panels at once, whose tasks are long.  Three resident workgroups keep chain and queues going.  Where
// fewer have come (a launch beside others on streams that share a few CUs, a small partition of the chip) the chain does tasks itself when it would
// wait, in the same order: so the waits end however few workgroups run, one included, and the results have the same bits.  (A launch that has its
// CUs pays nothing: K = N = 4096 3209 us a call with a chain that only waits, 3198 so; K = 2048, N = 5632 with group scales 1479 and 1474; with the
// chain's first block always in the body that looks for tasks 3204 and 1478, K = 1024 .. 3072 0.4 to 0.8 % slower than one that only waits.)  What a task needs is told by flags: a block
// factored, a tile solved, the number of panels that a tile has received.
// Tiles receive the panels of their own four blocks (kOuter) one by one, those of the next four two at a time, and those of later blocks four at a time, during the
// steps of the four blocks after them; the columns whose turn to factor comes next first, in 64 x 64 tiles, the others in 128 x 128.
// Between XCDs caches are coherent at kernel boundaries only, so what one workgroup writes for another goes through to memory (agent-scope
// stores, a wait, then the flag).  R D is kept transposed below the diagonal, each line written once and read only after its flag, so updates read it
// with plain loads, and take R from it too (x = y / d, the same bits); tiles that change are read at agent scope.
// One workgroup a CU: with two, solves and updates on a CU held each other up and the chain with them (K = 4096, 64 x 64 tiles only: 2530 us, 1660 with one).
// K = 2048 / 4096: 536 / 1220 us (a launch per block, its workgroups all factoring the tile again, with the updates carried in or between: 800 / 1960).
// A block of the chain takes 16.5 us of waiting for nobody: the tile 7.7, the row tile 3.6, off the next tile 2.1, flags and loads 3.
// At K = 4096 the first half of the blocks waits for updates: a 64 x 64 tile takes 5 us for one panel, 7 for two, 15 for four, a 128 x 128 tile 44 for four.
// A thread's number, new to the compiler: what follows from it is computed where it is used.  (Where the chain does tasks, the compiler would otherwise
// keep the addresses of all their parts in registers while it factors, 47 to 80 more than there are.)
__device__ __forceinline__ int thread_id() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
constexpr int kS = 66;  // row stride of a 64 x 64 block in LDS

struct Factor {
  double* A;        // [K][ld], ld a multiple of 16: a tile's rows are whole cache lines
  double* rcp;      // [K] 1 / d_j
  uint32_t* ticket;  // [0]: workgroups that have come; [1], [2]: tasks drawn from the queues
  uint32_t* flags;   // see Flags
  int K, ld, nb;
};

template <typename T>
__device__ __forceinline__ T agent_load(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ void agent_store(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Until flag[l] >= least[l] for every lane l of wave 0 that asks; all threads wait.
__device__ __forceinline__ void await(const uint32_t* flag, uint32_t least, bool asks) {
  if (threadIdx.x < 64)
    while (!__all(!asks || agent_load(flag) >= least)) __builtin_amdgcn_s_sleep(1);
  lds_barrier();
}
// What this workgroup has written stands in memory: then the flag.
__device__ __forceinline__ void publish(uint32_t* flag, uint32_t v) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier();
  if (threadIdx.x == 0) agent_store(flag, v);
}

// What a tile of EDGE x EDGE at rows 64 i, columns 64 j receives from panels [p0, p0 + np): -= R[rows, panels] (R D)[columns, panels]^T, a wave per
// quarter of it, 32 channels at a time through two LDS stages: the next one is placed, and the one after it requested, behind half of a
// stage's products.  Both operands are k-major, R = R D / d is formed on the way.  MFMA layout and row strides as in update_tile.  `mine`: this wave's
// quarter is wanted (of a 128 x 128 tile on the diagonal three are).
template <int EDGE>
__device__ __forceinline__ void factor_update(const Factor& f, int tid, int i, int j, int p0, int np, bool mine, double* stages) {
  constexpr int kStride = EDGE + 16, kQ = EDGE / 32, kRows = 512 / EDGE, kLoads = 32 / kRows;  // 16 x 16 tiles a side of a quarter; rows of a load
  const int lane = tid & 63, wave = tid >> 6, l16 = lane & 15, q = lane >> 4;
  const int wr = (wave >> 1) * (EDGE / 2), wc = (wave & 1) * (EDGE / 2);
  const int k1 = min((p0 + np) * 64, f.K), row0 = tid / (EDGE / 2), col0 = 2 * (tid % (EDGE / 2));
  const double* pa = f.A + 64 * i + col0;
  const double* pb = f.A + 64 * j + col0;
  double2 ra[kLoads], rb[kLoads];
  double rk[kLoads];
  auto fetch = [&](int k0) {  // (past the end: the last row again)
#pragma unroll
    for (int x = 0; x < kLoads; ++x) {
      const int k = min(k0 + row0 + kRows * x, k1 - 1);
      ra[x] = *reinterpret_cast<const double2*>(pa + (int64_t)k * f.ld);
      rb[x] = *reinterpret_cast<const double2*>(pb + (int64_t)k * f.ld);
      rk[x] = f.rcp[k];
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto place = [&](int h, int k0) {
    double* const sa = stages + h * 2 * 32 * kStride;
    double* const sb = sa + 32 * kStride;
#pragma unroll
    for (int x = 0; x < kLoads; ++x) {
      const int row = row0 + kRows * x;
      const bool in = k0 + row < k1;
      const double2 a = in ? make_double2(-(ra[x].x * rk[x]), -(ra[x].y * rk[x])) : make_double2(0.0, 0.0);
      const double2 b = in ? rb[x] : make_double2(0.0, 0.0);
      *reinterpret_cast<double2*>(&sa[row * kStride + col0]) = a;
      *reinterpret_cast<double2*>(&sb[row * kStride + col0]) = b;
    }
  };
  fetch(64 * p0);
  double* const c = f.A + (int64_t)(64 * i + wr + q) * f.ld + 64 * j + wc + l16;
  v4d acc[kQ][kQ];
#pragma unroll
  for (int x = 0; x < kQ; ++x)
#pragma unroll
    for (int y = 0; y < kQ; ++y) acc[x][y] = (v4d){0.0, 0.0, 0.0, 0.0};
  if (mine)
#pragma unroll
    for (int x = 0; x < kQ; ++x)
#pragma unroll
      for (int y = 0; y < kQ; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[x][y][v] = agent_load(c + (int64_t)(16 * x + 4 * v) * f.ld + 16 * y);
  place(0, 64 * p0);
  fetch(64 * p0 + 32);
  lds_barrier();
  int h = 0;
#pragma nounroll
  for (int k0 = 64 * p0; k0 < k1; k0 += 32) {
    const double* const sa = stages + h * 2 * 32 * kStride;
    const double* const sb = sa + 32 * kStride;
    double a[2][kQ], b[2][kQ];
    auto read = [&](int s) {
#pragma unroll
      for (int x = 0; x < kQ; ++x) {
        a[s & 1][x] = sa[(4 * s + q) * kStride + wr + 16 * x + l16];
        b[s & 1][x] = sb[(4 * s + q) * kStride + wc + 16 * x + l16];
      }
    };
    read(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (s < 7) read(s + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 0; x < kQ; ++x)
#pragma unroll
        for (int y = 0; y < kQ; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s & 1][x], b[s & 1][y], acc[x][y], 0, 0, 0);
      if (s == 3) {
        place(h ^ 1, k0 + 32);
        fetch(k0 + 64);
      }
    }
    h ^= 1;
    lds_barrier();
  }
  if (mine)
#pragma unroll
    for (int x = 0; x < kQ; ++x)
#pragma unroll
      for (int y = 0; y < kQ; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v) agent_store(c + (int64_t)(16 * x + 4 * v) * f.ld + 16 * y, (double)acc[x][y][v]);
}

// The diagonal block in ys, 16 columns at a time from the last: they receive what the columns after them owe (fp64 MFMA, a wave per 16 rows);
// one wave takes the 16 steps of the 16 x 16 tile on the diagonal, a lane a row, with what is broadcast as part of the
// multiply-adds and the next pivot's reciprocal between them; the waves of the rows above solve theirs by it, 16 lanes per row.
// [i][j], in 16 x 16 tiles.  ys: the block's upper triangle; tiles above the diagonal become R D when their columns' turn comes, those on it
// keep the block as the columns after left it.  xs: R in the tiles above the diagonal and on it, there 0 from the diagonal on,
// each from its columns' turn on; the tiles below are never written, nor read.
// Both halves walk 16 columns at a time in a loop, so that one body of a few KiB serves the whole block (written out straight, 42 KiB of
// instructions took 44.7 us a block whatever the row count).  In clocks: 16 columns 4600 (a pivot 150, the rest the products, the rows above, barriers).
__device__ __forceinline__ void factor_diagonal(double* ys, double* xs, double* rcp) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, q = lane >> 4;
#pragma nounroll
  for (int p = 3; p >= 0; --p) {
    // a wave's 16 rows of these columns less what the columns after owe them: register v is row 16 wave + 4 v + q, column 16 p + l16
    double u[4];
    if (wave <= p) {
      v4d acc;
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = ys[(16 * wave + 4 * v + q) * kS + 16 * p + l16];
      for (int k = 16 * (p + 1); k < 64; k += 16) {
        double x[4], yk[4];  // (all requested before the first is multiplied)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          x[w] = -xs[(16 * wave + l16) * kS + k + 4 * w + q];
          yk[w] = ys[(16 * p + l16) * kS + k + 4 * w + q];
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[w], yk[w], acc, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        u[v] = acc[v];
        if (wave == p) ys[(16 * wave + 4 * v + q) * kS + 16 * p + l16] = acc[v];
      }
    }
    __syncthreads();
    if (wave == 0) {
      // t[k]: element (16 p + l16, 16 p + k) of the diagonal tile, once in every sixteen lanes.  Below the diagonal whatever the
      // steps leave, never used
      double t[16], own_rd = 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) t[k] = ys[(16 * p + l16) * kS + 16 * p + k];
      double rd;  // 1 / d within an ulp or so: two Newton steps
      {
        const double d = row_broadcast<15>(t[15]);
        rd = __builtin_amdgcn_rcp(d);
        rd = __builtin_fma(__builtin_fma(-d, rd, 1.0), rd, rd);
        rd = __builtin_fma(__builtin_fma(-d, rd, 1.0), rd, rd);
      }
      // The next pivot first, and the steps of its reciprocal between the other multiply-adds (each is pinned to its place:
      // left to the compiler they stand in a row, waiting for one another)
      auto step = [&](auto at) {
        constexpr int j = decltype(at)::value;
        const double x = t[j] * rd;
        own_rd = l16 == j ? rd : own_rd;
        if constexpr (j > 0) {
          constexpr int n = j - 1;  // columns left after the next pivot's
          fmac_lanes<j - 1, 1>(t, t[j], x);
          const double d = row_broadcast<j - 1>(fmac_settled(t[j - 1]));
          double r = __builtin_amdgcn_rcp(d);
          asm volatile("" : "+v"(r));
          if constexpr (n > 0) fmac_lanes<n - 1, (n < 4 ? n : 4)>(t, t[j], x);
          double e = __builtin_fma(-d, r, 1.0);
          asm volatile("" : "+v"(e));
          if constexpr (n > 4) fmac_lanes<n - 5, (n < 8 ? n - 4 : 4)>(t, t[j], x);
          r = __builtin_fma(e, r, r);
          asm volatile("" : "+v"(r));
          if constexpr (n > 8) fmac_lanes<n - 9, (n < 12 ? n - 8 : 4)>(t, t[j], x);
          e = __builtin_fma(-d, r, 1.0);
          asm volatile("" : "+v"(e));
          if constexpr (n > 12) fmac_lanes<n - 13, n - 12>(t, t[j], x);
          rd = __builtin_fma(e, r, r);
        }
        xs[(16 * p + l16) * kS + 16 * p + j] = l16 < j ? x : 0.0;  // (nothing reads R D in a diagonal tile)
      };
      step(Width<15>{}); step(Width<14>{}); step(Width<13>{}); step(Width<12>{}); step(Width<11>{}); step(Width<10>{});
      step(Width<9>{}); step(Width<8>{}); step(Width<7>{}); step(Width<6>{}); step(Width<5>{}); step(Width<4>{});
      step(Width<3>{}); step(Width<2>{}); step(Width<1>{}); step(Width<0>{});
      if (lane < 16) rcp[16 * p + lane] = own_rd;
    }
    __syncthreads();
    if (wave < p) {  // the rows above, column by column from the last
      const double* rr = xs + (16 * p + l16) * kS + 16 * p;
      double m[16];
#pragma unroll
      for (int j = 15; j > 0; --j) m[j] = rr[j];
      fmac_own<15>(u, m[15]); fmac_own<14>(u, m[14]); fmac_own<13>(u, m[13]); fmac_own<12>(u, m[12]); fmac_own<11>(u, m[11]);
      fmac_own<10>(u, m[10]); fmac_own<9>(u, m[9]); fmac_own<8>(u, m[8]); fmac_own<7>(u, m[7]); fmac_own<6>(u, m[6]);
      fmac_own<5>(u, m[5]); fmac_own<4>(u, m[4]); fmac_own<3>(u, m[3]); fmac_own<2>(u, m[2]); fmac_own<1>(u, m[1]);
      const double rd = rcp[16 * p + l16];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        ys[(16 * wave + 4 * v + q) * kS + 16 * p + l16] = u[v];
        xs[(16 * wave + 4 * v + q) * kS + 16 * p + l16] = u[v] * rd;
      }
    }
    __syncthreads();
  }
}

// Tile i of panel k (block at c0 = 64 k, its R in xs and rcp), a wave per 16 rows: 16 columns at a time from the last receive what the columns
// after them owe (fp64 MFMA), then the 16 one after the other, 16 lanes a row.  u[p][v]: row 16 wave + 4 v + q, column 16 p + l16.  R goes to
// its place, R D to ys, [column][row].  (All columns after each column in vector multiply-adds: 4.8 us,
// 2.7 so.)
__device__ __forceinline__ void load_rows(const Factor& f, int tid, int i, int c0, double (&u)[4][4]) {
  const int lane = tid & 63, wave = tid >> 6, l16 = lane & 15, q = lane >> 4, nb = min(64, f.K - c0);
#pragma unroll
  for (int p = 3; p >= 0; --p)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      u[p][v] = agent_load(f.A + (int64_t)(64 * i + 16 * wave + 4 * v + q) * f.ld + c0 + min(16 * p + l16, nb - 1));
}
__device__ __forceinline__ void solve_rows(const Factor& f, int tid, int i, int c0, double (&u)[4][4], double* ys, const double* xs, const double* rcp) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, q = lane >> 4, nb = min(64, f.K - c0);
#pragma unroll
  for (int p = 3; p >= 0; --p) {
    v4d acc = {u[p][0], u[p][1], u[p][2], u[p][3]};
#pragma unroll
    for (int k = 16 * (p + 1); k < 64; k += 4)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-ys[(k + q) * kS + 16 * wave + l16], xs[(16 * p + l16) * kS + k + q], acc, 0, 0, 0);
    const double* rr = xs + (16 * p + l16) * kS + 16 * p;
    double m[16];
#pragma unroll
    for (int j = 15; j > 0; --j) m[j] = rr[j];
    double y[4] = {acc[0], acc[1], acc[2], acc[3]};
    fmac_own<15>(y, m[15]); fmac_own<14>(y, m[14]); fmac_own<13>(y, m[13]); fmac_own<12>(y, m[12]); fmac_own<11>(y, m[11]);
    fmac_own<10>(y, m[10]); fmac_own<9>(y, m[9]); fmac_own<8>(y, m[8]); fmac_own<7>(y, m[7]); fmac_own<6>(y, m[6]);
    fmac_own<5>(y, m[5]); fmac_own<4>(y, m[4]); fmac_own<3>(y, m[3]); fmac_own<2>(y, m[2]); fmac_own<1>(y, m[1]);
    const int col = 16 * p + l16;
    const double rd = rcp[col];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 16 * wave + 4 * v + q;
      ys[col * kS + row] = col < nb ? y[v] : 0.0;
      if (col < nb) f.A[(int64_t)(64 * i + row) * f.ld + c0 + col] = y[v] * rd;
    }
  }
  lds_barrier();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int j = 4 * e + wave;
    if (j < nb) agent_store(f.A + (int64_t)(c0 + j) * f.ld + 64 * i + lane, ys[j * kS + lane]);
  }
}

// Two blocks of 64 x 64, or two stages of an update of 128 x 128: each workgroup, the chain above all, has its CU to itself
struct FactorLds {
  __attribute__((aligned(16))) double ys[4 * 32 * 144];
  double rcp[64];
  int ticket, queue;
};
static_assert(2 * 64 * kS <= 4 * 32 * 144, "the blocks fit");
typedef __attribute__((address_space(3))) FactorLds* FactorLdsPtr;

// R of the block at c0 and its 1 / d, as factor_diagonal left them; channels past K are identity.  load() places what the constructor requests
struct BlockOfR {
  double r[16], rd;
  int tid, cols;
  __device__ __forceinline__ BlockOfR(const Factor& f, int tid_, int c0) : tid(tid_), cols(min(64, f.K - c0)) {
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int e = 0; e < 16; ++e) r[e] = agent_load(f.A + (int64_t)(c0 + min(4 * e + wave, cols - 1)) * f.ld + c0 + lane);
    rd = agent_load(f.rcp + c0 + min(lane, cols - 1));
  }
  __device__ __forceinline__ void place(double* xs, double* rcp) const {
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = 4 * e + wave;
      xs[lane * kS + j] = lane < j && j < cols ? r[e] : 0.0;
    }
    if (tid < 64) rcp[tid] = tid < cols ? rd : 1.0;
    lds_barrier();
  }
};

// WIDE: a tile of 128 x 128 as one, else as its four of 64 x 64 (the same bits, half the registers)
template <bool WIDE>
__device__ __forceinline__ void do_task(const Factor& f, int tid, const Task& t, double* ys, double* rcp) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Flags told = {f.nb};
  const Need need = need_of(told, t, lane);
  await(f.flags + need.flag, (uint32_t)need.least, need.asks);
  if (t.kind == kSolve) {
    double rows[4][4];
    load_rows(f, tid, t.i, 64 * t.j, rows);
    const BlockOfR block(f, tid, 64 * t.j);
    block.place(ys + 64 * kS, rcp);
    solve_rows(f, tid, t.i, 64 * t.j, rows, ys, ys + 64 * kS, rcp);
  } else if (t.kind == kUpdate64) {
    factor_update<64>(f, tid, t.i, t.j, t.p0, t.np, true, ys);
  } else if constexpr (!WIDE) {
#pragma nounroll
    for (int x = 0; x < 4; ++x)
      if (t.i + x / 2 <= t.j + x % 2) factor_update<64>(f, tid, t.i + x / 2, t.j + x % 2, t.p0, t.np, true, ys);
  } else {
    factor_update<128>(f, tid, t.i, t.j, t.p0, t.np, t.i + (wave >> 1) <= t.j + (wave & 1), ys);
  }
  const Done done = done_of(told, t, lane);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier();
  if (wave == 0 && done.tells) agent_store(f.flags + done.flag, (uint32_t)done.value);
}

// Where the chain would wait (block k, its tile factored or not yet) and no crew has been seen: 0 if the wait is over, 2 if there is a crew by now; 1 after
// a task done or looked for, to be asked again.  `away`: its blocks are not in LDS any more.  A task that it does not find is in the hands of a workgroup
// whose own waits end (see queue_for_chain).
__device__ __forceinline__ int instead_of_waiting(const Factor& f, FactorLds& lds, int k, bool factored, bool& away) {
  const int id = thread_id(), nb = f.nb;
  const Flags told = {nb};
  const Need need = need_of_chain(told, k, factored);
  if (id == 0) lds.ticket = agent_load(f.ticket) >= (uint32_t)kFactorCrew ? 2 : agent_load(f.flags + need.flag) < (uint32_t)need.least;
  __syncthreads();
  const int found = __builtin_amdgcn_readfirstlane(lds.ticket);
  __syncthreads();
  if (found != 1) return found;
  if (!away) publish(f.flags + (factored ? told.factored(k) : told.solved(k + 1, k)), 1u);  // (what it owes the others)
  away = true;
  if (id == 0) {
    Queue head(1, nb);
    const uint32_t drawn1 = agent_load(f.ticket + 1), drawn2 = agent_load(f.ticket + 2);
    const int queue = queue_for_chain(nb, k, (int)drawn1, (int)drawn2, &head);
    uint32_t drawn = queue == 2 ? drawn2 : drawn1;
    const bool mine = queue != 0 && __hip_atomic_compare_exchange_strong(f.ticket + queue, &drawn, drawn + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                         __HIP_MEMORY_SCOPE_AGENT);
    lds.ticket = mine ? (int)drawn : -1;
    lds.queue = queue;
  }
  __syncthreads();
  const int ticket = __builtin_amdgcn_readfirstlane(lds.ticket);
  Queue from(__builtin_amdgcn_readfirstlane(lds.queue), nb);
  __syncthreads();
  if (ticket < 0) return 1;
  from.reach(ticket);
  const Task t = task_of(from.step, from.queue, ticket - from.base);
  if (t.kind != kNothing) do_task<false>(f, id, t, lds.ys, lds.rcp);
  return 1;
}

// The chain from block k on.  FEW: until a crew has been seen; returns the block to go on with, or -1 after the last.  (Two bodies: the one that nearly
// all blocks go through waits, and holds no registers for tasks: K = 1024 .. 4096 1 to 2 % slower with one.)
template <bool FEW>
__device__ __forceinline__ int chain(const Factor& f, FactorLds& lds, int k) {
  double* const ys = lds.ys;
  double* const xs = ys + 64 * kS;
  double* const rcp = lds.rcp;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, q = lane >> 4, nb = f.nb;
  const Flags told = {nb};
  bool few = FEW, away = false;
  int found = 1;
  for (;; --k) {
    const int c0 = 64 * k, cols = min(64, f.K - c0);
    if constexpr (FEW) {
      if (!few) return k;
      while ((found = instead_of_waiting(f, lds, k, false, away)) == 1) {}
      few = found != 2;
    }
    await(f.flags + told.applied(k, k), (uint32_t)need_of_chain(told, k, false).least, lane == 0);
    if constexpr (FEW) {
      if (away) {  // R D of the row tile that was solved last, and 1 / d of its block
        const int before = min(64, f.K - c0 - 64);
        for (int j = wave; j < 64; j += 4) ys[j * kS + lane] = j < before ? agent_load(f.A + (int64_t)(c0 + 64 + j) * f.ld + c0 + lane) : 0.0;
        if (tid < 64) rcp[tid] = tid < before ? agent_load(f.rcp + c0 + 64 + tid) : 1.0;
        lds_barrier();
      }
      away = false;
    }
    // the block's upper triangle, a wave's 16 x 16 tiles u = wave, wave + 4, wave + 8 of ten; channels past K are identity
    v4d acc[3];
    int tr[3], tc[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      const int u = min(wave + 4 * x, 9);
      tc[x] = u >= 6 ? 3 : u >= 3 ? 2 : u >= 1 ? 1 : 0;
      tr[x] = u - tc[x] * (tc[x] + 1) / 2;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        acc[x][v] = agent_load(f.A + (int64_t)(c0 + min(16 * tr[x] + 4 * v + q, cols - 1)) * f.ld + c0 + min(16 * tc[x] + l16, cols - 1));
    }
    if (k + 1 < nb) {
      publish(f.flags + told.solved(k + 1, k), 1u);  // (the row tile that the last round solved: its stores went out before these loads)
      double a[2][3], b[2][3];
      auto read = [&](int s) {
        const double rd = -rcp[4 * s + q];
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          b[s & 1][x] = ys[(4 * s + q) * kS + 16 * tc[x] + l16];
          a[s & 1][x] = ys[(4 * s + q) * kS + 16 * tr[x] + l16] * rd;
        }
      };
      read(0);
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        if (s < 15) read(s + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < 3; ++x) acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s & 1][x], b[s & 1][x], acc[x], 0, 0, 0);
      }
      lds_barrier();
    }
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 16 * tr[x] + 4 * v + q, j = 16 * tc[x] + l16;
        if (wave + 4 * x < 10) ys[i * kS + j] = i <= j && j < cols ? (double)acc[x][v] : i == j ? 1.0 : 0.0;
      }
    lds_barrier();
    factor_diagonal(ys, xs, rcp);
    // R transposed below the diagonal
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = 4 * e + wave;
      if (lane < j && j < cols) agent_store(f.A + (int64_t)(c0 + j) * f.ld + c0 + lane, xs[lane * kS + j]);
    }
    if (tid < cols) agent_store(f.rcp + c0 + tid, rcp[tid]);
    if (k == 0) return -1;
    if constexpr (FEW) {
      while (few && (found = instead_of_waiting(f, lds, k, true, away)) == 1) {}
      few = found != 2;
    }
    await(f.flags + told.applied(k - 1, k), (uint32_t)need_of_chain(told, k, true).least, lane == 0);
    if constexpr (FEW) {
      if (away) {
        const BlockOfR block(f, tid, c0);
        block.place(xs, rcp);
      }
      away = false;
    }
    double rows[4][4];
    load_rows(f, tid, k - 1, c0, rows);
    publish(f.flags + told.factored(k), 1u);
    solve_rows(f, tid, k - 1, c0, rows, ys, xs, rcp);
  }
}

__global__ __launch_bounds__(256, 1) void factor_kernel(const Factor f) {
  __shared__ FactorLds lds;
  double* const ys = lds.ys;
  double* const rcp = lds.rcp;
  const int tid = threadIdx.x, nb = f.nb;
  auto draw = [&](int queue) {
    if (tid == 0) lds.ticket = (int)__hip_atomic_fetch_add(f.ticket + queue, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(lds.ticket);
    __syncthreads();
    return t;
  };
  const int number = draw(0);
  if (number == 0) {
    __builtin_amdgcn_s_setprio(3);
    // Two blocks have no waits in them.  Otherwise a launch that has its CUs has a crew in a microsecond: worth a few looks, since a block in the body that does
    // tasks costs that body's instructions from memory, then the other's (5 to 7 us).
    if (tid == 0) {
      uint32_t come = kFactorCrew;
      if (nb > 2)
        for (int i = 0; i < 8 && (come = agent_load(f.ticket)) < (uint32_t)kFactorCrew; ++i) __builtin_amdgcn_s_sleep(1);
      lds.ticket = come >= (uint32_t)kFactorCrew;
    }
    __syncthreads();
    const bool crew = __builtin_amdgcn_readfirstlane(lds.ticket) != 0;
    __syncthreads();
    const int k = crew ? nb - 1 : chain<true>(f, lds, nb - 1);
    if (k >= 0) chain<false>(f, lds, k);
    return;
  }

  // ---- everything else
  Queue from(number % 3 == 1 ? 1 : 2, nb);
  for (;;) {
    const int ticket = draw(from.queue);
    if (!from.reach(ticket)) {
      if (from.queue == 1) return;
      from = Queue(1, nb);
      continue;
    }
    const Task t = task_of(from.step, from.queue, ticket - from.base);
    if (t.kind != kNothing) do_task<true>(f, tid, t, ys, rcp);
  }
}

// the u-th 16 x 16 tile (rows 16 r, columns 16 t >= 16 r) of a sweep block's R, u < 36
struct Tile { int r, t; bool transposed; };
__device__ __forceinline__ Tile upper_tile(int u) {
  int r = 0;
#pragma unroll
  for (int x = 1; x < 8; ++x) r += u >= 8 * x - x * (x - 1) / 2;
  const int t = u - (8 * r - r * (r - 1) / 2) + r;
  return {r, t, (16 * r) / kFB == (16 * t) / kFB};
}

// Channels [o0, o1) of every output channel, one after the other: code of the running weight, then the
// move of the later channels,
//   q = clamp(rne(fp32(w / s)), -7, 7), s == 0 gives 0;  w_j += (W_i - q s) R[i,j] for j > i.
// An output channel never needs another one, so a workgroup takes 16 of them through all these channels, 128 at a time:
// what the 128 owe to those before (from o0 on) as one fp64 MFMA product, then the chain.  Bound by that chain of
// dependent fp64 operations (about 12 a channel): sixteen lanes per output channel, lane's channels 16 r + (lane % 16) in
// registers, so that 4096 output channels put a wave on every SIMD; a step is the quotient, its rounding and one
// multiply-add per 16 later channels, the broadcast of W_i - q s inside the sixteen lanes being part of it.
// The steps are a loop over 16 channels whose registers move down one place each time: one body for 128 channels
// (written out straight, 40 to 73 KiB of instructions, each fetched for one use, took 65 to 81 us per 128 channels and the
// separate products 20 more).  In clocks, 128 channels of 4096 output channels at K = 4096: weights 2500 (8600 as conditional loads),
// product 8500 per 128 channels before, R 5000, chain 19500 (153 a step); 512 channels 78 us.
// R's block sits in LDS as rows of what a step still needs: row i from channel 16 (i / 16) on, zeros up to the diagonal, one
// double apart from a multiple of the banks.
// The quotient: w * (1/s) corrected by its exact remainder, which is the correctly rounded w / s.
// Where that is no number (an infinite or NaN weight or scale, a Hessian that holds one), the code is 0 and what it leaves
// behind is NaN, so that the output channel's later codes and group scales are 0 too: the clamp is the pair of minimum and maximum that
// keep a NaN (v_med3_f32 would make it -7), one instruction more in the chain.
// GROUP: the scale is taken here, s = fp16(fp32(max |w|) / 7) over the block as Eq. 4 leaves its weights when the
// sweep enters it.  What has been added up so far for channel j, P_j = sum over i < c0 of (W_i - Q_i) R[i,j], is
// its move once the block's earlier channels have had theirs; with none of them quantised yet, the move z of
// all channels solves z R = P over the block's triangle (z = P for its first channel).
// W64 is overwritten with W_i - q s, the left operand of the update of the channels after.
// The first `sweepers` workgroups do that; the others, one to a CU beside them, take 64 x 64 tiles of what the 512 channels before these owe to
// columns that neither they nor these touch (Carried): products for matrix cores that the chains leave idle most of the time, though a chain's fp64
// steps wait for them (wave priorities change nothing), so most tiles stay with f64_update_kernel, three workgroups a CU.  us with none / 2 / 4 / 8 for each
// workgroup that fits beside the sweep: K = N = 4096 3327 / 3290 / 3262 / 3299, K = 2048, N = 5632 with group scales 1537 / 1499 / 1473 / 1471 (whole calls).
struct Carried { const double *A, *B; double* C; int N, cols, rows_of_tiles; };  // as f64_update_kernel's operands, kSO deep
template <bool GROUP>
__global__ __launch_bounds__(256, 2) void sweep_kernel(const _Float16* w, const double* A, int ld, const double* keep, int64_t N,
                                                    int64_t K, int o0, int o1, uint16_t* scales, double* W64,
                                                    uint32_t* w_nat, int sweepers, const Carried cr) {
  constexpr int kRows = 16 * (16 * 36 + 8);  // doubles: 16 rows of 129 - 16 r for r = 0 .. 7
  // in the same place before R is: the product's 16 rows of the left operand and of the result
  constexpr int kLs = kSO - kSB + 2, kXs = kSB + 2;
  static_assert(16 * (kLs + kXs) <= kRows, "the product's operand and result fit");
  __shared__ __attribute__((aligned(16))) double rl[kRows + 64];  // (a step reads up to three vectors of 16 past its row)
  if ((int)blockIdx.x >= sweepers) {
    const int u = (int)blockIdx.x - sweepers;
    update_tile(cr.A, K, cr.B, ld, cr.C, K, cr.N, cr.cols, kSO, u % cr.rows_of_tiles, u / cr.rows_of_tiles, rl, rl + 64 * kAs);
    return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, q = lane >> 4;
  const int64_t n0 = (int64_t)blockIdx.x * 16;
  const int64_t row = n0 + 4 * wave + q;
  const int64_t n = row < N ? row : N - 1;  // (rows past N repeat the last one and store nothing)
  auto r_base = [](int r) { return 16 * (129 * r - 8 * r * (r - 1)); };
  // row 16 r + o of R from channel 16 r on, this lane's channels.  A step's row is read during the step before.  The scheduling
  // barriers between steps keep the compiler from reading all sixteen at once, the multiply-adds as volatile asm statements from
  // putting those of later channels off until after the loop (either way 16 rows of R in registers, and spills)
  auto fetch_row = [&](int r, int o, auto& to) {
    const double* from = rl + r_base(r) + o * (129 - 16 * r) + l16;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(to) / sizeof(double)); ++k) to[k] = from[16 * k];
  };

#pragma nounroll
  for (int c0 = o0; c0 < o1; c0 += kSB) {
    const int nb = min(kSB, (int)K - c0);
    const int64_t at = n * K + c0 + l16;
    // every load in range and unconditional, all requested before the first is used (a load under its own condition waits for
    // the one before: 8.6 thousand clocks for these 24); channels past K count nothing
    double acc[8], kept[8];
    float wo[8];
    const int last = nb - 1 - l16;  // (nb is a multiple of 8: what is clamped may be another lane's)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int at_r = min(16 * r, last);
      acc[r] = W64[at + at_r];
      kept[r] = keep[c0 + l16 + at_r];
      wo[r] = (float)w[at + at_r];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const bool in = 16 * r + l16 < nb;
      acc[r] = in ? acc[r] : 0.0;
      wo[r] = in && kept[r] != 0.0 ? wo[r] : 0.0f;
    }
    if (c0 > o0) {
      // This workgroup's W_i - q s of the channels since o0, by R; a wave takes channels 32 wave .. + 32, column 2 l16 + t in
      // tile t: both tiles' elements of a row of R are one 128-bit load.  The left operand, the same for every wave, goes
      // through LDS.  (Each wave fetching it for itself, and R in 64-bit loads, 80 loads a wave and 128 channels took 8.3
      // thousand clocks where the products take 4.1.)
#pragma nounroll
      for (int k = 2 * l16; k < c0 - o0; k += 32) {
        const int r = 4 * wave + q;
        *reinterpret_cast<double2*>(&rl[r * kLs + k]) = *reinterpret_cast<const double2*>(W64 + (n0 + r < N ? n0 + r : N - 1) * K + o0 + k);
      }
      __syncthreads();
      v4d m[2] = {};
      const uint32_t right = (uint32_t)(4 * q * ld + min((int64_t)c0 + 32 * wave + 2 * l16, K - 2));  // of row k + s: k = 4 q + s
      // 16 channels of k at a time, requested kAhead sixteens (1.5 thousand clocks of products) before they are multiplied
      constexpr int kAhead = 3;
      double2 rb[8][4];
      auto request = [&](int h, int k) {
#pragma unroll
        for (int s = 0; s < 4; ++s) rb[h][s] = *reinterpret_cast<const double2*>(A + (int64_t)(k + s) * ld + right);
        __builtin_amdgcn_sched_barrier(0);
      };
#pragma unroll
      for (int h = 0; h < kAhead; ++h) request(h, o0 + 16 * h);
#pragma nounroll
      for (int k = o0; k < c0; k += 128) {  // (c0 - o0 is a multiple of kSB)
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          request((h + kAhead) % 8, min(k + 16 * (h + kAhead), c0 - 16));  // (past the end: the last ones once more, unused)
          const double2* left = reinterpret_cast<const double2*>(&rl[l16 * kLs + k - o0 + 16 * h + 4 * q]);
          const double2 l0 = left[0], l1 = left[1];
          const double la[4] = {l0.x, l0.y, l1.x, l1.y};
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            m[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(la[x], rb[h][x].x, m[0], 0, 0, 0);
            m[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(la[x], rb[h][x].y, m[1], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v)
        *reinterpret_cast<double2*>(&rl[16 * kLs + (4 * v + q) * kXs + 32 * wave + 2 * l16]) = make_double2(m[0][v], m[1][v]);
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 8; ++r) acc[r] += rl[16 * kLs + (4 * wave + q) * kXs + 16 * r + l16];
      __syncthreads();
    }
    // R: strictly upper part; where i and j share a factorisation block it lies transposed below the diagonal.  16 x 16
    // tiles on and above the diagonal, nine to a wave; every load is requested before the first value is placed
    double e[9][4];
    {
      const double* block = A + (int64_t)c0 * ld + c0;
#pragma unroll
      for (int x = 0; x < 9; ++x) {
        const Tile g = upper_tile(wave + 4 * x);
        const int hi = (g.transposed ? g.t : g.r) * 16, lo = (g.transposed ? g.r : g.t) * 16;
        // nb is a multiple of 8, so four rows exist or not together; eight columns past the matrix's last row are still
        // the workspace's
#pragma unroll
        for (int v = 0; v < 4; ++v)
          e[x][v] = (block + (hi + 4 * v < nb ? hi + 4 * v : 0) * ld + (lo < nb ? lo : 0))[q * ld + l16];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int x = 0; x < 9; ++x) {
      const Tile g = upper_tile(wave + 4 * x);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = g.transposed ? l16 : 4 * v + q, j = g.transposed ? 4 * v + q : l16;
        const bool in = 16 * g.t + j > 16 * g.r + i && 16 * g.t + j < nb;
        rl[r_base(g.r) + 16 * (g.t - g.r) + i * (129 - 16 * g.r) + j] = in ? e[x][v] : 0.0;
      }
    }
    __syncthreads();

    double s;
    if constexpr (GROUP) {
      double z[8];
      float m = 0.0f;  // rounding is monotonic: the maximum may be rounded before it is complete (and passes over a NaN)
      float wz[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const bool number = __builtin_isfinite(wo[r]);
        wz[r] = wo[r];
        z[r] = acc[r] - (number ? (double)wo[r] : 0.0);
        acc[r] = number ? acc[r] : (double)wo[r];
      }
#define QQQ_SOLVE(O)                                                                                       \
  {                                                                                                        \
    double next[W];                                                                                        \
    if (O < 15) fetch_row(r, O + 1, next);                                                                 \
    fmac_row<O, true, W>(z, z[0], ri);                                                                     \
    if (O < 15) {                                                                                          \
      _Pragma("unroll") for (int k = 0; k < W; ++k) ri[k] = next[k];                                       \
    }                                                                                                      \
    __builtin_amdgcn_sched_barrier(0);                                                                     \
  }
      auto solve = [&](int r, auto width) {
        constexpr int W = decltype(width)::value;
        double ri[W];
        fetch_row(r, 0, ri);
        QQQ_SOLVE(0) QQQ_SOLVE(1) QQQ_SOLVE(2) QQQ_SOLVE(3) QQQ_SOLVE(4) QQQ_SOLVE(5) QQQ_SOLVE(6) QQQ_SOLVE(7)
        QQQ_SOLVE(8) QQQ_SOLVE(9) QQQ_SOLVE(10) QQQ_SOLVE(11) QQQ_SOLVE(12) QQQ_SOLVE(13) QQQ_SOLVE(14) QQQ_SOLVE(15)
        m = fmaxf(m, (float)fabs((double)wz[0] + z[0]));
#pragma unroll
        for (int k = 0; k < W - 1; ++k) {
          z[k] = z[k + 1];
          wz[k] = wz[k + 1];
        }
      };
#undef QQQ_SOLVE
      if (c0 == 0) {  // no moves yet, whatever R holds
#pragma unroll
        for (int r = 0; r < 8; ++r) m = fmaxf(m, fabsf(wo[r]));
      } else {
#pragma nounroll
        for (int r = 0; r < 4; ++r) solve(r, Width<8>{});
#pragma nounroll
        for (int r = 4; r < 8; ++r) solve(r, Width<4>{});
      }
      m = row_max(m);
      const uint16_t sb = __builtin_bit_cast(uint16_t, (_Float16)(m / 7.0f));
      if (l16 == 0 && row < N) scales[(int64_t)(c0 / kSB) * N + n] = sb;
      s = (double)half_bits_to_float(sb);
    } else {
      s = (double)half_bits_to_float(scales[n]);
    }
    const double rs = s == 0.0 ? 0.0 : 1.0 / s;  // 0 makes every quotient, and so every code, 0

#define QQQ_STEP(O)                                                                                        \
  {                                                                                                        \
    double next[W];                                                                                        \
    if (O < 15) fetch_row(r, O + 1, next);                                                                 \
    const double v = acc[0];                                                                               \
    const double q0 = v * rs;                                                                              \
    const double quo = __builtin_fma(__builtin_fma(-q0, s, v), rs, q0);                                    \
    const float code = keep_nan_clamp(__builtin_rintf((float)quo), 7.0f);                                  \
    const double diff = __builtin_fma(-(double)code, s, w0);                                               \
    fmac_row<O, false, W>(acc, diff, ri);                                                                  \
    own_code = l16 == O ? code : own_code;                                                                 \
    own_diff = l16 == O ? diff : own_diff;                                                                 \
    if (O < 15) {                                                                                          \
      _Pragma("unroll") for (int k = 0; k < W; ++k) ri[k] = next[k];                                       \
    }                                                                                                      \
    __builtin_amdgcn_sched_barrier(0);                                                                     \
  }
    auto steps = [&](int r, auto width) {
      constexpr int W = decltype(width)::value;
      const double w0 = (double)wo[0];
      float own_code = 0.0f;
      double own_diff = 0.0;
      double ri[W];
      fetch_row(r, 0, ri);
      QQQ_STEP(0) QQQ_STEP(1) QQQ_STEP(2) QQQ_STEP(3) QQQ_STEP(4) QQQ_STEP(5) QQQ_STEP(6) QQQ_STEP(7)
      QQQ_STEP(8) QQQ_STEP(9) QQQ_STEP(10) QQQ_STEP(11) QQQ_STEP(12) QQQ_STEP(13) QQQ_STEP(14) QQQ_STEP(15)
      const int nibble = own_code == own_code ? (int)own_code : 0;
      uint32_t word = ((uint32_t)nibble & 0xFu) << (4 * (l16 & 7));  // eight lanes make a word
      word |= quad_swap<1>(word);
      word |= quad_swap<2>(word);
      word |= half_row_mirror(word);
      if (row < N && 16 * r + l16 < nb) {
        if ((l16 & 7) == 0) w_nat[n * (K / 8) + c0 / 8 + 2 * r + (l16 >> 3)] = word;
        if (c0 + kSB < K) W64[at + 16 * r] = own_diff;
      }
#pragma unroll
      for (int k = 0; k < W - 1; ++k) {
        acc[k] = acc[k + 1];
        wo[k] = wo[k + 1];
      }
    };
#undef QQQ_STEP
#pragma nounroll
    for (int r = 0; r < 4; ++r) steps(r, Width<8>{});
#pragma nounroll
    for (int r = 4; r < 8; ++r) steps(r, Width<4>{});
    __syncthreads();  // R's place is free again, and W64 holds what the other waves wrote
  }
}

// After a per-group sweep, what the front-end derives from codes and group scales (Sec. 3.3.2, Fig. 5 offline):
// s_Wc[n] = fp16(max_k |code * s_Wg| / 127) with the product in fp32, s*_Wg = fp16(s_Wg / s_Wc) capped at
// 18.203125 (0 where s_Wc is 0), integer form clamp(rne(s*_Wg), 1, 18).  Sixteen lanes per output channel, a group each
// (one thread per output channel left most CUs idle: 48 us at K = 2048, N = 5632).
__global__ __launch_bounds__(256) void group_finish_kernel(const uint32_t* w_nat, const uint16_t* s_wg, int64_t N,
                                                           int64_t K, uint16_t* s_wc, uint16_t* s_star, int8_t* s_int) {
  const int l16 = threadIdx.x & 15;
  const int64_t row = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int64_t n = row < N ? row : N - 1;  // (rows past N repeat the last one and store nothing)
  const int G = (int)(K / QQQ_GROUP);
  float dmax = 0.0f;
  for (int g = l16; g < G; g += 16) {
    const uint32_t* words = w_nat + n * (K / 8) + g * (QQQ_GROUP / 8);
    uint32_t word[QQQ_GROUP / 8];
#pragma unroll
    for (int j = 0; j < QQQ_GROUP / 8; ++j) word[j] = words[j];
    int cmax = 0;
#pragma unroll
    for (int j = 0; j < QQQ_GROUP / 8; ++j)
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int code = ((int)(word[j] << (28 - 4 * b))) >> 28;  // sign-extended nibble
        cmax = max(cmax, code < 0 ? -code : code);
      }
    dmax = fmaxf(dmax, (float)cmax * half_bits_to_float(s_wg[g * N + n]));
  }
  dmax = row_max(dmax);
  if (row >= N) return;
  const uint16_t wcb = __builtin_bit_cast(uint16_t, (_Float16)(dmax / 127.0f));
  if (l16 == 0) s_wc[n] = wcb;
  const float wc = half_bits_to_float(wcb);
  for (int g = l16; g < G; g += 16) {
    uint16_t star = 0;
    if (wc != 0.0f) {
      const _Float16 h = (_Float16)(half_bits_to_float(s_wg[g * N + n]) / wc);
      star = __builtin_bit_cast(uint16_t, (float)h > 18.203125f ? (_Float16)18.203125f : h);
    }
    s_star[g * N + n] = star;
    if (s_int) s_int[g * N + n] = (int8_t)fminf(fmaxf(__builtin_rintf(half_bits_to_float(star)), 1.0f), 18.0f);
  }
}

int g_factor_workgroups = 0;  // qqq_set_factor_workgroups

// what both sweeps share: argument checks, the working copies, damping and the factorisation
struct Work { double *A, *W64, *keep; int ld; };
int64_t row_stride(int64_t K) { return ((K + 15) & ~(int64_t)15) + 16; }
int64_t flag_count(int64_t K) { const int64_t nb = (K + 63) / 64; return 32 + nb + 2 * nb * nb; }
int begin(const char* who, const void* w_fp16, const double* H, int64_t N, int64_t K, double percdamp,
          const uint32_t* w_nat, void* workspace, size_t workspace_bytes, hipStream_t st, Work* out) {
  if (N < 1 || N > 65535 || K < 8 || K % 8 != 0 || K > 16384 || !(percdamp >= 0.0) || percdamp > 1e6)
    return set_error(QQQ_ERR_SHAPE, "%s: unsupported N=%lld K=%lld percdamp=%g (need N <= 65535, K%%8==0, K <= 16384, "
                     "percdamp >= 0)", who, (long long)N, (long long)K, percdamp);
  if (!w_fp16 || !H || !w_nat || !workspace) return set_error(QQQ_ERR_NULL, "%s: null pointer argument", who);
  if (!aligned16(w_fp16) || !aligned16(workspace) || (reinterpret_cast<uintptr_t>(H) & 7u) ||
      (reinterpret_cast<uintptr_t>(w_nat) & 3u))
    return set_error(QQQ_ERR_SHAPE, "%s: w_fp16 and workspace must be 16-byte, H 8-byte, w_nat 4-byte aligned", who);
  const size_t need = qqq_gptq_workspace_bytes(N, K);
  if (workspace_bytes < need)
    return set_error(QQQ_ERR_WORKSPACE, "%s: workspace %zu bytes < %zu needed", who, workspace_bytes, need);
  char* base = (char*)((reinterpret_cast<uintptr_t>(workspace) + 127) & ~(uintptr_t)127);  // (cache lines: see factor_kernel)
  const int64_t ld = row_stride(K), n_flags = flag_count(K);
  double* A = (double*)base;
  double* W64 = (double*)(base + align256((size_t)K * ld * 8));
  double* keep = (double*)((char*)W64 + align256((size_t)N * K * 8));
  double* rcp = (double*)((char*)keep + align256((size_t)K * 8));
  uint32_t* flags = (uint32_t*)((char*)rcp + align256((size_t)K * 8));
  double* damp = (double*)((char*)flags + align256((size_t)n_flags * 4));
  int rc;
  hipLaunchKernelGGL(diagonal_kernel, dim3(1), dim3(1024), 0, st, H, K, percdamp, keep, damp);
  if ((rc = check_launch("gptq diagonal")) != QQQ_OK) return rc;
  hipLaunchKernelGGL(prepare_kernel, dim3((unsigned)(K + N < 4096 ? K + N : 4096)), dim3(256), 0, st, H,
                     (const _Float16*)w_fp16, keep, damp, N, K, A, ld, W64, flags, (int)n_flags);
  if ((rc = check_launch("gptq prepare")) != QQQ_OK) return rc;
  Factor f;
  f.A = A;
  f.rcp = rcp;
  f.K = (int)K;
  f.ld = (int)ld;
  f.nb = (int)((K + 63) / 64);
  f.ticket = flags;
  f.flags = flags + 32;
  // one workgroup of it fits a CU: the chain, and a tile for each of the others
  const int tiles = f.nb * (f.nb - 1) / 2, groups = 1 + min(tiles, num_cus() - 1), most = g_factor_workgroups;
  hipLaunchKernelGGL(factor_kernel, dim3((unsigned)(most > 0 && most < groups ? most : groups)), dim3(256), 0, st, f);
  if ((rc = check_launch("gptq factorisation")) != QQQ_OK) return rc;
  out->A = A;
  out->W64 = W64;
  out->keep = keep;
  out->ld = (int)ld;
  return QQQ_OK;
}

// Eq. 4 over all channels; scales: [N], or [K/128, N] (written) with group scales
template <bool GROUP>
int sweep(const Work& wk, const void* w_fp16, int64_t N, int64_t K, uint16_t* scales, uint32_t* w_nat, hipStream_t st) {
  // kSO channels at a time; all channels after those are moved by them together: passes over the running weights kept few,
  // and products deep enough for the matrix cores.  The next kSO channels need that at once; of the others the last ones go along with the next kSO's
  // sweep, whose chains leave the matrix cores idle: as many tiles as the workgroups that fit beside it get done in its time.
  const int sweepers = (int)((N + 15) / 16), row_tiles = (int)((N + 63) / 64), beside = 2 * num_cus() - sweepers;
  const int64_t carry = (int64_t)(beside > 0 ? beside * kCarried / row_tiles : 0) * 64;
  Carried cr = {};
  for (int64_t o0 = 0; o0 < K; o0 += kSO) {
    const int64_t o1 = o0 + kSO < K ? o0 + kSO : K, o2 = o1 + kSO < K ? o1 + kSO : K;
    const int tiles = cr.cols ? row_tiles * ((cr.cols + 63) / 64) : 0;
    hipLaunchKernelGGL((sweep_kernel<GROUP>), dim3((unsigned)(sweepers + tiles)), dim3(256), 0, st, (const _Float16*)w_fp16,
                       wk.A, wk.ld, wk.keep, N, K, (int)o0, (int)o1, scales, wk.W64, w_nat, sweepers, cr);
    if (o1 == K) break;
    const int64_t from = K - o2 > carry ? K - carry : o2;  // columns from here on go with the next sweep
    hipLaunchKernelGGL(f64_update_kernel, dim3((unsigned)((from - o1 + 63) / 64), (unsigned)row_tiles), dim3(256), 0, st,
                       wk.W64 + o0, K, wk.A + o0 * wk.ld + o1, (int64_t)wk.ld, wk.W64 + o1, K, (int)N, (int)(from - o1), kSO);
    cr = {wk.W64 + o0, wk.A + o0 * wk.ld + from, wk.W64 + from, (int)N, (int)(K - from), row_tiles};
  }
  return check_launch("gptq sweep");
}

}  // namespace

}  // namespace qqq

using namespace qqq;

extern "C" {

int qqq_set_factor_workgroups(int most) {
  const int before = g_factor_workgroups;
  if (most >= 0) g_factor_workgroups = most;
  return before;
}

size_t qqq_gptq_workspace_bytes(int64_t N, int64_t K) {
  if (N < 1 || N > 65535 || K < 8 || K % 8 != 0 || K > 16384) return 0;
  return align256((size_t)K * row_stride(K) * 8) + align256((size_t)N * K * 8) + 2 * align256((size_t)K * 8) +
         align256((size_t)flag_count(K) * 4) + 256 + 128;
}

int qqq_gptq_quantize_w4_perchannel(const void* w_fp16, const double* H, int64_t N, int64_t K, double percdamp,
                                    uint32_t* w_nat, void* s_w_fp16, void* workspace, size_t workspace_bytes,
                                    void* stream) {
  if (!s_w_fp16) return set_error(QQQ_ERR_NULL, "gptq: null pointer argument");
  if (reinterpret_cast<uintptr_t>(s_w_fp16) & 1u) return set_error(QQQ_ERR_SHAPE, "gptq: s_w must be 2-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  Work wk;
  int rc = begin("gptq", w_fp16, H, N, K, percdamp, w_nat, workspace, workspace_bytes, st, &wk);
  if (rc != QQQ_OK) return rc;
  // scales from the original weights (and round-to-nearest codes, overwritten block by block below)
  rc = launch_quant_weight(w_fp16, N, K, K, false, w_nat, (uint16_t*)s_w_fp16, nullptr, nullptr, nullptr, st);
  if (rc != QQQ_OK) return rc;
  return sweep<false>(wk, w_fp16, N, K, (uint16_t*)s_w_fp16, w_nat, st);
}

int qqq_gptq_quantize_w4_pergroup(const void* w_fp16, const double* H, int64_t N, int64_t K, int group, double percdamp,
                                  uint32_t* w_nat, void* s_wg_fp16, void* s_star_fp16, int8_t* s_int, void* s_wc_fp16,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  if (group != QQQ_GROUP) return set_error(QQQ_ERR_SHAPE, "gptq_pergroup: group must be 128, got %d", group);
  if (K % QQQ_GROUP != 0) return set_error(QQQ_ERR_SHAPE, "gptq_pergroup: K=%lld must be a multiple of 128", (long long)K);
  if (!s_wg_fp16 || !s_star_fp16 || !s_wc_fp16) return set_error(QQQ_ERR_NULL, "gptq_pergroup: null pointer argument");
  if ((reinterpret_cast<uintptr_t>(s_wg_fp16) | reinterpret_cast<uintptr_t>(s_star_fp16) |
       reinterpret_cast<uintptr_t>(s_wc_fp16)) & 1u)
    return set_error(QQQ_ERR_SHAPE, "gptq_pergroup: scale tables must be 2-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  Work wk;
  int rc = begin("gptq_pergroup", w_fp16, H, N, K, percdamp, w_nat, workspace, workspace_bytes, st, &wk);
  if (rc != QQQ_OK) return rc;
  uint16_t* s_wg = (uint16_t*)s_wg_fp16;
  if ((rc = sweep<true>(wk, w_fp16, N, K, s_wg, w_nat, st)) != QQQ_OK) return rc;
  hipLaunchKernelGGL(group_finish_kernel, dim3((unsigned)((N + 15) / 16)), dim3(256), 0, st, w_nat, s_wg, N, K,
                     (uint16_t*)s_wc_fp16, (uint16_t*)s_star_fp16, s_int);
  return check_launch("gptq_pergroup finish");
}

}  // extern "C"
