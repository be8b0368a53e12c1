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
// Both parts are blocked so that almost all of their arithmetic is fp64 MFMA (f64_update_kernel):
//   factorisation  per 64 channels, from the last: factor_panel_kernel, then the update of the channels before
//   sweep          per 512 channels, from the first: sweep_kernel, then the update of the channels after
// What is left serial is one dependent step per channel, in registers.
// Bound, without the Hessian: K = N = 4096 holds 2.3e10 + 6.9e10 fp64 operations, 1.2 ms at the nominal 78.6 TFLOP/s of the
// fp64 matrix cores (1.7 ms at the 54 that f64_update_kernel reaches).  Measured, K = N = 4096: 3.7 ms, and 4.0 ms with the
// Hessian of 2048 tokens (an inverse by K rank-1 sweeps and a rank-1 update of both matrices per channel: 360 ms); K = 2048,
// N = 5632 with group scales: 1.75 ms, 1.8 ms with the Hessian of 1111 tokens (81 ms).
#include "qqq_calib.h"
#include "qqq_internal.h"

#include <type_traits>

namespace qqq {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kFB = 64;    // channels per factorisation block
constexpr int kSB = 128;   // channels per sweep block (= a group of the per-group quantiser)
constexpr int kFO = 256, kSO = 512;  // channels after which the rest of the matrix is updated
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
                                                      const double* damp, int64_t N, int64_t K, double* A, double* W64) {
  for (int64_t r = blockIdx.x; r < K + N; r += gridDim.x) {
    if (r < K) {
      for (int64_t j = (r & ~(int64_t)1) + 2 * threadIdx.x; j < K; j += 512) {
        const int64_t at = r * K + j;
        double h0 = H[at], h1 = H[at + 1];  // (H is 8-byte aligned)
        if (j == r) h0 = (h0 == 0.0 ? 1.0 : h0) + damp[0];
        if (j + 1 == r) h1 = (h1 == 0.0 ? 1.0 : h1) + damp[0];
        *reinterpret_cast<double2*>(A + at) = make_double2(h0, h1);
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

// C += (or -=) A B in fp64: C [M,N], A [M,kd], B [kd,N], all row-major and 16-byte aligned, N, kd and the strides even.
// 64 x 64 tile per workgroup, a wave per 32 x 32 quarter, 32 of kd at a time through LDS with the next
// 32 already requested.  v_mfma_f64_16x16x4_f64 (64 clocks): lane l holds row (column) l % 16 and k = l / 16
// of the operands, register v of the result is row 4 v + l / 16, column l % 16.  Row strides of the LDS tiles
// (34 and 80 doubles) put the 32 lanes of half a wave on all 64 banks; each fragment read feeds two MFMAs.  M = 4096,
// N = 3584, kd = 512: 280 us, 54 TFLOP/s (MFMAs alone, operands in registers, reach 70 at the 2.15 GHz they then leave); 128 x 64
// tiles and fragments read four k ahead measured the same.  The second launch bound keeps the accumulators in the vector
// registers: left alone the compiler moves them to the accumulation registers and back every 32 of kd (303 us).
constexpr int kAs = 34, kBs = 80;  // row strides of the LDS tiles: 64 rows of A, 32 of B
template <bool SUB>
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
      double2 a = SUB ? make_double2(-ra[j].x, -ra[j].y) : ra[j];
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

// UPPER: C is columns col0 .. col0 + N of a symmetric matrix kept as its upper triangle; only the tiles that reach the
// diagonal or lie above it.
template <bool UPPER, bool SUB>
__global__ __launch_bounds__(256, 3) void f64_update_kernel(const double* A, int64_t lda, const double* B, int64_t ldb,
                                                         double* C, int64_t ldc, int M, int N, int kd, int col0) {
  __shared__ __attribute__((aligned(16))) double sa[64 * kAs];
  __shared__ __attribute__((aligned(16))) double sb[32 * kBs];
  if (UPPER && col0 + (int)blockIdx.x * 64 + 63 < (int)blockIdx.y * 64) return;
  update_tile<SUB>(A, lda, B, ldb, C, ldc, M, N, kd, blockIdx.y, blockIdx.x, sa, sb);
}

// One block [c0, c0 + 64) of H = R D R^T, the channels after it already eliminated from A.
// Every workgroup factors the 64 x 64 diagonal block for itself (64 dependent steps: column j's pivot
// d_j, R[i,j] = A[i,j] / d_j for i < j, A[i,k] -= R[i,j] A[k,j] for k < j) and then solves for its own 16 of
// the c0 rows above: y_j = a_j - sum_{k > j} y_k R[j,k], x_j = y_j / d_j, i.e. R = x and R D = y there.
// Written: x in place (A[row, c0 + j]) and y transposed into the unused lower triangle (A[c0 + j, row]),
// which is the row-major operand the update of the rows above wants; the diagonal block's R goes
// transposed below the diagonal (its upper half is still being read by other workgroups).
// Bound by the chain of 64 pivots and, where code runs once, by its fetch: both halves walk 16 columns at a time
// in a loop, so that one body of a few KiB serves the whole block (written out straight, 42 KiB of instructions
// took 44.7 us a block whatever the row count).
// Diagonal block, 16 columns at a time from the last: they receive what the columns after them owe (fp64 MFMA, a wave per 16 rows);
// one wave takes the 16 steps of the 16 x 16 tile on the diagonal, a lane a row, with what is broadcast as part of the
// multiply-adds and the next pivot's reciprocal between them; the waves of the rows above solve theirs by it, 16 lanes per row.
// In clocks, a block: loads 3900, 16 columns 4600 (a pivot 150, the rest the products, the rows above, barriers), rows 5000; 13.3 us a
// launch.  With lane = row for all 64 rows in one wave, pivots and column elements through v_readlane 8200 and 7400 for 32 rows: 21 us.
// The first `solvers` workgroups do that.  The others, on the CUs the chain leaves idle, take a part of what the kFO
// channels [t0, t0 + td) before these owe to the columns this kFO does not contain (Trailing): A[0..td0) -= R (R D)^T there,
// 64 x 64 tiles of the upper triangle numbered column by column from `tile0`.  They touch nothing a block of this kFO reads
// or writes: rows and columns below t0 - kFO, from operands at t0 and past it.
struct Trailing { int t0, td, n, tile0; };  // first channel, channels, rows (= columns) updated, first tile
__global__ __launch_bounds__(256, 2) void factor_panel_kernel(double* A, int64_t K, int c0, int solvers, Trailing tr) {
  constexpr int kS = 66;
  static_assert(64 * kS >= 64 * kAs && 64 * kS >= 32 * kBs, "an update tile's stages fit");
  // [i][j], in 16 x 16 tiles.  ys: the block's upper triangle; tiles above the diagonal become R D when their columns' turn comes, those on it
  // keep the block as the columns after left it.  xs: R in the tiles above the diagonal and on it, there 0 from the diagonal on,
  // each from its columns' turn on; the tiles below are never written, nor read
  __shared__ __attribute__((aligned(16))) double ys[64 * kS];
  __shared__ __attribute__((aligned(16))) double xs[64 * kS];
  __shared__ double rcp[64];                                   // 1 / d_j
  if ((int)blockIdx.x >= solvers) {
    const int u = tr.tile0 + (int)blockIdx.x - solvers;
    int tn = (int)((__builtin_sqrtf(8.0f * (float)u + 1.0f) - 1.0f) * 0.5f);  // tile column tn starts at tn (tn + 1) / 2
    while (tn * (tn + 1) / 2 > u) --tn;
    while ((tn + 1) * (tn + 2) / 2 <= u) ++tn;
    update_tile<true>(A + tr.t0, K, A + (int64_t)tr.t0 * K, K, A, K, tr.n, tr.n, tr.td, u - tn * (tn + 1) / 2, tn, ys, xs);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, q = lane >> 4;
  const int nb = min(64, (int)K - c0);
  // ---- the row this thread's sixteen lanes solve, this lane's columns 16 r + l16 in y[3 - r]
  const int64_t row = (int64_t)blockIdx.x * 16 + 4 * wave + q;
  double y[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) y[3 - r] = A[min(row, (int64_t)c0) * K + c0 + min(16 * r + l16, nb - 1)];  // (what is not there is not stored)

  // ---- the diagonal block, upper triangle; channels past K are identity
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int i = 4 * e + wave, j = lane;
    const double a = A[(int64_t)(c0 + min(i, nb - 1)) * K + c0 + max(min(i, nb - 1), min(j, nb - 1))];
    ys[i * kS + j] = (i <= j && j < nb) ? a : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
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
  if (blockIdx.x == 0) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = 4 * e + wave, i = lane;
      if (i < j && j < nb) A[(int64_t)(c0 + j) * K + c0 + i] = xs[i * kS + j];
    }
  }
  if (c0 == 0) return;
  // ---- the solve, column by column from the last; xs is zero from the diagonal on in the tiles on it.  The 16 columns in turn are always
  // y[0]: the others move up behind them (what moves into finished places is not used)
#pragma nounroll
  for (int p = 3; p >= 0; --p) {
    // R[16 (p - 3 + r) + l16][16 p + j]; where that row is before the block, row l16 feeds places no longer used
    const double* rr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) rr[3 - r] = xs + (16 * max(p - 3 + r, 0) + l16) * kS + 16 * p;
    double m[2][4];  // a column's, requested during the column before
#pragma unroll
    for (int r = 0; r < 4; ++r) m[1][r] = rr[r][15];
#define QQQ_SOLVE(J)                                                                                          \
  {                                                                                                           \
    if (J > 0) {                                                                                              \
      _Pragma("unroll") for (int r = 0; r < 4; ++r) m[(J + 1) & 1][r] = rr[r][J > 0 ? J - 1 : 0];             \
      __builtin_amdgcn_sched_barrier(0);                                                                      \
    }                                                                                                         \
    fmac_row<J, true, 4>(y, y[0], m[J & 1]);                                                                  \
  }
    QQQ_SOLVE(15) QQQ_SOLVE(14) QQQ_SOLVE(13) QQQ_SOLVE(12) QQQ_SOLVE(11) QQQ_SOLVE(10) QQQ_SOLVE(9) QQQ_SOLVE(8)
    QQQ_SOLVE(7) QQQ_SOLVE(6) QQQ_SOLVE(5) QQQ_SOLVE(4) QQQ_SOLVE(3) QQQ_SOLVE(2) QQQ_SOLVE(1) QQQ_SOLVE(0)
#undef QQQ_SOLVE
    const int col = 16 * p + l16;
    if (row < c0 && col < nb) A[row * K + c0 + col] = y[0] * rcp[col];
    ys[col * kS + 4 * wave + q] = y[0];  // (nothing reads the block's R D any more)
#pragma unroll
    for (int r = 0; r < 3; ++r) y[r] = y[r + 1];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int j = 16 * e + (tid >> 4), i = tid & 15;
    const int64_t to = (int64_t)blockIdx.x * 16 + i;
    if (j < nb && to < c0) A[(int64_t)(c0 + j) * K + to] = ys[j * kS + i];
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
template <bool GROUP>
__global__ __launch_bounds__(256, 2) void sweep_kernel(const _Float16* w, const double* A, const double* keep, int64_t N,
                                                    int64_t K, int o0, int o1, uint16_t* scales, double* W64,
                                                    uint32_t* w_nat) {
  constexpr int kRows = 16 * (16 * 36 + 8);  // doubles: 16 rows of 129 - 16 r for r = 0 .. 7
  // in the same place before R is: the product's 16 rows of the left operand and of the result
  constexpr int kLs = kSO - kSB + 2, kXs = kSB + 2;
  static_assert(16 * (kLs + kXs) <= kRows, "the product's operand and result fit");
  __shared__ __attribute__((aligned(16))) double rl[kRows + 64];  // (a step reads up to three vectors of 16 past its row)
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
      const uint32_t right = (uint32_t)(4 * q * K + min((int64_t)c0 + 32 * wave + 2 * l16, K - 2));  // of row k + s: k = 4 q + s
      // 16 channels of k at a time, requested kAhead sixteens (1.5 thousand clocks of products) before they are multiplied
      constexpr int kAhead = 3;
      double2 rb[8][4];
      auto request = [&](int h, int k) {
#pragma unroll
        for (int s = 0; s < 4; ++s) rb[h][s] = *reinterpret_cast<const double2*>(A + (int64_t)(k + s) * K + right);
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
      const double* block = A + (int64_t)c0 * K + c0;
#pragma unroll
      for (int x = 0; x < 9; ++x) {
        const Tile g = upper_tile(wave + 4 * x);
        const int hi = (g.transposed ? g.t : g.r) * 16, lo = (g.transposed ? g.r : g.t) * 16;
        // nb is a multiple of 8, so four rows exist or not together; eight columns past the matrix's last row are still
        // the workspace's
#pragma unroll
        for (int v = 0; v < 4; ++v)
          e[x][v] = (block + (hi + 4 * v < nb ? hi + 4 * v : 0) * (int)K + (lo < nb ? lo : 0))[q * (int)K + l16];
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

// what both sweeps share: argument checks, the working copies, damping and the factorisation
struct Work { double *A, *W64, *keep; };
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
  char* base = (char*)workspace;
  double* A = (double*)base;
  double* W64 = (double*)(base + align256((size_t)K * K * 8));
  double* keep = (double*)((char*)W64 + align256((size_t)N * K * 8));
  double* damp = (double*)((char*)keep + align256((size_t)K * 8));
  int rc;
  hipLaunchKernelGGL(diagonal_kernel, dim3(1), dim3(1024), 0, st, H, K, percdamp, keep, damp);
  if ((rc = check_launch("gptq diagonal")) != QQQ_OK) return rc;
  hipLaunchKernelGGL(prepare_kernel, dim3((unsigned)(K + N < 4096 ? K + N : 4096)), dim3(256), 0, st, H,
                     (const _Float16*)w_fp16, keep, damp, N, K, A, W64);
  if ((rc = check_launch("gptq prepare")) != QQQ_OK) return rc;
  // Blocks of 64 from the last; each at once reduces the columns of its own kFO, and all columns before those are
  // reduced by the whole kFO together (see sweep): the next kFO's columns at once, the rest inside the launches of the next
  // kFO's blocks, whose chains leave CUs idle.  Two workgroups of that kernel fit a CU, and up to seven for every four CUs what a
  // launch carries costs less in it than by itself (K = 4096: a launch takes 14.4 us without tiles, 17.7 with 226 workgroups, 23.4 with 436,
  // 27.7 with 498, 38.8 with 635); what is left then (the first columns) goes at once as well.
  auto reduce = [&](int64_t c0, int64_t kd, int64_t col0, int64_t cols, int64_t rows) {
    if (cols <= 0 || rows <= 0) return;
    hipLaunchKernelGGL((f64_update_kernel<true, true>), dim3((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64)),
                       dim3(256), 0, st, A + c0, K, A + c0 * K + col0, K, A + col0, K, (int)rows, (int)cols, (int)kd, (int)col0);
  };
  Trailing tr = {};
  int tiles_left = 0;  // of tr
  for (int64_t o0 = (K - 1) / kFO * kFO; o0 >= 0; o0 -= kFO) {
    const int64_t o1 = o0 + kFO < K ? o0 + kFO : K;
    for (int64_t c0 = (o1 - 1) / kFB * kFB; c0 >= o0; c0 -= kFB) {
      const int solvers = c0 ? (int)(c0 / 16) : 1;
      const int blocks_left = (int)((c0 - o0) / kFB) + 1;
      const int carried = (tiles_left + blocks_left - 1) / blocks_left;
      hipLaunchKernelGGL(factor_panel_kernel, dim3((unsigned)(solvers + carried)), dim3(256), 0, st, A, K, (int)c0, solvers, tr);
      tr.tile0 += carried;
      tiles_left -= carried;
      reduce(c0, K - c0 < kFB ? K - c0 : kFB, o0, c0 - o0, c0);
    }
    if (o0 == 0) break;
    const int64_t p0 = o0 - kFO;
    reduce(o0, o1 - o0, p0, kFO, o0);
    const int nt = (int)(p0 / 64), most = (kFO / kFB) * max(num_cus() * 7 / 4 - (int)(p0 / 16), 0);
    int at_once = 0;  // tile columns
    while (nt * (nt + 1) / 2 - at_once * (at_once + 1) / 2 > most) ++at_once;
    reduce(o0, o1 - o0, 0, (int64_t)at_once * 64, (int64_t)at_once * 64);
    tr = {(int)o0, (int)(o1 - o0), (int)p0, at_once * (at_once + 1) / 2};
    tiles_left = nt * (nt + 1) / 2 - tr.tile0;
  }
  if ((rc = check_launch("gptq factorisation")) != QQQ_OK) return rc;
  out->A = A;
  out->W64 = W64;
  out->keep = keep;
  return QQQ_OK;
}

// Eq. 4 over all channels; scales: [N], or [K/128, N] (written) with group scales
template <bool GROUP>
int sweep(const Work& wk, const void* w_fp16, int64_t N, int64_t K, uint16_t* scales, uint32_t* w_nat, hipStream_t st) {
  // kSO channels at a time; all channels after those are moved by them together: passes over the running weights kept few,
  // and products deep enough for the matrix cores
  for (int64_t o0 = 0; o0 < K; o0 += kSO) {
    const int64_t o1 = o0 + kSO < K ? o0 + kSO : K;
    hipLaunchKernelGGL((sweep_kernel<GROUP>), dim3((unsigned)((N + 15) / 16)), dim3(256), 0, st, (const _Float16*)w_fp16,
                       wk.A, wk.keep, N, K, (int)o0, (int)o1, scales, wk.W64, w_nat);
    if (o1 < K)
      hipLaunchKernelGGL((f64_update_kernel<false, false>), dim3((unsigned)((K - o1 + 63) / 64), (unsigned)((N + 63) / 64)),
                         dim3(256), 0, st, wk.W64 + o0, K, wk.A + o0 * K + o1, K, wk.W64 + o1, K, (int)N, (int)(K - o1),
                         (int)kSO, 0);
  }
  return check_launch("gptq sweep");
}

}  // namespace

}  // namespace qqq

using namespace qqq;

extern "C" {

size_t qqq_gptq_workspace_bytes(int64_t N, int64_t K) {
  if (N < 1 || N > 65535 || K < 8 || K % 8 != 0 || K > 16384) return 0;
  return align256((size_t)K * K * 8) + align256((size_t)N * K * 8) + 2 * align256((size_t)K * 8) + 256;
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
