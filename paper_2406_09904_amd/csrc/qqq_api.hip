// C-ABI entry points of libqqq: argument validation and kernel-family dispatch (host code only).
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <mutex>

#include "qqq_internal.h"

namespace qqq {

static thread_local char g_err[256] = "no error";
static thread_local char g_route[256] = "";
static int g_override = 0;
static int g_group_mode = 0;
static int g_fuse_quant = 1;

int set_error(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

// the kernels a call enqueued, for qqq_last_route(): launchers append, entry points reset
void route_reset() { g_route[0] = 0; }
void route_note(const char* fmt, ...) {
  const size_t used = strlen(g_route);
  if (used + 4 >= sizeof(g_route)) return;
  size_t at = used;
  if (used > 0) at += (size_t)snprintf(g_route + used, sizeof(g_route) - used, " + ");
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_route + at, sizeof(g_route) - at, fmt, ap);
  va_end(ap);
}

int num_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

static int g_prefill_tune = 0;    // 0 = automatic, see qqq_set_prefill_tuning
static int g_prefill_ksplit = 0;  // 0 = automatic
void set_prefill_tuning(int tune) { g_prefill_tune = tune; }
int get_prefill_tuning() { return g_prefill_tune; }
// ring depth of the 4-wave per-tile shapes: 0 = by the launch's workgroup count, else forced
int get_prefill_ring_depth() {
  return g_prefill_tune == 27 ? 6 : g_prefill_tune == 37 ? 3 : 0;
}
void set_prefill_ksplit(int s) { g_prefill_ksplit = s; }
int get_prefill_ksplit() { return g_prefill_ksplit; }

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

static bool gemm_shape_ok(int64_t M, int64_t N, int64_t K) {
  return M >= 0 && M <= 0x7FFFFFFF && N >= 16 && N % 16 == 0 && N <= 0x7FFFFFF0 && K >= 128 &&
         K % 128 == 0 && K <= 131072;
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// split-K slabs of the per-tile prefill kernel: up to kSplitRows rows of int32 partial sums in all
// (k_splits * M <= kSplitRows), for the row counts where a K split can pay
constexpr int64_t kSplitRows = 1024, kSplitMaxM = 512;
static size_t split_bytes(int64_t M, int64_t N) {
  return (M > kDecodeAlwaysMaxM && M <= kSplitMaxM) ? align256((size_t)kSplitRows * (size_t)N * 4) : 0;
}

// ---------------------------------------------------------------------------------------------
// Dispatch model: every fitted constant the automatic kernel choice uses, in one place.  Fitted to every forced
// choice on 2145 shapes (K = 1024 .. 11008, N = 1024 .. 28672, M = 17 .. 4096, five layers of the benchmark among them) and on 964 beyond
// them (K = 128 .. 65536, N = 16 .. 65536) times four conversions on one MI355X: GEMM launches back to back from HIP graphs replayed in turn, packed weights rotated through
// 512 MiB and more.
//   tile[]        one row per conversion (what an int4 weight costs to convert decides how much a tile gains from
//                 having many rows), one entry per tile shape.  With x workgroups per CU, r the whole part of x and f the
//                 rest, a launch of T k-steps (128 k) takes, in microseconds,
//                   x <= 1:  fixed + per_round     + T (alone (1 - x) + full x)
//                   x >  1:  fixed + per_round * x + T (rounds x + [f > 0] rest (1 - f))
//                 alone: a k-step of one workgroup on an idle chip; full: with one on every CU (shared bandwidth, lower
//                 clock); rounds: of a whole round when there are several; rest: what a partial last round costs beyond its
//                 share.  2 to 3 % rms on all of them.  An even spread or whole rounds alone miss by 10 to 30 %: M = 2048, K = 4096, N = 11008
//                 took 89 us in 1.4 rounds of 128 x 512 and takes 80 in 2.7 rounds of 128 x 256.  (The smoothing search's row is
//                 fitted to the differences between the four tiles on 2082 searches, so only its differences mean anything; on 4316 others,
//                 with the loops and quantisers of now, its pick is 0.2 % behind the best tile, 4 % in one of a hundred, 9 % at most, and
//                 a row fitted to those is no better.)  The rows of 192 x 256, 128 x 128 and 64 x 128, and from 8 k-steps on
//                 all of the per-channel (but 128 x 512) and biased ones, are fitted to 30000 launches of 3457 shapes of their own
//                 (2 to 4 % rms; 3 to 5 % below 8 k-steps); 2 % stand on rounds and rest of the per-channel 128 x 128 and 64 x 128, whose
//                 wrong choice costs more than the larger tiles' (up to 20 % on M = 309, K = 6656, N = 16432).
//   short_tile[]  the same below short_ksteps k-steps, where the filling of the ring and the epilogue make up most of a tile, with a
//                 last round that costs its own time whatever T:  x <= 1: fixed + per_round x + T (alone (1 - x) + full x);
//                 x > 1: fixed + per_round x + T rounds x + [f > 0] rest (1 - f).  5 % rms (7 to 9 % in the other form; with the
//                 rows of longer K the pick was up to 30 % off there, M = 1264, K = 256, N = 50432 62.6 us for 48.9).
//   trimmed[]     what a launch of shapes 1 to 4 takes of that where their tiles go without their last 32 rows: fitted to 32000 launches of 2485 shapes on
//                 kernels with and without (K = 1024 .. 11008, M = 33 .. 2000, also with a K split), 1 to 2 % rms, no bias; half as much below
//                 short_ksteps.  (Medians of 50 launches each were up to 0.04 lower, and 3 to 9 % were lost where they decided.)
//   stream_tbs    what the weight stream of a prefill launch reaches at best; where it is what bounds several tiles, the one with the
//                 least to do beside it is ahead (behind_stream).
//   prepass_*     the biased route beyond the K that its rows were fitted to: a part per 1000 of K (K = 37760, M = 66, N = 4496 48.8 us
//                 where the FMA route takes 38.2).
//   split_*       the K-split's slabs and its second kernel: a launch, a part per split (they are read one after the other), and a
//                 part per million raw int32 of the slabs (6 TB/s written and read).
//   margin_split, min_ksteps_per_split  a split must be 3 % cheaper (modelled), its parts four k-steps long.
//   margin_trimmed_split  a split 128 x 128 tile without its last 32 rows is modelled 4 % too cheap beside the 64 x 128 tile with its deep ring (scales
//                 <= 15, M = 148, K = 4352, N = 7376 22.4 us, 20.9 on 64 x 128): on 2000 shapes of M = 65 .. 1500 four picks are 3 % or more slower than
//                 those of untrimmed kernels with it, none 5 %; without it nine and three.
//   margin_persistent  per-channel, the persistent kernel and the same tile one by one are as close as the model's error up to
//                 40 k-steps (K = 5120, M = 2048, N = 13824: 118.8 and 119.0 us): there the persistent one keeps what is within
//                 3.5 %; from 64 on it is 5 % behind on average.
//   decode[]      the decode kernel at 17..64 rows, per conversion (per-channel; scale on partial sums; real-valued; saturating)
//                 and channel tiles of a workgroup (1, 2, 4 or more): with g = N K / 1e6 weights, x workgroups per CU, w the
//                 whole rounds over x, R the row tiles,  base + per_wg x R + g (w (a + b R) + c M).  5 to 9 % rms.
//   sliced[]      the same where a narrow layer's K is cut into S slices:  base + rows R + K / (1000 S) (step + step_rows R) +
//                 slice S + c g M.  7 to 11 % rms.  (M = 30, K = 58240, N = 16: 5.6 us sliced, 30 in the prefill kernels.)
// On 2000 other shapes of the first kind (four conversions each) the pick is 0.8 % behind the best forced choice on average, 7 % in
// one of a hundred, 27 % at most; on 988 of the second kind 1.1, 13 and 30 %.  Rows fitted anew, also with a term for the weight
// stream beside the tiles, change that by less than 0.1 % (what is missed most: 64 x 128 tiles of two to seven row tiles, whose weights
// come from memory for few rows, 10 to 25 % slower than modelled; fewer than 8 k-steps; saturating calls of 17 .. 32 rows that stay with
// the decode kernel for too long).
// Tests time the automatic pick against every forced pick on small grids (10 and 15 % bars).
enum CostClass : int { kCostChannel, kCostBias, kCostFma, kCostReal, kCostClamp, kCostLoss, kCostClasses };
static int cost_class(int mode) {
  switch (mode) {
    case kPerChannel: return kCostChannel;
    case kGroupBias:
    case kGroupBiasWide: return kCostBias;
    case kGroupClamp: return kCostClamp;
    case kGroupReal:
    case kGroupCvt: return kCostReal;
  }
  return kCostFma;
}
constexpr int kPersistent = 6;  // as a shape: the persistent kernel; the others are those of launch_gemm_prefill_dma
struct TileCost { int shape, bm, bn; double alone, full, rounds, rest, fixed, per_round; };
struct DecodeCost { double base, per_wg, a, b, c; };
struct SlicedCost { double base, rows, step, step_rows, slice, c; };
static const struct DispatchModel {
  TileCost tile[kCostClasses][7] = {
      {  // per-channel
          {0, 128, 512, 0.866, 1.409, 1.244, 1.272, -4.0, 12.5},
          {2, 192, 256, 0.672, 1.067, 0.976, 1.002, -1.5, 9.0},
          {3, 128, 256, 0.484, 0.752, 0.691, 0.736, -0.8, 6.8},
          {4, 128, 128, 0.351, 0.491, 0.421, 0.320, 2.6, 2.8},
          {5, 64, 128, 0.240, 0.320, 0.253, 0.156, 3.4, 1.2},
          {kPersistent, 128, 512, 0.968, 1.492, 1.380, 1.229, 0.9, 6.9}},
      {  // biased integer (with its pre-pass)
          {0, 128, 512, 1.140, 1.686, 1.498, 1.676, -1.9, 15.4},
          {1, 256, 256, 1.043, 1.592, 1.422, 1.591, -1.6, 15.4},
          {2, 192, 256, 0.842, 1.277, 1.151, 1.233, 0.9, 11.3},
          {3, 128, 256, 0.633, 0.970, 0.842, 0.983, 1.8, 8.4},
          {4, 128, 128, 0.439, 0.641, 0.506, 0.380, 5.8, 3.3},
          {5, 64, 128, 0.344, 0.483, 0.320, 0.259, 7.0, 1.2},
          {kPersistent, 128, 512, 1.228, 1.717, 1.599, 1.635, 2.1, 11.3}},
      {  // fp16 FMA
          {0, 128, 512, 1.717, 2.148, 2.074, 2.122, -4.4, 13.7},
          {1, 256, 256, 1.252, 1.677, 1.594, 1.715, -4.2, 13.0},
          {2, 192, 256, 1.052, 1.447, 1.381, 1.319, -1.6, 9.5},
          {3, 128, 256, 0.885, 1.146, 1.073, 1.080, -1.3, 7.6},
          {4, 128, 128, 0.572, 0.695, 0.561, 0.477, 2.6, 3.0},
          {5, 64, 128, 0.439, 0.540, 0.392, 0.366, 4.0, 0.7},
          {kPersistent, 128, 512, 1.704, 2.111, 2.087, 1.942, 0.2, 7.6}},
      {  // real-valued scale
          {0, 128, 512, 1.879, 2.220, 2.110, 2.285, -3.7, 13.0},
          {1, 256, 256, 1.318, 1.692, 1.613, 1.768, -3.4, 12.1},
          {2, 192, 256, 1.094, 1.396, 1.321, 1.374, -1.7, 9.5},
          {3, 128, 256, 0.923, 1.155, 1.065, 1.170, -0.8, 7.1},
          {4, 128, 128, 0.602, 0.723, 0.575, 0.521, 2.9, 2.8},
          {5, 64, 128, 0.526, 0.605, 0.422, 0.477, 4.2, 0.8}},
      {  // saturating
          {0, 128, 512, 2.642, 2.916, 2.728, 3.140, -3.9, 13.9},
          {1, 256, 256, 1.734, 2.045, 1.902, 2.213, -3.3, 12.5},
          {2, 192, 256, 1.536, 1.775, 1.624, 1.857, -1.6, 9.8},
          {3, 128, 256, 1.355, 1.564, 1.426, 1.659, -0.9, 7.6},
          {4, 128, 128, 0.783, 0.907, 0.697, 0.773, 3.4, 2.4},
          {5, 64, 128, 0.698, 0.780, 0.599, 0.689, 4.3, 0.5},
          {kPersistent, 128, 512, 2.720, 2.961, 2.840, 2.993, 0.9, 7.0}},
      {  // per-channel with the smoothing search's loss for an epilogue
          {0, 128, 512, 1.241, 1.263, 1.603, 2.400, -0.4, 12.4},
          {3, 128, 256, 0.806, 0.341, 0.898, 0.494, 0.8, 0.7},
          {4, 128, 128, 0.717, 0.446, 0.476, 0.185, 0.9, 0.4},
          {5, 64, 128, 0.551, 0.382, 0.235, 0.241, -1.2, 0.8}}};
  TileCost short_tile[kCostLoss][7] = {
      {  // per-channel
          {0, 128, 512, 1.043, 0.802, 1.454, 4.510, 6.3, 6.7},
          {2, 192, 256, 0.800, 0.859, 1.321, 3.741, 5.6, 4.6},
          {3, 128, 256, 0.595, 0.458, 0.869, 3.563, 4.4, 3.8},
          {4, 128, 128, 0.360, 0.409, 0.497, 0.304, 4.7, 2.0},
          {5, 64, 128, 0.261, 0.391, 0.273, 0.268, 3.9, 0.9},
          {kPersistent, 128, 512, 1.058, 0.414, 0.879, 4.655, 6.2, 7.2}},
      {  // biased integer (with its pre-pass)
          {0, 128, 512, 1.392, 0.916, 1.736, 6.391, 10.6, 8.7},
          {1, 256, 256, 1.312, 0.544, 1.711, 5.160, 11.2, 8.3},
          {2, 192, 256, 0.982, 0.793, 1.590, 5.199, 10.0, 6.0},
          {3, 128, 256, 0.775, 0.495, 0.938, 4.567, 8.3, 5.4},
          {4, 128, 128, 0.477, 0.444, 0.571, 0.387, 8.3, 2.7},
          {5, 64, 128, 0.353, 0.705, 0.334, 0.719, 7.2, 1.2},
          {kPersistent, 128, 512, 1.541, 0.624, 1.226, 6.961, 10.5, 9.1}},
      {  // fp16 FMA
          {0, 128, 512, 1.958, 1.462, 2.294, 7.365, 7.0, 6.9},
          {1, 256, 256, 1.455, 0.983, 1.841, 5.057, 6.8, 6.2},
          {2, 192, 256, 1.194, 1.149, 1.720, 4.806, 6.0, 4.7},
          {3, 128, 256, 1.011, 0.743, 1.201, 4.662, 4.8, 4.1},
          {4, 128, 128, 0.619, 0.642, 0.661, 1.047, 4.7, 2.0},
          {5, 64, 128, 0.477, 0.594, 0.363, 1.235, 3.8, 0.9},
          {kPersistent, 128, 512, 1.625, 0.686, 1.302, 7.576, 7.2, 7.7}},
      {  // real-valued scale
          {0, 128, 512, 2.105, 1.642, 2.494, 7.697, 7.0, 6.9},
          {1, 256, 256, 1.513, 1.067, 1.944, 5.290, 6.7, 6.1},
          {2, 192, 256, 1.222, 1.071, 1.669, 4.766, 6.0, 4.8},
          {3, 128, 256, 1.053, 0.769, 1.257, 4.754, 4.8, 4.1},
          {4, 128, 128, 0.655, 0.655, 0.695, 1.117, 4.8, 2.0},
          {5, 64, 128, 0.556, 0.688, 0.452, 1.345, 4.1, 0.9}},
      {  // saturating
          {0, 128, 512, 2.889, 2.406, 3.416, 9.570, 7.5, 6.9},
          {1, 256, 256, 1.945, 1.441, 2.398, 6.286, 7.0, 6.2},
          {2, 192, 256, 1.682, 1.438, 2.017, 5.916, 6.2, 5.1},
          {3, 128, 256, 1.505, 1.184, 1.733, 5.759, 5.0, 4.2},
          {4, 128, 128, 0.842, 0.843, 0.753, 2.243, 4.8, 2.0},
          {5, 64, 128, 0.727, 0.884, 0.582, 2.031, 3.8, 0.8},
          {kPersistent, 128, 512, 2.503, 1.467, 2.313, 9.922, 7.8, 7.8}}};
  double trimmed[kCostClasses][4] = {{1.0, 0.887, 0.930, 0.911}, {0.923, 0.905, 0.934, 0.911}, {0.928, 0.920, 0.938, 0.905},
                                     {0.931, 0.916, 0.949, 0.913}, {0.951, 0.949, 0.942, 0.951}, {1.0, 1.0, 1.0, 1.0}};
  double stream_tbs = 4.6, behind_stream = 0.1;
  double split_us = 2.05, split_part_us = 0.28, split_mint32_us = 1.33;
  double margin_split = 0.97, margin_persistent = 0.965, margin_trimmed_split = 1.04;
  int margin_persistent_ksteps = 40;
  int min_ksteps_per_split = 4, short_ksteps = 8;
  int prepass_k = 11800;
  double prepass_us = 0.227;
  DecodeCost decode[4][3] = {
      {{2.97, 0.131, 0.0384, 0.0299, 0.0012}, {2.92, 0.202, 0.0226, 0.0233, 0.0007}, {2.58, 0.498, 0.0401, 0.0138, 0.0002}},
      {{3.02, 0.110, 0.0341, 0.0338, 0.0014}, {3.07, 0.206, 0.0161, 0.0287, 0.0009}, {2.88, 0.467, 0.0333, 0.0214, 0.0002}},
      {{3.19, 0.180, 0.0443, 0.0395, 0.0009}, {3.20, 0.265, 0.0484, 0.0269, 0.0006}, {3.12, 0.528, 0.0793, 0.0170, 0.0}},
      {{3.21, 0.192, 0.1050, 0.0374, 0.0001}, {3.40, 0.269, 0.0908, 0.0275, 0.0003}, {3.28, 0.565, 0.1223, 0.0167, 0.0}}};
  SlicedCost sliced[4] = {{2.75, 0.521, 0.718, -0.135, 0.0228, 0.0048},
                          {3.07, 0.439, 0.526, -0.096, 0.0306, 0.0061},
                          {2.98, 0.582, 0.784, -0.184, 0.0270, 0.0064},
                          {1.57, 1.012, 1.906, -0.480, 0.0255, 0.0071}};
} kModel;

// Tile shape and K split of the prefill path.  A split launches splits x tiles workgroups of T / splits k-steps plus
// the reduce kernel, which writes and reads splits * M * N int32: it pays for long K and few tiles only (at most 1024 /
// splits rows).  products: that many of the same size in one launch.
struct PrefillPlan {
  int shape, k_splits;
  double us;  // modelled time of the GEMM
};
static PrefillPlan plan_prefill(int64_t M, int64_t N, int64_t K, int cost, bool can_split, int forced_split, int products = 1) {
  const int cus = num_cus();
  const int T = (int)(K / 128);
  const int splits[8] = {1, 2, 3, 4, 6, 8, 12, 16};
  const double stream_us = (double)N * (double)K * 0.5 / (kModel.stream_tbs * 1e6);
  PrefillPlan best = {0, 1, 0.0};
  double best_score = 0.0;
  const bool short_k = T < kModel.short_ksteps && cost < kCostLoss;
  const double prepass_us = cost == kCostBias && K > kModel.prepass_k ? kModel.prepass_us * 1e-3 * (double)(K - kModel.prepass_k) : 0.0;
  for (const TileCost& c : short_k ? kModel.short_tile[cost] : kModel.tile[cost]) {
    if (c.bm == 0) continue;
    // (the persistent kernel needs three k-steps a tile and does not split them)
    if (c.shape == kPersistent && (T < 3 || forced_split > 1)) continue;
    const int64_t tiles_c = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    for (int j = 0; j < 8; ++j) {
      int ks = splits[j];
      if (forced_split > 0) {  // the tuning knob: one split count, as far as it is allowed
        if (j > 0) break;
        ks = forced_split;
        if (M <= kSplitMaxM && ks > kSplitRows / M) ks = (int)(kSplitRows / M);
        if (!can_split || ks < 1) ks = 1;
      } else if (ks > 1 && (!can_split || c.shape == kPersistent || ks > kSplitRows / M || T / ks < kModel.min_ksteps_per_split)) {
        break;
      }
      const double x = (double)(tiles_c * ks * products) / cus, f = x - floor(x), t = (double)T / ks;
      double us = c.fixed + prepass_us;
      us += short_k || x > 1.0 ? c.per_round * x : c.per_round;
      if (x <= 1.0) us += t * (c.alone * (1.0 - x) + c.full * x);
      else us += t * c.rounds * x + (f > 0.0 ? (short_k ? 1.0 : t) * c.rest * (1.0 - f) : 0.0);
      const bool trimmed = c.shape >= 1 && c.shape <= 4 && trimmed_rows(M, c.bm) < c.bm;
      if (trimmed) {
        const double part = kModel.trimmed[cost][c.shape - 1];
        us *= short_k ? 0.5 * (1.0 + part) : part;
      }
      if (us < stream_us) us = stream_us - kModel.behind_stream * (stream_us - us);
      if (ks > 1) us += kModel.split_us + ks * (kModel.split_part_us + kModel.split_mint32_us * 1e-6 * (double)M * (double)N);
      double score = us;
      if (ks > 1) score /= kModel.margin_split;
      if (ks > 1 && trimmed && c.shape == 4) score *= kModel.margin_trimmed_split;
      if (c.shape == kPersistent && cost == kCostChannel && T <= kModel.margin_persistent_ksteps) score *= kModel.margin_persistent;
      if (best_score == 0.0 || score < best_score) best = {c.shape, ks, us}, best_score = score;
    }
  }
  return best;
}

int loss_shape(int64_t M, int64_t N, int64_t K, int points) { return plan_prefill(M, N, K, kCostLoss, false, 0, points).shape; }

// Modelled time of the clamp-free per-group prefill GEMM and which conversion gives it: the biased integer
// route pays a pre-pass launch, the fp16-FMA route more per k-step, so short launches take the latter.
static double pergroup_prefill_us(int64_t M, int64_t N, int64_t K, bool* bias_route) {
  const double bias = plan_prefill(M, N, K, kCostBias, true, g_prefill_ksplit).us;
  const double fma = plan_prefill(M, N, K, kCostFma, true, g_prefill_ksplit).us;
  if (bias_route) *bias_route = bias < fma;
  return bias < fma ? bias : fma;
}

// Kernel family of a call: 1 = decode (split-K) kernel, 2 = prefill kernels.  Up to 16 rows the
// decode kernel streams the weights at memory speed; beyond 64 it does not apply.  In between it
// re-reads the activations once per 32 or 64 channels and its time grows with M, while the prefill
// path's 64-row tiles do not care about M: the models decide, each with what the call's own conversion costs there.
// `cost`: any clamp-free integer scale is kCostFma (in the decode kernel its scale goes onto partial sums, in the
// prefill kernels it takes the better of two routes).
static int kernel_family(int64_t M, int64_t N, int64_t K, int cost) {
  if (g_override != 0) return g_override;
  if (M <= kDecodeAlwaysMaxM) return 1;
  if (M > kSkinnyMaxM) return 2;
  const bool clamp_free = cost == kCostFma || cost == kCostBias;
  const int row_tiles = (int)((M + 15) / 16);
  const int nt = decode_channel_tiles(N, row_tiles, cost == kCostChannel || clamp_free);  // the launcher's own rule
  const int row = cost == kCostChannel ? 0 : clamp_free ? 1 : cost == kCostReal ? 2 : 3;
  const int slices = decode_k_slices(N, K, nt);
  const double g = (double)N * (double)K * 1e-6, x = (double)(N / (16 * nt)) / num_cus();
  double decode_us;
  if (slices > 1) {
    const SlicedCost& d = kModel.sliced[row];
    decode_us = d.base + d.rows * row_tiles + 1e-3 * (double)K / slices * (d.step + d.step_rows * row_tiles) + d.slice * slices + d.c * g * (double)M;
  } else {
    const DecodeCost& d = kModel.decode[row][nt >= 4 ? 2 : nt - 1];
    decode_us = d.base + d.per_wg * x * row_tiles + g * (ceil(x) / x * (d.a + d.b * row_tiles) + d.c * (double)M);
  }
  const double prefill_us = clamp_free ? pergroup_prefill_us(M, N, K, nullptr) : plan_prefill(M, N, K, cost, true, g_prefill_ksplit).us;
  return prefill_us < decode_us ? 2 : 1;
}

// The family of one call.  The decode kernel cannot do without its workspace, the prefill kernels can: where both serve, the model
// only ranks them, and a call without the workspace (or with a smaller one, for instance one sized for more than 512 rows, which
// holds no slabs) is not refused for that rank.
static int call_family(int64_t M, int64_t N, int64_t K, int cost, const void* workspace, size_t workspace_bytes) {
  const int family = kernel_family(M, N, K, cost);
  const bool ranked = g_override == 0 && M > kDecodeAlwaysMaxM && M <= kSkinnyMaxM;
  if (family == 1 && ranked && (!workspace || workspace_bytes < qqq_gemm_workspace_bytes(M, N, K))) return 2;
  return family;
}

// per-group conversion route from the caller's promises about the group scales (and the codes)
static int group_mode(int sg_arg, int64_t M, int64_t N, int64_t K, const void* workspace, size_t workspace_bytes) {
  const bool symmetric = (sg_arg & QQQ_SG_SYMMETRIC_CODES) != 0;  // no code is -8
  const int sg_max = sg_arg & ~QQQ_SG_SYMMETRIC_CODES;
  int mode = kGroupClamp;
  const bool decode = call_family(M, N, K, kCostFma, workspace, workspace_bytes) == 1;
  if (sg_max >= 1 && sg_max <= 16) mode = decode ? kGroupLinear : kGroupFused;
  else if (symmetric && sg_max >= 17 && sg_max <= 18) mode = decode ? kGroupLinear : kGroupFusedWide;
  // (knob 3 asks for the fp16-FMA conversion: with scales of 17 and 18 that is its wide form)
  if (g_group_mode >= 1 && g_group_mode <= 3) mode = (g_group_mode == 3 && mode == kGroupFusedWide) ? mode : g_group_mode;
  return mode;
}

static bool sg_arg_ok(int sg_arg) {
  const int sg_max = sg_arg & ~QQQ_SG_SYMMETRIC_CODES;
  return sg_arg >= 0 && sg_max <= 127;
}

static size_t ws_rows(int64_t M) { return (size_t)(M < kSkinnyMaxM ? M : kSkinnyMaxM); }
// pre-pass buffers of the biased per-group route (prefill only): Rl, Rh [M][Gp], Bc [N][Gp]
static size_t bias_rows_bytes(int64_t M, int64_t K) {
  return M > kDecodeAlwaysMaxM ? align256((size_t)M * (size_t)(((K / 128) + 31) & ~31)) : 0;
}
static size_t bias_cols_bytes(int64_t M, int64_t N, int64_t K) {
  return M > kDecodeAlwaysMaxM ? align256((size_t)N * (size_t)(((K / 128) + 31) & ~31)) : 0;
}
static size_t ws_counter_bytes(int64_t N) { return ((size_t)(N / 16) * 4 + 255) & ~(size_t)255; }

static void bias_buffers(void* workspace, int64_t M, int64_t N, int64_t K, int8_t*& r_lo, int8_t*& r_hi,
                         int8_t*& bc) {
  char* base = (char*)workspace + ws_counter_bytes(N) + align256(ws_rows(M) * (size_t)N * 4);
  r_lo = (int8_t*)base;
  r_hi = (int8_t*)(base + bias_rows_bytes(M, K));
  bc = (int8_t*)(base + 2 * bias_rows_bytes(M, K));
}

// does gemm_common take the biased per-group route for this call? (same conditions as in there)
static bool takes_bias_route(int mode, int64_t M, int64_t N, int64_t K);

// Everything a GEMM call checks on the host; runs before the first launch of a call, so that an
// error means nothing was enqueued.  `fused`: the decode kernel quantises fp16 rows itself and takes
// no a_q / s_a.  `ws_needed`: out, the bytes the chosen kernel family requires (0 = optional).
static int gemm_validate(const int8_t* a_q, const float* s_a, const void* w_packed, const int8_t* s_g,
                         const void* s_w, void* y, int64_t M, int64_t N, int64_t K, void* workspace,
                         size_t workspace_bytes, int mode, bool fused) {
  if (!gemm_shape_ok(M, N, K))
    return set_error(QQQ_ERR_SHAPE, "gemm: unsupported shape M=%lld N=%lld K=%lld (need N%%16==0, "
                     "K%%128==0, 128<=K<=131072)", (long long)M, (long long)N, (long long)K);
  if (M == 0) return QQQ_OK;
  if ((!fused && (!a_q || !s_a)) || !w_packed || !s_w || !y || (mode != kPerChannel && !s_g))
    return set_error(QQQ_ERR_NULL, "gemm: null pointer argument");
  if (!aligned16(a_q) || !aligned16(w_packed) || !aligned16(y) || !aligned16(workspace) ||
      (reinterpret_cast<uintptr_t>(s_a) & 3u) || (reinterpret_cast<uintptr_t>(s_w) & 3u) ||
      (reinterpret_cast<uintptr_t>(s_g) & 3u))
    return set_error(QQQ_ERR_SHAPE, "gemm: a_q, w_packed, y and workspace must be 16-byte aligned, "
                     "s_a, s_w and s_g 4-byte aligned");
  if (((M + 63) / 64) * ((N + 127) / 128) > 0x7FFFFFFF)
    return set_error(QQQ_ERR_SHAPE, "gemm: too many output tiles for one launch");
  const int family = call_family(M, N, K, cost_class(mode), workspace, workspace_bytes);
  if (family == 1 && M > kSkinnyMaxM)
    return set_error(QQQ_ERR_SHAPE, "gemm: skinny kernel forced but M=%lld > %d", (long long)M,
                     kSkinnyMaxM);
  if (fused && family != 1) return set_error(QQQ_ERR_SHAPE, "gemm: fused quantisation needs the decode kernel");
  if (family == 1) {
    const size_t need = qqq_gemm_workspace_bytes(M, N, K);
    if (!workspace) return set_error(QQQ_ERR_NULL, "gemm: workspace is NULL");
    if (workspace_bytes < need)
      return set_error(QQQ_ERR_WORKSPACE, "gemm: workspace %zu bytes < %zu needed", workspace_bytes,
                       need);
  }
  return QQQ_OK;
}

static int gemm_common(const int8_t* a_q, const float* s_a, const void* w_packed, const int8_t* s_g,
                       const void* s_w, void* y, int32_t* acc_out, int64_t M, int64_t N, int64_t K,
                       void* workspace, size_t workspace_bytes, void* stream, int mode,
                       const void* a_fp16 = nullptr, int64_t lda = 0, bool row_sums_ready = false) {
  const bool fused = a_fp16 != nullptr;  // the decode kernel quantises the rows itself
  {
    const int rc = gemm_validate(a_q, s_a, w_packed, s_g, s_w, y, M, N, K, workspace, workspace_bytes, mode, fused);
    if (rc != QQQ_OK || M == 0) return rc;
  }
  const int family = call_family(M, N, K, cost_class(mode), workspace, workspace_bytes);
  GemmParams p;
  p.a_q = a_q;
  p.s_a = s_a;
  p.w = (const uint4*)w_packed;
  p.s_g = s_g;
  p.s_w = (const _Float16*)s_w;
  p.y = (_Float16*)y;
  p.acc_out = acc_out;
  p.M = (int)M;
  p.N = (int)N;
  p.K = (int)K;
  p.T = (int)(K / 128);
  p.ws_cnt = nullptr;
  p.ws_acc = nullptr;
  p.r_lo = p.r_hi = p.bias_w = nullptr;
  p.y_ref = nullptr;
  p.loss = nullptr;
  p.point_bytes = 0;
  p.k_splits = 1;
  p.part = nullptr;
  p.a_fp16 = (const uint4*)a_fp16;
  p.lda_vec = lda / 8;
  if (family == 1) {
    p.ws_cnt = (int32_t*)workspace;
    p.ws_acc = (int32_t*)((char*)workspace + ws_counter_bytes(N));
    return launch_gemm_skinny(p, mode, (hipStream_t)stream);
  }
  const int tune = get_prefill_tuning();
  if (mode == kGroupCvt) return launch_gemm_prefill_dma(p, mode, 0, (hipStream_t)stream);
  // Clamp-free per-group request with a workspace of the queried size: the biased integer
  // conversion (a pre-pass computes the per-group row sums it needs) instead of the fp16 FMA one
  if (takes_bias_route(mode, M, N, K) && workspace && workspace_bytes >= qqq_gemm_workspace_bytes(M, N, K)) {
    int8_t *r_lo, *r_hi, *bc;
    bias_buffers(workspace, M, N, K, r_lo, r_hi, bc);
    // (scales up to 18 with symmetric codes: bytes of (7 - code) * s_g instead of (code + 8) * s_g)
    const bool wide = mode == kGroupFusedWide;
    const int rc = launch_group_bias_prepass(a_q, s_g, M, N, K, r_lo, r_hi, bc, !row_sums_ready, wide ? 7 : 8,
                                             (hipStream_t)stream);
    if (rc != QQQ_OK) return rc;
    p.r_lo = r_lo;
    p.r_hi = r_hi;
    p.bias_w = bc;
    mode = wide ? kGroupBiasWide : kGroupBias;
  }
  // per-tile kernel, optionally with K split over several workgroups per tile (raw tiles into the
  // workspace's slabs, then the reduce kernel); the split needs a workspace of the queried size
  const bool can_split = split_bytes(M, N) > 0 && workspace &&
                         workspace_bytes >= qqq_gemm_workspace_bytes(M, N, K);
  auto per_tile = [&](int shape, int k_splits) {
    const int64_t cap = kSplitRows / M;
    if (k_splits > cap) k_splits = (int)cap;
    if (k_splits > p.T) k_splits = p.T;
    if (!can_split || k_splits < 2) return launch_gemm_prefill_dma(p, mode, shape, (hipStream_t)stream);
    p.k_splits = k_splits;
    p.part = (int32_t*)((char*)workspace + ws_counter_bytes(N) + align256(ws_rows(M) * (size_t)N * 4) +
                        2 * bias_rows_bytes(M, K) + bias_cols_bytes(M, N, K));
    const int rc = launch_gemm_prefill_dma(p, mode, shape, (hipStream_t)stream);
    return rc != QQQ_OK ? rc : launch_splitk_reduce(p, mode, (hipStream_t)stream);
  };
  const int forced_split = get_prefill_ksplit();
  if ((tune >= 10 && tune <= 12) || (tune >= 15 && tune <= 17) || tune == 27 || tune == 37)
    return per_tile(tune == 12 ? 2 : tune >= 15 ? tune % 10 - 2 : (tune == 10 && mode != kPerChannel ? 1 : 0), forced_split > 0 ? forced_split : 1);
  if (tune == 13) return launch_gemm_prefill_ring(p, mode, (hipStream_t)stream);
  {
    const PrefillPlan plan = plan_prefill(M, N, K, cost_class(mode), can_split, forced_split);
    // The persistent kernel's next tile loads its first k-steps under the epilogue: ahead on short K with many tiles (per-channel K = 1024,
    // N = 27664, M = 2650 81 us against 95; saturating K = 1024, N = 16448, M = 1874 60 against 68), behind elsewhere.
    if (plan.shape == kPersistent) return launch_gemm_prefill_ring(p, mode, (hipStream_t)stream);
    return per_tile(plan.shape, plan.k_splits);
  }
}

static bool takes_bias_route(int mode, int64_t M, int64_t N, int64_t K) {
  // (the workspace holds the pre-pass buffers only above the rows that always take the decode kernel)
  if (!((mode == kGroupFused || mode == kGroupFusedWide) && M > kDecodeAlwaysMaxM &&
        (g_group_mode == 0 || g_group_mode == 5) &&
        kernel_family(M, N, K, kCostFma) == 2))
    return false;
  if (g_group_mode == 5) return true;  // forced
  bool bias = true;
  pergroup_prefill_us(M, N, K, &bias);
  return bias;
}

// One launch that quantises and multiplies.  Every workgroup quantises all M rows for itself, which a
// second launch (2.7-3.3 us) costs more than: always up to 8192 activations, up to 32768 with two or three
// rows, and with four rows on the large layers only (measured on five layers: M=2 0.8-2.5 us ahead everywhere,
// M=3 0.1-1.7 us; M=4 0.8 us ahead on 8192 x 28672, 0.2 us behind on the layers of 70 M weights and less).
static bool fused_ok(int64_t M, int64_t N, int64_t K) {
  if (!(g_override == 0 && g_fuse_quant && M >= 1 && M <= kFusedMaxM && M * K <= kFusedLdsBytes)) return false;
  return M * K <= kFusedLdsSmall || M <= 3 || (double)N * (double)K >= 1.5e8;
}

// quant_act followed by the GEMM; for a few decode rows a single launch that does both
static int linear_common(const void* a_fp16, int64_t lda, const void* w_packed, const int8_t* s_g,
                         const void* s_w, void* y, int32_t* acc_out, int64_t M, int64_t N, int64_t K,
                         void* workspace, size_t workspace_bytes, void* stream, int mode) {
  if (!gemm_shape_ok(M, N, K))
    return set_error(QQQ_ERR_SHAPE, "linear: unsupported shape M=%lld N=%lld K=%lld (need N%%16==0, "
                     "K%%128==0, 128<=K<=131072)", (long long)M, (long long)N, (long long)K);
  if (lda < K || lda % 8 != 0)
    return set_error(QQQ_ERR_SHAPE, "linear: lda=%lld must be >= K and a multiple of 8", (long long)lda);
  if (M == 0) return QQQ_OK;
  if (!a_fp16 || !workspace) return set_error(QQQ_ERR_NULL, "linear: null pointer argument");
  if (!aligned16(a_fp16) || !aligned16(workspace))
    return set_error(QQQ_ERR_SHAPE, "linear: a_fp16 and workspace must be 16-byte aligned");
  const size_t need = qqq_linear_workspace_bytes(M, N, K);
  if (workspace_bytes < need)
    return set_error(QQQ_ERR_WORKSPACE, "linear: workspace %zu bytes < %zu needed", workspace_bytes, need);
  const size_t gemm_ws = align256(qqq_gemm_workspace_bytes(M, N, K));
  if (fused_ok(M, N, K))
    return gemm_common(nullptr, nullptr, w_packed, s_g, s_w, y, acc_out, M, N, K, workspace, gemm_ws,
                       stream, mode, a_fp16, lda);
  float* s_a = (float*)((char*)workspace + gemm_ws);
  int8_t* a_q = (int8_t*)((char*)workspace + gemm_ws + align256((size_t)M * 4));
  {  // the GEMM's own checks, before the quantiser is enqueued: an error leaves nothing behind
    const int rc = gemm_validate(a_q, s_a, w_packed, s_g, s_w, y, M, N, K, workspace, gemm_ws, mode, false);
    if (rc != QQQ_OK) return rc;
  }
  // the per-group prefill GEMM's biased route wants per-group row sums of the codes: the quantiser
  // has them in registers, so it writes them on the way
  int8_t *r_lo = nullptr, *r_hi = nullptr, *bc = nullptr;
  const bool sums = takes_bias_route(mode, M, N, K);
  if (sums) bias_buffers(workspace, M, N, K, r_lo, r_hi, bc);
  const int rc = launch_quant_act(a_fp16, M, K, lda, a_q, s_a, (hipStream_t)stream, r_lo, r_hi);
  if (rc != QQQ_OK) return rc;
  return gemm_common(a_q, s_a, w_packed, s_g, s_w, y, acc_out, M, N, K, workspace, gemm_ws, stream, mode,
                     nullptr, 0, sums);
}

// ---- scratch of the entry point that allocates nothing: a device array that lives in the code
// object (one copy per GPU, held until the process ends).  Host code never uses the array's name as
// an address: the per-device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[QQQ_STATIC_SCRATCH_BYTES];
static void* g_scratch_ptr[64] = {nullptr};
static std::mutex g_scratch_mu;

static int static_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
    return set_error(QQQ_ERR_HIP, "static scratch: no current device");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || ptr == nullptr)
      return set_error(QQQ_ERR_HIP, "static scratch: hipGetSymbolAddress: %s", hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return QQQ_OK;
}

// entries of an int8 group-scale table outside 0..sg_max, counted by one workgroup (a diagnostic:
// speed is beside the point, a single plain store of the total is)
__global__ __launch_bounds__(1024) void sg_violation_kernel(const uint32_t* s_g, int64_t words, int sg_max,
                                                            int32_t* out) {
  __shared__ int total;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  int bad = 0;
  for (int64_t i = threadIdx.x; i < words; i += 1024) {
    const uint32_t w = s_g[i];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int v = (int)(int8_t)((w >> (8 * b)) & 0xFFu);
      bad += (v < 0 || v > sg_max) ? 1 : 0;
    }
  }
  if (bad) atomicAdd(&total, bad);
  __syncthreads();
  if (threadIdx.x == 0) *out = total;
}

// zero fill by a kernel (a memset node recorded into a captured graph is avoided on purpose)
__global__ __launch_bounds__(256) void zero_fill_kernel(uint4* p, size_t n16) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
    p[i] = make_uint4(0, 0, 0, 0);
}

}  // namespace qqq

using namespace qqq;

extern "C" {

int qqq_version(void) { return 100; }

const char* qqq_last_error(void) { return g_err; }

const char* qqq_last_route(void) { return g_route; }

int qqq_debug_count_sg_violations(const int8_t* s_g, int64_t N, int64_t K, int sg_max, int32_t* violations,
                                  void* stream) {
  if (N < 4 || N % 4 != 0 || K < 128 || K % 128 != 0 || sg_max < 0 || sg_max > 127 || (K / 128) * N > 0x7FFFFFFFLL * 4)
    return set_error(QQQ_ERR_SHAPE, "count_sg_violations: unsupported N=%lld K=%lld sg_max=%d", (long long)N,
                     (long long)K, sg_max);
  if (!s_g || !violations) return set_error(QQQ_ERR_NULL, "count_sg_violations: null pointer argument");
  if ((reinterpret_cast<uintptr_t>(s_g) & 3u) || (reinterpret_cast<uintptr_t>(violations) & 3u))
    return set_error(QQQ_ERR_SHAPE, "count_sg_violations: pointers must be 4-byte aligned");
  const int64_t words = (K / 128) * N / 4;
  hipLaunchKernelGGL(sg_violation_kernel, dim3(1), dim3(1024), 0, (hipStream_t)stream, (const uint32_t*)s_g, words,
                     sg_max, violations);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(QQQ_ERR_HIP, "count_sg_violations launch: %s", hipGetErrorString(e));
  return QQQ_OK;
}

int qqq_set_kernel_override(int family) {
  const int old = g_override;
  if (family >= 0 && family <= 2) g_override = family;
  return old;
}

int qqq_quant_act(const void* a_fp16, int64_t M, int64_t K, int64_t lda, int8_t* a_q, float* s_a,
                  void* stream) {
  route_reset();
  if (M < 0 || M > 0x7FFFFFFF || K < 8 || K % 8 != 0 || K > (1 << 24) || lda < K || lda % 8 != 0)
    return set_error(QQQ_ERR_SHAPE, "quant_act: unsupported M=%lld K=%lld lda=%lld (need K%%8==0, "
                     "lda%%8==0, lda>=K)", (long long)M, (long long)K, (long long)lda);
  if (M == 0) return QQQ_OK;
  if (!a_fp16 || !a_q || !s_a) return set_error(QQQ_ERR_NULL, "quant_act: null pointer argument");
  if (!aligned16(a_fp16) || (reinterpret_cast<uintptr_t>(a_q) & 7u))
    return set_error(QQQ_ERR_SHAPE, "quant_act: a_fp16 must be 16-byte and a_q 8-byte aligned");
  return launch_quant_act(a_fp16, M, K, lda, a_q, s_a, (hipStream_t)stream);
}

static int quantize_w4_check(const char* who, const void* w_fp16, int64_t N, int64_t K, int64_t ldw,
                             int64_t k_mult, const void* w_nat, const void* s_ch) {
  if (N < 0 || N > 0x7FFFFFFF || K < k_mult || K % k_mult != 0 || K > (1 << 24) || ldw < K || ldw % 8 != 0)
    return set_error(QQQ_ERR_SHAPE, "%s: unsupported N=%lld K=%lld ldw=%lld (need K%%%lld==0, ldw%%8==0, "
                     "ldw>=K)", who, (long long)N, (long long)K, (long long)ldw, (long long)k_mult);
  if (N == 0) return QQQ_OK;
  if (!w_fp16 || !w_nat || !s_ch) return set_error(QQQ_ERR_NULL, "%s: null pointer argument", who);
  if (!aligned16(w_fp16) || (reinterpret_cast<uintptr_t>(w_nat) & 3u) || (reinterpret_cast<uintptr_t>(s_ch) & 1u))
    return set_error(QQQ_ERR_SHAPE, "%s: w_fp16 must be 16-byte, w_nat 4-byte and the scales 2-byte aligned", who);
  return QQQ_OK;
}

int qqq_quantize_w4_perchannel(const void* w_fp16, int64_t N, int64_t K, int64_t ldw, uint32_t* w_nat,
                               void* s_w_fp16, void* stream) {
  const int rc = quantize_w4_check("quantize_w4_perchannel", w_fp16, N, K, ldw, 8, w_nat, s_w_fp16);
  if (rc != QQQ_OK || N == 0) return rc;
  return launch_quant_weight(w_fp16, N, K, ldw, false, w_nat, (uint16_t*)s_w_fp16, nullptr, nullptr, nullptr,
                             (hipStream_t)stream);
}

int qqq_quantize_w4_pergroup(const void* w_fp16, int64_t N, int64_t K, int64_t ldw, int group,
                             uint32_t* w_nat, void* s_star_fp16, int8_t* s_int, void* s_wc_fp16,
                             void* s_wg_fp16, void* stream) {
  if (group != QQQ_GROUP) return set_error(QQQ_ERR_SHAPE, "quantize_w4_pergroup: group must be %d", QQQ_GROUP);
  const int rc = quantize_w4_check("quantize_w4_pergroup", w_fp16, N, K, ldw, QQQ_GROUP, w_nat, s_wc_fp16);
  if (rc != QQQ_OK || N == 0) return rc;
  if (!s_star_fp16) return set_error(QQQ_ERR_NULL, "quantize_w4_pergroup: null s_star_fp16");
  if ((reinterpret_cast<uintptr_t>(s_star_fp16) & 1u) || (reinterpret_cast<uintptr_t>(s_wg_fp16) & 1u))
    return set_error(QQQ_ERR_SHAPE, "quantize_w4_pergroup: fp16 scale tables must be 2-byte aligned");
  return launch_quant_weight(w_fp16, N, K, ldw, true, w_nat, (uint16_t*)s_wc_fp16, (uint16_t*)s_wg_fp16,
                             (uint16_t*)s_star_fp16, s_int, (hipStream_t)stream);
}

int qqq_set_group_mode_override(int mode) {
  const int old = g_group_mode;
  if (mode >= 0 && mode <= 5) g_group_mode = mode;
  return old;
}

int qqq_set_skinny_tuning(int channel_tiles, int k_slices, int waves, int depth) {
  set_skinny_tuning(channel_tiles, k_slices, waves, depth);
  return 0;
}

int qqq_set_prefill_ksplit(int k_splits) {
  const int old = get_prefill_ksplit();
  if (k_splits >= 0) set_prefill_ksplit(k_splits);
  return old;
}

int qqq_set_prefill_tuning(int tune) {
  set_prefill_tuning(tune);
  return 0;
}


size_t qqq_packed_w4_bytes(int64_t N, int64_t K) {
  if (N < 16 || N % 16 != 0 || K < 128 || K % 128 != 0 || K > 131072 || N > 0x7FFFFFF0) return 0;
  return (size_t)N * (size_t)K / 2;
}

static int pack_common(const void* src, int64_t N, int64_t K, void* dst, bool inverse, void* stream) {
  if (qqq_packed_w4_bytes(N, K) == 0)
    return set_error(QQQ_ERR_SHAPE, "pack: unsupported N=%lld K=%lld (need N%%16==0, K%%128==0)",
                     (long long)N, (long long)K);
  if (!src || !dst) return set_error(QQQ_ERR_NULL, "pack: null pointer argument");
  if (src == dst) return set_error(QQQ_ERR_SHAPE, "pack: in-place repack is not supported");
  return launch_pack((const uint32_t*)src, N, K, (uint32_t*)dst, inverse, (hipStream_t)stream);
}

int qqq_pack_w4(const uint32_t* w_nat, int64_t N, int64_t K, void* w_packed, void* stream) {
  return pack_common(w_nat, N, K, w_packed, false, stream);
}

int qqq_unpack_w4(const void* w_packed, int64_t N, int64_t K, uint32_t* w_nat, void* stream) {
  return pack_common(w_packed, N, K, w_nat, true, stream);
}

size_t qqq_gemm_workspace_zero_bytes(int64_t M, int64_t N, int64_t K) {
  if (!gemm_shape_ok(M, N, K)) return 0;
  return ws_counter_bytes(N) + align256(ws_rows(M) * (size_t)N * 4);
}

size_t qqq_gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) {
  if (!gemm_shape_ok(M, N, K)) return 0;
  return ws_counter_bytes(N) + align256(ws_rows(M) * (size_t)N * 4) + 2 * bias_rows_bytes(M, K) +
         bias_cols_bytes(M, N, K) + split_bytes(M, N);
}

int qqq_gemm_w4a8_perchannel(const int8_t* a_q, const float* s_a, const void* w_packed,
                             const void* s_w_fp16, void* y_fp16, int32_t* acc_out, int64_t M,
                             int64_t N, int64_t K, void* workspace, size_t workspace_bytes,
                             void* stream) {
  route_reset();
  return gemm_common(a_q, s_a, w_packed, nullptr, s_w_fp16, y_fp16, acc_out, M, N, K, workspace,
                     workspace_bytes, stream, kPerChannel);
}

int qqq_gemm_w4a8_pergroup(const int8_t* a_q, const float* s_a, const void* w_packed,
                           const int8_t* s_g, const void* s_w_fp16, int group, int sg_max,
                           void* y_fp16, int32_t* acc_out, int64_t M, int64_t N, int64_t K,
                           void* workspace, size_t workspace_bytes, void* stream) {
  route_reset();
  if (group != QQQ_GROUP) return set_error(QQQ_ERR_SHAPE, "pergroup: group must be 128, got %d", group);
  if (!sg_arg_ok(sg_max))
    return set_error(QQQ_ERR_SHAPE, "pergroup: sg_max must be in 0..127 (optionally or-ed with "
                     "QQQ_SG_SYMMETRIC_CODES), got %d", sg_max);
  return gemm_common(a_q, s_a, w_packed, s_g, s_w_fp16, y_fp16, acc_out, M, N, K, workspace,
                     workspace_bytes, stream, group_mode(sg_max, M, N, K, workspace, workspace_bytes));
}

int qqq_gemm_w4a8_pergroup_f16scale(const int8_t* a_q, const float* s_a, const void* w_packed,
                                    const void* s_g_fp16, const void* s_w_fp16, int group,
                                    void* y_fp16, int32_t* acc_out, int64_t M, int64_t N, int64_t K,
                                    void* workspace, size_t workspace_bytes, void* stream) {
  route_reset();
  if (group != QQQ_GROUP) return set_error(QQQ_ERR_SHAPE, "pergroup: group must be 128, got %d", group);
  // knob 4: the conventional-conversion ablation of Fig. 9 (prefill kernel only)
  const int mode = (g_group_mode == 4 && call_family(M, N, K, kCostReal, workspace, workspace_bytes) == 2) ? kGroupCvt : kGroupReal;
  return gemm_common(a_q, s_a, w_packed, (const int8_t*)s_g_fp16, s_w_fp16, y_fp16, acc_out, M, N, K,
                     workspace, workspace_bytes, stream, mode);
}

size_t qqq_linear_workspace_bytes(int64_t M, int64_t N, int64_t K) {
  if (!gemm_shape_ok(M, N, K)) return 0;
  return align256(qqq_gemm_workspace_bytes(M, N, K)) + align256((size_t)M * 4) + (size_t)M * (size_t)K;
}

int qqq_set_fused_quant(int enable) {
  const int old = g_fuse_quant;
  g_fuse_quant = enable ? 1 : 0;
  return old;
}

int qqq_linear_w4a8_perchannel(const void* a_fp16, int64_t lda, const void* w_packed,
                               const void* s_w_fp16, void* y_fp16, int32_t* acc_out, int64_t M,
                               int64_t N, int64_t K, void* workspace, size_t workspace_bytes,
                               void* stream) {
  route_reset();
  return linear_common(a_fp16, lda, w_packed, nullptr, s_w_fp16, y_fp16, acc_out, M, N, K, workspace,
                       workspace_bytes, stream, kPerChannel);
}

int qqq_linear_w4a8_pergroup(const void* a_fp16, int64_t lda, const void* w_packed, const int8_t* s_g,
                             const void* s_w_fp16, int group, int sg_max, void* y_fp16,
                             int32_t* acc_out, int64_t M, int64_t N, int64_t K, void* workspace,
                             size_t workspace_bytes, void* stream) {
  route_reset();
  if (group != QQQ_GROUP) return set_error(QQQ_ERR_SHAPE, "pergroup: group must be 128, got %d", group);
  if (!sg_arg_ok(sg_max))
    return set_error(QQQ_ERR_SHAPE, "pergroup: sg_max must be in 0..127 (optionally or-ed with "
                     "QQQ_SG_SYMMETRIC_CODES), got %d", sg_max);
  return linear_common(a_fp16, lda, w_packed, s_g, s_w_fp16, y_fp16, acc_out, M, N, K, workspace,
                       workspace_bytes, stream, group_mode(sg_max, M, N, K, workspace, workspace_bytes));
}

int qqq_linear_w4a8_perchannel_static(const void* a_fp16, int64_t lda, const void* w_packed,
                                      const void* s_w_fp16, void* y_fp16, int32_t* acc_out, int64_t M,
                                      int64_t N, int64_t K, void* stream) {
  route_reset();
  if (!gemm_shape_ok(M, N, K))
    return set_error(QQQ_ERR_SHAPE, "linear_static: unsupported shape M=%lld N=%lld K=%lld (need N%%16==0, "
                     "K%%128==0, 128<=K<=131072)", (long long)M, (long long)N, (long long)K);
  const size_t need = qqq_linear_workspace_bytes(M, N, K);
  if (need > (size_t)QQQ_STATIC_SCRATCH_BYTES)
    return set_error(QQQ_ERR_WORKSPACE, "linear_static: M=%lld N=%lld K=%lld needs %zu bytes of scratch, the "
                     "static scratch holds %zu; use qqq_linear_w4a8_perchannel with a workspace",
                     (long long)M, (long long)N, (long long)K, need, (size_t)QQQ_STATIC_SCRATCH_BYTES);
  if (M == 0) return QQQ_OK;
  // everything linear_common checks before its first launch, checked here before the fill below
  if (lda < K || lda % 8 != 0)
    return set_error(QQQ_ERR_SHAPE, "linear_static: lda=%lld must be >= K and a multiple of 8", (long long)lda);
  if (!a_fp16 || !w_packed || !s_w_fp16 || !y_fp16)
    return set_error(QQQ_ERR_NULL, "linear_static: null pointer argument");
  if (!aligned16(a_fp16) || !aligned16(w_packed) || !aligned16(y_fp16) ||
      (reinterpret_cast<uintptr_t>(s_w_fp16) & 3u))
    return set_error(QQQ_ERR_SHAPE, "linear_static: a_fp16, w_packed and y must be 16-byte aligned, s_w 4-byte");
  void* ws = nullptr;
  const int rc = static_scratch(&ws);
  if (rc != QQQ_OK) return rc;
  // The array keeps the previous call's contents.  The decode kernel (M <= 64) wants its arrival
  // counters and split-K sums zero, and a previous call of another shape may have left other
  // scratch there: clear that part.  (Every call leaves its own such part zero, so the fill is
  // what protects against the OTHER parts of an earlier layout.)
  if (M <= kSkinnyMaxM) {
    const size_t n16 = (qqq_gemm_workspace_zero_bytes(M, N, K) + 15) / 16;
    const unsigned blocks = (unsigned)((n16 + 255) / 256 < 1024 ? (n16 + 255) / 256 : 1024);
    hipLaunchKernelGGL(zero_fill_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, (uint4*)ws, n16);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(QQQ_ERR_HIP, "linear_static: fill launch: %s", hipGetErrorString(e));
  }
  return linear_common(a_fp16, lda, w_packed, nullptr, s_w_fp16, y_fp16, acc_out, M, N, K, ws, need, stream,
                       kPerChannel);
}

}  // extern "C"
