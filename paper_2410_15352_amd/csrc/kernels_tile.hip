// The one-workgroup-per-tile bf16 GEMM (gemm_tile.hpp), the rule that picks its
// tile shape and its launcher.  Built with the machine scheduler off, like
// kernels_w4.hip: the K steps are written in issue order.
#include "gemm_tile.hpp"

#include <atomic>
#include <cmath>

namespace compact {

template <int BM, int BN, int WGM, int WGN, int S, bool KMASK>
__global__ __launch_bounds__(WGM* WGN* kWave, 2) void k_gemm_tile(TGemm g) {
  gemm_tile<BM, BN, WGM, WGN, S, KMASK>(g);
}

namespace {

constexpr int kMaxDevices = 64;
std::atomic<bool> g_lds_set[kMaxDevices][2 * kTileKinds];
std::atomic<int> g_cus[kMaxDevices];

struct Variant {
  const void* fn[2];  // K % 8 == 0, K % 8 != 0
  int rows, cols, threads;
  size_t lds;
};

template <int BM, int BN, int WGM, int WGN, int S>
Variant variant() {
  using T = TileShape<BM, BN, WGM, WGN, S>;
  return Variant{{reinterpret_cast<const void*>(k_gemm_tile<BM, BN, WGM, WGN, S, false>),
                  reinterpret_cast<const void*>(k_gemm_tile<BM, BN, WGM, WGN, S, true>)},
                 BM, BN, T::kThreads, T::kLds};
}

// Eight waves (two per SIMD) for all but the smallest tile, which has four: what
// bounds a small tile is the issue of its copies, reads and MFMAs, and more waves
// issue more (64 x 64 with two waves: 15.1 us for 1000 x 512 over K 2752, with four
// 13.1).  LDS for one, one, two and three workgroups per CU.
const Variant& variant_of(int kind) {
  static const Variant v[kTileKinds] = {variant<256, 128, 4, 2, 3>(), variant<128, 128, 2, 4, 4>(),
                                        variant<64, 128, 2, 4, 3>(), variant<64, 64, 2, 2, 3>()};
  return v[kind];
}

// Time of a launch, in microseconds, fitted to measurements on MI355X (67 products
// of 200 to 65000 rows, 266 to 5461 columns, K 320 to 32000; a kernel's error is 8 to
// 10% rms).  On 90 other products of these ranges the choice, with the margin below,
// was on average 0.2% from the best of the five, at most 14% (12000 x 700 + 37, K 300:
// 22.9 us, the 64 x 64 tiles 20.2) and at most 1.3% slower than the persistent kernel,
// which is what two runs differ by.  The tiles run in rounds of `slots` per CU,
// a last round of c tiles per CU lasting as long as its fullest CU: a 64-deep K step
// with c tiles on a CU takes alone[c - 1] with few CUs at work and full[c - 1] with
// all (the copies then share L2), a round `ov` more (first copies and output), the
// launch `base`.  The persistent kernel's dL/dx first copies its N x K operand
// (stage_cost); the forward stages its operand for either.
// Counting parts of a round as their part took 5 to 15% longer than the persistent
// kernel just past a whole round (26310 x 1254, K 1816: 168 us against 135).
struct TileCost {
  int rows, cols, slots;
  double base, ov, alone[3], full[3];
};
constexpr TileCost kCost[kTileKinds + 1] = {
    {256, 128, 1, 0.0, 6.17, {0.519}, {1.007}},
    {128, 128, 1, 1.24, 2.96, {0.340}, {0.603}},
    {64, 128, 2, 2.19, 1.93, {0.229, 0.777}, {0.463, 0.709}},
    {64, 64, 3, 3.53, 0.57, {0.198, 0.364, 1.071}, {0.258, 0.545, 0.703}},
    {256, 256, 1, 8.1, 4.53, {0.931}, {1.687}},
};

double stage_cost(int64_t N, int64_t K) { return 1.65 + 1.58e-6 * double(N) * double(K); }

double tile_cost(int k, int64_t M, int64_t n0, int64_t n1, int64_t K, int cus) {
  const TileCost& c = kCost[k];
  const int64_t tiles = ceil_div(M, c.rows) * (ceil_div(n0, c.cols) + ceil_div(n1, c.cols)), per = int64_t(cus) * c.slots;
  const double steps = double(ceil_div(K, 64));
  const int64_t rounds = tiles / per, rest = tiles - rounds * per;
  double t = c.base + double(rounds) * (c.ov + steps * c.full[c.slots - 1]);
  if (rest > 0) {
    const int64_t on = ceil_div(rest, cus);  // tiles on the fullest CU
    const double busy = double(rest) / double(on * cus);
    t += c.ov + steps * (c.alone[on - 1] + (c.full[on - 1] - c.alone[on - 1]) * busy);
  }
  return t;
}

}  // namespace

hipError_t device_cus(int* cus) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  int n = g_cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    n = n > 0 ? n : 1;
    g_cus[dev].store(n, std::memory_order_relaxed);
  }
  *cus = n;
  return hipSuccess;
}

// The cheapest kernel by the measured costs; a tile kernel has to win by 6%, most
// of the estimate's error (without the margin 24040 x 317, K 1384, went to one that won
// by 5% on paper: 44.6 us against 41.1).  Where the persistent kernel does not
// take the shape (K < 320, mostly), the other choice is the eight-wave kernel of 256 x
// 256 tiles: the tile kernels are faster until its tiles fill the CUs (K 300, 700 + 150
// columns: 5000 rows, 80 tiles, 22 -> 15 us; 12000 rows, 188 tiles, 25 us either way;
// 30000 rows, 472 tiles, 43 against 46 us; K 256, 3072 + 64 columns, 65536 rows: 207
// against 257 us).
TileKind gemm_tile_choose(int64_t M, int64_t n0, int64_t n1, int64_t K, bool persistent, bool copies, int cus) {
  if (!persistent && 10 * ceil_div(M, 256) * (ceil_div(n0, 256) + ceil_div(n1, 256)) > 7 * int64_t(cus))
    return TileKind::kPersistent;
  int best = kTileKinds;
  double t = HUGE_VAL;
  if (persistent) t = 0.94 * (tile_cost(kTileKinds, M, n0, n1, K, cus) + (copies ? stage_cost(n0, K) : 0.0));
  for (int k = 0; k < kTileKinds; ++k) {
    const double c = tile_cost(k, M, n0, n1, K, cus);
    if (c < t) {
      t = c;
      best = k;
    }
  }
  return static_cast<TileKind>(best);
}

bool gemm_tile_eligible(int64_t M, int64_t K, int64_t lda, int64_t ldb, int64_t rows_b, int64_t ldc0, int64_t ldc1) {
  const int64_t lim = int64_t(1) << 31;
  if (M < 1 || K < 1 || M >= lim || rows_b >= lim || ldc0 >= lim || ldc1 >= lim) return false;
  if (lda % 8 != 0 || ldb % 8 != 0 || lda < K || ldb < K) return false;
  // at most 256 rows of an operand per tile, and K
  return (256 * lda + K + 512) * 2 < lim && (256 * ldb + K + 512) * 2 < lim;
}

hipError_t gemm_tile_launch(const TGemm& g0, TileKind kind, hipStream_t stream) {
  const int k = static_cast<int>(kind), mask = g0.K % 8 != 0 ? 1 : 0;
  if (k < 0 || k >= kTileKinds) return hipErrorInvalidValue;
  const Variant& v = variant_of(k);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (!g_lds_set[dev][2 * k + mask].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute(v.fn[mask], hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(v.lds));
    if (e != hipSuccess) return e;
    g_lds_set[dev][2 * k + mask].store(true, std::memory_order_release);
  }
  TGemm g = g0;
  for (int s = 0; s < 2; ++s)
    g.seg[s].tiles = g.seg[s].cols > 0 ? static_cast<int>(ceil_div(g.seg[s].cols, v.cols)) : 0;
  g.tiles_n = g.seg[0].tiles + g.seg[1].tiles;
  const int64_t rows = ceil_div(g.M, v.rows), tiles = rows * g.tiles_n;
  if (tiles <= 0) return hipSuccess;
  if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
  g.tiles = static_cast<int>(tiles);
  g.band_rows = static_cast<int>(rows < 4 ? rows : 4);
  void* args[] = {&g};
  e = hipLaunchKernel(v.fn[mask], dim3(static_cast<uint32_t>(tiles)), dim3(v.threads), args, v.lds, stream);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace compact
