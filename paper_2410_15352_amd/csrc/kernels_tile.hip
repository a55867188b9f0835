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

// Time of a launch, in microseconds, from measurements on MI355X over 23 shapes
// (256 to 32768 rows, 512 to 5728 columns, K 512 to 5472): the tiles run in
// rounds of `slots` per CU; a 64-deep K step of a round takes `alone` with few
// workgroups on the chip and `full` with all slots taken (the copies then share
// L2), a round `ov` more (first copies and output), the launch `base`.  Over many
// rounds, or with several workgroups per CU, a CU takes the next tile when it is
// free and a part of a round costs its part; otherwise the last round lasts as long
// as a tile.  The persistent kernel deals its tiles out beforehand (always the
// latter).
struct TileCost {
  int rows, cols, slots;
  double alone, full, ov, base;
};
constexpr TileCost kCost[kTileKinds + 1] = {
    {256, 128, 1, 0.57, 0.863, 5.6, 3.0}, {128, 128, 1, 0.35, 0.485, 3.2, 3.0}, {64, 128, 2, 0.21, 0.62, 2.0, 3.0},
    {64, 64, 3, 0.14, 0.61, 1.2, 3.0},    {256, 256, 1, 1.08, 1.65, 4.0, 5.5},
};

double tile_cost(int k, int64_t M, int64_t n0, int64_t n1, int64_t K, int cus) {
  const TileCost& c = kCost[k];
  const double tiles = double(ceil_div(M, c.rows)) * double(ceil_div(n0, c.cols) + ceil_div(n1, c.cols));
  const double steps = double(ceil_div(K, 64)), per = double(cus) * c.slots, rounds = tiles / per;
  if (k < kTileKinds && rounds > (c.slots > 1 ? 1.0 : 4.0)) return c.base + rounds * (c.ov + steps * c.full);
  const double full = double(int64_t(rounds)), rest = tiles - full * per;
  const double part = rest > 0 ? c.ov + steps * (c.alone + (c.full - c.alone) * rest / per) : 0.0;
  return c.base + full * (c.ov + steps * c.full) + part;
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

// The cheapest kernel by the measured costs; a tile kernel has to win by 5%, about
// the error of the estimate.
TileKind gemm_tile_choose(int64_t M, int64_t n0, int64_t n1, int64_t K, bool persistent, int cus) {
  int best = kTileKinds;
  double t = persistent ? 0.95 * tile_cost(kTileKinds, M, n0, n1, K, cus) : HUGE_VAL;
  for (int k = 0; k < kTileKinds; ++k) {
    const double c = tile_cost(k, M, n0, n1, K, cus);
    if (c < t) {
      t = c;
      best = k;
    }
  }
  return static_cast<TileKind>(best);
}

bool gemm_tile_eligible(int64_t M, int64_t K, int64_t lda, int64_t ldb, int64_t rows_b) {
  const int64_t lim = int64_t(1) << 31;
  if (M < 1 || K < 1 || M >= lim || rows_b >= lim) return false;
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
