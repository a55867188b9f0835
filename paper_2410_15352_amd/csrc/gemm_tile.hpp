// bf16 GEMM C = A B^T for calls that leave the persistent 256 x 256 kernel
// (gemm_w4.hpp) short of tiles: A [M][K] and B [N][K] both row-major with K
// contiguous, C bf16, one workgroup per BM x BN output tile.
//
// Pipeline: 64-deep K steps in S LDS stages, filled by buffer_load_dwordx4 ...
// lds (8 rows x 128 bytes per wave instruction, whole cache lines, so row-major
// operands need no K-tiled copy).  A step is two halves of two 16-deep MFMA
// steps:
//   first half:  its MFMAs; between them the fragment reads of the second half
//                and the second half of the copies of step kt + S - 1
//   wait until this wave's copies of step kt + 1 have landed; barrier (every
//   wave's copies landed, every read of step kt's stage done)
//   second half: its MFMAs; between them the fragment reads of step kt + 1's
//                first half and the first half of the copies of step kt + S
//                into the stage of step kt
// The source order is the issue order (the unit is compiled with the machine
// scheduler off): a wave that issues its copies in one burst, or waits for its
// fragments before each MFMA, leaves its SIMD idle, because only one or two
// waves share it (a 128 x 128 tile alone on the chip: 0.57 us per step with
// bursts).
//
// What bounds it: with few tiles, the K step of one workgroup (256 x 128: 0.57 us
// per 64-deep step alone on the chip, 128 x 128: 0.35, 64 x 64: 0.235; the MFMAs
// alone 0.43, 0.21, 0.05); with every CU busy, the operand bytes through L2
// (about 13 TB/s over the chip).  The persistent kernel moves fewer bytes per
// flop, so it stays the better one when its tiles fill the CUs; below that
// (M x N, K; persistent -> tile kernel, MI355X): 8192 x 1024, 3072: 71 -> 50 us;
// 8192 x 512, 2752: 55 -> 26.5 us; 4096 x 1024, 3072: 62 -> 29 us; 1000 x 512,
// 2752: 52 -> 13.1 us; 1024 x 1920, 512: 18.3 -> 6.2 us.
//
// LDS: stage s holds A [BM][64] and B [BN][64] at s * (BM + BN) * 128 bytes.
// Logical 16-byte chunk c of row R sits at c ^ ((R >> 1) & 7): the 16 rows that
// 16 lanes of a ds_read_b128 read fill 16 distinct 16-byte bank groups.
//
// Every output element is one fp32 accumulator that takes the 32x32x16 MFMAs of
// its K steps in order from zero, as in the other bf16 GEMMs of this library, so
// the results are bitwise theirs.
//
// Edges: rows past the matrix and chunks at k >= K read as zero (buffer range
// check); with K % 8 != 0 the chunk that holds element K - 1 is read whole and
// its elements past K are cleared in registers, in both operands.
#pragma once
#include <type_traits>

#include "gemm_bf16.hpp"
#include "gemm_w4.hpp"

namespace compact {

// Output column tile ct < seg[0].tiles writes columns BN ct .. of seg[0].C from
// B rows BN ct .., the others columns BN (ct - seg[0].tiles) .. of seg[1].C
// from B rows b_row1 + BN (ct - seg[0].tiles) ...
struct TGemm {
  const uint16_t* A;  // [M][lda]
  const uint16_t* B;  // [rows_b][ldb]
  int lda, M, K;
  int ldb, rows_b, b_row1;
  W4Seg seg[2];       // seg[1].tiles == 0 when unused
  int tiles_n, tiles;
  int band_rows;      // rows of tiles per band of the walk order
};

template <int BM, int BN, int WGM, int WGN, int S>
struct TileShape {
  static constexpr int kThreads = WGM * WGN * kWave;
  static constexpr int kFm = BM / WGM / 32, kFn = BN / WGN / 32;
  static constexpr int kStage = (BM + BN) * 128;               // bytes
  static constexpr int kCopies = (BM + BN) / 8 / (WGM * WGN);  // per wave and step
  static constexpr int kStore = BM * BN * 2;                   // the bf16 tile staged for its stores
  static constexpr size_t kLds = size_t(S) * kStage > size_t(kStore) ? size_t(S) * kStage : size_t(kStore);
  static_assert((BM + BN) / 8 % (WGM * WGN) == 0, "copies split evenly over the waves");
};

// s_waitcnt vmcnt(N) lgkmcnt(0), s_barrier, with the accumulators and the
// fragments of the following MFMAs passed through, so that MFMAs stay on their
// side of it.
template <int N, int FM, int FN>
__device__ __forceinline__ void tile_wait_barrier(u32x4 (&fa)[2][FM], u32x4 (&fb)[2][FN], f32x16 (&acc)[FM][FN]) {
  static_assert(N >= 0 && N < 64, "vmcnt immediate");
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(acc[i][j]));
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
#pragma unroll
  for (int k = 0; k < 2; ++k) {
#pragma unroll
    for (int i = 0; i < FM; ++i) asm volatile("" : "+v"(fa[k][i]));
#pragma unroll
    for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(fb[k][j]));
  }
}

template <int BM, int BN, int WGM, int WGN, int S, bool KMASK>
__device__ __forceinline__ void gemm_tile(const TGemm& g) {
  using T = TileShape<BM, BN, WGM, WGN, S>;
  constexpr int FM = T::kFm, FN = T::kFn, CPW = T::kCopies;
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  // walk order: bands of band_rows rows of tiles, column by column inside a
  // band; an XCD's workgroups take one contiguous stretch (operand reuse in L2)
  const int p = static_cast<int>(xcd_remap(blockIdx.x, gridDim.x));
  const int rows_total = g.tiles / g.tiles_n, per_band = g.band_rows * g.tiles_n;
  const int band = p / per_band, r0 = band * g.band_rows, within = p - band * per_band;
  const int rows_in = min(g.band_rows, rows_total - r0);
  const int ct = within / rows_in, rt = r0 + within - ct * rows_in;
  const int sg = ct >= g.seg[0].tiles ? 1 : 0;
  const int cts = sg ? ct - g.seg[0].tiles : ct;
  const int64_t row0 = static_cast<int64_t>(rt) * BM;
  const int64_t brow0 = static_cast<int64_t>(sg ? g.b_row1 : 0) + static_cast<int64_t>(cts) * BN;
  const __amdgpu_buffer_rsrc_t ra = w4_rsrc(g.A + row0 * g.lda, view_bytes(g.M, g.K, g.lda, row0, 0, 2));
  const __amdgpu_buffer_rsrc_t rb = w4_rsrc(g.B + brow0 * g.ldb, view_bytes(g.rows_b, g.K, g.ldb, brow0, 0, 2));

  // copy block j (8 rows x 128 bytes) of the stage's BM + BN rows: blocks
  // j < BM / 8 are A.  Lane L lands at row 8 j + L / 8, physical chunk L % 8,
  // so it fetches logical chunk (L % 8) ^ (L / 16) ^ 4 (j % 2).
  const int ch0 = (lane & 7) ^ (lane >> 4);
  const uint32_t lbase = __builtin_amdgcn_groupstaticsize();
  const int nk = static_cast<int>(ceil_div(g.K, 64));
  uint32_t voff[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    const int j = wave * CPW + c;  // wave-uniform
    const int jr = j < BM / 8 ? j : j - BM / 8;
    voff[c] = static_cast<uint32_t>((8 * jr + (lane >> 3)) * (j < BM / 8 ? g.lda : g.ldb) * 2 + 16 * (ch0 ^ (4 * (j & 1))));
  }
  // copy c (0 .. CPW - 1) of this wave for K step kt into stage st; past the
  // last K step every lane is out of range and the copy writes zeros
  auto copy = [&](int kt, int st, int c) {
    const int j = wave * CPW + c;
    // bit 31 set where the lane's chunk starts at k >= K
    const uint32_t oob = ~static_cast<uint32_t>(kt * 64 + 8 * ((j & 1) ? ch0 ^ 4 : ch0) - g.K) & kW4Oob;
    const uint32_t vo = (voff[c] + 128u * static_cast<uint32_t>(kt)) | oob;
    const uint32_t dst = lbase + static_cast<uint32_t>(st) * T::kStage + static_cast<uint32_t>(j) * 1024u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(j < BM / 8 ? ra : rb,
                                             reinterpret_cast<w4_lds_void*>(static_cast<uintptr_t>(dst)), 16,
                                             static_cast<int>(vo), 0, 0, 0);
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
#pragma unroll
  for (int s = 0; s < S - 1; ++s)
#pragma unroll
    for (int c = 0; c < CPW; ++c) copy(s, s, c);
  // fragment of row lr, 16-deep step kk: chunk 2 kk + lh at byte
  // 128 lr + 16 ((2 kk + lh) ^ ((lr >> 1) & 7)) (every fragment starts at a
  // multiple of 16 rows)
  const int lr = lane & 31, lh = lane >> 5;
  const uint32_t c0 = 16u * (static_cast<uint32_t>(lh) ^ static_cast<uint32_t>((lr >> 1) & 7));
  const uint32_t fa0 = lbase + static_cast<uint32_t>((wm * FM * 32 + lr) * 128);
  const uint32_t fb0 = lbase + static_cast<uint32_t>(BM * 128 + (wn * FN * 32 + lr) * 128);
  u32x4 fa[2][2][FM], fb[2][2][FN];  // [half of the step][kk][fragment]
  constexpr int NM = 2 * FM * FN, NR = 2 * (FM + FN), HC = CPW / 2;  // per half: MFMAs, fragment reads, copies
  // read r (0 .. NR - 1) of half hf of the stage at byte offset so
  auto read = [&](uint32_t so, int hf, int r) {
    const int k2 = r / (FM + FN), f = r % (FM + FN);
    const uint32_t co = so + (c0 ^ (32u * static_cast<uint32_t>(2 * hf + k2)));
    if (f < FM)
      fa[hf][k2][f] = *reinterpret_cast<const w4_lds_u32x4*>(static_cast<uintptr_t>(fa0 + co + f * 4096));
    else
      fb[hf][k2][f - FM] = *reinterpret_cast<const w4_lds_u32x4*>(static_cast<uintptr_t>(fb0 + co + (f - FM) * 4096));
  };
  // The MFMAs of half hf of K step kt, in issue order with the reads of the
  // other half (stage at byte offset so) and with copies c_begin .. of K step
  // kc into stage sc between them.
  auto half = [&](auto hf_, int kt, uint32_t so, int kc, int sc) {
    constexpr int hf = decltype(hf_)::value, c_begin = hf ? 0 : HC, nc = hf ? HC : CPW - HC;
    if constexpr (KMASK) {
      if (kt == nk - 1) {
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
          if ((((g.K - 1) & 63) >> 4) == 2 * hf + k2) {  // the 16 k that hold element K - 1
            const int keep = lh == ((((g.K - 1) & 63) >> 3) & 1) ? (g.K & 7) : 8;
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[hf][k2][i] = keep_first(fa[hf][k2][i], keep);
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[hf][k2][j] = keep_first(fb[hf][k2][j], keep);
          }
      }
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int k2 = m / (FM * FN), i = (m / FN) % FM, j = m % FN;
      acc[i][j] = mfma32x32x16(fa[hf][k2][i], fb[hf][k2][j], acc[i][j]);
      // the reads go out first (two per MFMA at most), the copies evenly
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (r * NM / (NR > NM ? NR : NM) == m) read(so, 1 - hf, r);
#pragma unroll
      for (int c = 0; c < nc; ++c)
        if (c * NM / nc == m) copy(kc, sc, c_begin + c);
    }
  };
  // step 0 landed (the copies of steps 1 .. S - 2 may still be in flight)
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((S - 2) * CPW) : "memory");
#pragma unroll
  for (int r = 0; r < NR; ++r) read(0, 0, r);
#pragma unroll
  for (int c = 0; c < HC; ++c) copy(S - 1, S - 1, c);
  int st = 0;
  for (int kt = 0; kt < nk; ++kt) {
    const int sp = st == 0 ? S - 1 : st - 1, sn = st == S - 1 ? 0 : st + 1;  // stages of steps kt - 1 and kt + 1
    half(std::integral_constant<int, 0>{}, kt, static_cast<uint32_t>(st) * T::kStage, kt + S - 1, sp);
    tile_wait_barrier<(S - 2) * CPW, FM, FN>(fa[1], fb[1], acc);
    half(std::integral_constant<int, 1>{}, kt, static_cast<uint32_t>(sn) * T::kStage, kt + S, st);
    st = sn;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy may still be writing LDS
  __syncthreads();  // every read of the stages is done: the tile is staged in them for its stores
  const W4Seg& sgm = g.seg[sg];
  store_tile_bf16_lds<BM, BN, WGM, WGN>(acc, lds, sgm.C, sgm.ldc, g.M, sgm.cols, row0, static_cast<int64_t>(cts) * BN,
                                        1.0f);
}

// The tile shapes that are built (kernels_tile.hip), and the persistent
// 256 x 256 kernel as the fifth choice.
enum class TileKind : int { k256x128 = 0, k128x128 = 1, k64x128 = 2, k64x64 = 3, kPersistent = 4 };
constexpr int kTileKinds = 4;

// The kernel that should compute an M x (n0 + n1) product over K (n1 = 0: one
// output segment; each segment starts on a tile of its own); `persistent`: the
// persistent kernel takes the shape, `copies`: after a K-tiled copy of B that the
// tile kernels do without.
TileKind gemm_tile_choose(int64_t M, int64_t n0, int64_t n1, int64_t K, bool persistent, bool copies, int cus);

// True when the tile kernels take this product: 32-bit buffer offsets inside a tile,
// and output leading dimensions (ldc1 = 0: one segment) that W4Seg's int holds.
bool gemm_tile_eligible(int64_t M, int64_t K, int64_t lda, int64_t ldb, int64_t rows_b, int64_t ldc0, int64_t ldc1);

// Launches a tile kernel (kind != kPersistent); tiles_n, tiles, band_rows and
// the segments' tiles are filled in here.
hipError_t gemm_tile_launch(const TGemm& g, TileKind kind, hipStream_t stream);

// Compute units of the current device (queried once per device).
hipError_t device_cus(int* cus);

}  // namespace compact
