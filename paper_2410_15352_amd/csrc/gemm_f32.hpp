// fp32 GEMMs of the CompAct layer on the fp32 MFMA (v_mfma_f32_32x32x2_f32,
// exact fp32 products and fp32 accumulation).
//
//   C (M x N) = A (M x K) B (K x N)
//
// Operands are read as they lie in memory (or generated):
//   kKc   K-contiguous: element (row, k) at p[row * ld + k]
//   kMn   row-contiguous: element (row, k) at p[k * ld + row]
//   kPk   the projection stream with K = its rows i:    element (col j, k = i)
//   kPm   the projection stream with K = its columns j: element (row i, k = j)
// so no operand is transposed or copied first and the fp32 entry points need no
// workspace.
//
// One workgroup (4 waves) per output tile; 32-deep K steps in S LDS stages.  Memory
// operands are copied by buffer_load_dwordx4 ... lds S - 1 steps ahead, generated ones
// written to the same stages.  What bounds it: the fp32
// MFMA (256 flops per clock and CU, 157 TFLOP/s at 2.4 GHz), which shares its
// unit with the vector instructions: addresses are kept out of the K loop or
// left to the scalar unit (160 vector instructions per step made the backward of
// a 2048-token 768 -> 3072 layer take 207 us, 20 of them 154).  A 64 x 64 tile
// moves 16 KB into LDS per 1024 clocks of MFMA, a quarter of what the copies
// can do, so small tiles cost nothing and fill the chip for small layers.
//
// LDS stage layouts (kPk and kPm use kMn's):
//   kKc  [rows][32] fp32, 16-byte chunk c of row R at c ^ ((R >> 1) & 7): a
//        fragment is one ds_read_b128, lane half h of it k = 8 kk + 4 h .. + 3
//   kMn  [32][rows] fp32, chunk c of K row k at c ^ (8 ((k >> 2) & 1)) (at c
//        when there are only 32 rows, one pass of the banks): a
//        fragment element is one ds_read_b32, the two lane halves (K rows 4
//        apart) on different banks
// MFMA step (kk, s) takes k = 8 kk + s on lane half 0 and 8 kk + 4 + s on half
// 1, in both operands.
//
// Edges: reads past an operand's last element return zero (buffer range check); the
// last K step's elements past K of a kKc operand are cleared in registers (the
// row padding may hold anything).
#pragma once
#include <type_traits>

#include "gemm_bf16.hpp"
#include "gemm_w4.hpp"
#include "kernels_common.hpp"

namespace compact {

enum class OpF32 : int { kKc, kMn, kPk, kPm };

struct MatF32 {
  const float* p;   // memory operands
  int64_t ld, rows; // rows: the operand's M or N extent
  ProjDesc proj;    // generated operands
  PhiloxKey key;
  int64_t n;        // rows i of the stream
};

// mode 0: out = scale * C;  mode 1 (update): out = out - scale * C;  mode 2
// (accumulate): out = out + C.
struct JobF32 {
  MatF32 A, B;
  int64_t M, N, K;
  float* out;
  int64_t ldo;
  float scale;
  int mode;
  int tiles_n, tiles;
};

// Two products in one launch: workgroups 0 .. job[0].tiles - 1 compute job 0.
struct PairF32 {
  JobF32 job[2];
};

__device__ __forceinline__ f32x16 mfma32x32x2(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

constexpr int kF32K = 32;  // K step

// w4_rsrc for a range computed in the K loop: 32-bit comparisons only, which
// stay on the scalar unit (the fp32 MFMAs share the vector one).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t f32_rsrc(const float* base, int64_t bytes) {
  const int hi = static_cast<int>(bytes >> 32);
  const uint32_t lo = static_cast<uint32_t>(bytes);
  const uint32_t n = hi < 0 ? 0u : (hi > 0 || lo > 0x7FFFFFFFu ? 0x7FFFFFFFu : lo);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), static_cast<short>(0), static_cast<int>(n), 0x00020000);
}

// Wave arrangement of a tile: WM x WN x WK = 4 waves; a wave owns FM x FN
// fragments of 32 x 32.  WK == 1: the waves share the stages.  WK == 4: one 32 x 32
// tile, every wave takes each fourth K step with stages of its own and no barrier,
// and the four sums are added in wave order at the end.
template <int WM, int WN, int WK, int FM, int FN, int S>
struct F32Shape {
  static constexpr int kWm = WM, kWn = WN, kWk = WK, kFm = FM, kFn = FN, kS = S;
  static constexpr int kBM = 32 * WM * FM, kBN = 32 * WN * FN;
  static constexpr int kAStage = kBM * kF32K * 4, kStage = (kBM + kBN) * kF32K * 4;  // bytes
  static constexpr size_t kLds = size_t(S) * kStage * WK;
  static_assert(WM * WN * WK == 4 && (WK == 1 || (WK == 4 && FM * FN == 1)), "four waves");
};

// A tile of ROWS rows (M or N) of an operand, starting at `row0`: what a lane
// keeps over the K loop, the filling of a stage and the fragment reads.
// NW waves fill a stage together (4, or 1: each wave its own).  FR: fragments of 32
// rows per wave.
template <OpF32 OP, int ROWS, int NW, int FR>
struct OperandTile {
  static constexpr bool kMem = OP == OpF32::kKc || OP == OpF32::kMn;
  static constexpr int kBlocks = ROWS * kF32K * 4 / 1024 / NW;  // 1 KB copies per wave
  static constexpr int kThreads = 64 * NW;
  static constexpr int kCopies = kMem ? kBlocks : 0;
  static constexpr int kFrags = OP == OpF32::kKc ? 4 : FR;
  static constexpr int kSw = ROWS >= 64 ? 8 : 0;  // kMn: chunk bit flipped for half the K rows
  const MatF32& m;
  int64_t row0;
  int steps;                // K steps
  uint32_t voff[kBlocks];   // byte offsets of this lane's copies in a K step
  uint32_t foff[kFrags];    // LDS byte offsets of its fragments (kKc: per kk)
  const float* base;        // wave-uniform
  int64_t bytes;            // from base to the operand's last element

  __device__ __forceinline__ OperandTile(const MatF32& mat, int64_t r0, int64_t K, int wrow0, int tid)
      : m(mat), row0(r0), steps(static_cast<int>(ceil_div(K, kF32K))) {
    const int lane = tid & 63, wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, lh = lane >> 5;
    if constexpr (OP == OpF32::kKc) {
      base = m.p + row0 * m.ld;
      bytes = view_bytes(m.rows, K, m.ld, row0, 0, 4);
#pragma unroll
      for (int q = 0; q < kBlocks; ++q) {  // rows 8 j .. + 7, 128 bytes each
        const int j = wave * kBlocks + q;
        voff[q] = static_cast<uint32_t>((8 * j + (lane >> 3)) * m.ld * 4) + 16u * ((lane & 7) ^ (lane >> 4) ^ (4 * (j & 1)));
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        foff[kk] = static_cast<uint32_t>((wrow0 + lr) * 128) + 16u * static_cast<uint32_t>((2 * kk + lh) ^ ((lr >> 1) & 7));
    } else {
      if constexpr (kMem) {
        base = m.p + row0;
        bytes = view_bytes(K, m.rows, m.ld, 0, row0, 4);
        constexpr int cpr = ROWS / 4;  // chunks per K row
#pragma unroll
        for (int q = 0; q < kBlocks; ++q) {
          const int idx = 64 * (wave * kBlocks + q) + lane, k = idx / cpr;
          voff[q] = static_cast<uint32_t>(k * m.ld * 4) + 16u * ((idx % cpr) ^ (kSw * ((k >> 2) & 1)));
        }
      }
#pragma unroll
      for (int f = 0; f < FR; ++f) {
        const int c = wrow0 + 32 * f + lr;
        foff[f] = static_cast<uint32_t>(4 * lh * ROWS * 4 + (((c >> 2) ^ (kSw * lh)) * 16) + (c & 3) * 4);
      }
    }
  }

  // This wave's share of K step kt into the stage at LDS byte address `dst`.  A
  // copy may read past K or past the operand's last row (the next row's
  // elements, or zero past its end): past K the fragments are cleared (kKc) or
  // the K rows lie past the end, and rows past the last feed only outputs that
  // are not stored.  Steps past the last one copy zeros.
  __device__ __forceinline__ void stage(int kt, uint32_t dst, int tid) const {
    const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    if constexpr (NW == 1) tid &= 63;
    const int64_t k0 = static_cast<int64_t>(kt) * kF32K;
    if constexpr (kMem) {
      const int64_t adv = OP == OpF32::kKc ? k0 : k0 * m.ld;
      const __amdgpu_buffer_rsrc_t r = f32_rsrc(base + adv, kt < steps ? bytes - adv * 4 : 0);
#pragma unroll
      for (int q = 0; q < kBlocks; ++q)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            r, reinterpret_cast<w4_lds_void*>(static_cast<uintptr_t>(dst + (wave * kBlocks + q) * 1024u)), 16,
            static_cast<int>(voff[q]), 0, 0, 0);
    } else if constexpr (OP == OpF32::kPk) {
      // quad of K rows k0 + 4 kq .. + 3 of column row0 + c
#pragma unroll 1
      for (int u = tid; u < ROWS * (kF32K / 4); u += kThreads) {
        const int c = u % ROWS, kq = u / ROWS;
        float g[4];
        quad(k0 + 4 * kq, row0 + c, g);
        const uint32_t a = dst + static_cast<uint32_t>(4 * kq * ROWS * 4 + (((c >> 2) ^ (kSw * (kq & 1))) * 16) + (c & 3) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<__attribute__((address_space(3))) float*>(static_cast<uintptr_t>(a + e * ROWS * 4)) = g[e];
      }
    } else {
      // quad of rows row0 + 4 rq .. + 3 at k = k0 + kk
#pragma unroll 1
      for (int u = tid; u < (ROWS / 4) * kF32K; u += kThreads) {
        const int rq = u % (ROWS / 4), kk = u / (ROWS / 4);
        float g[4];
        quad(row0 + 4 * rq, k0 + kk, g);
        const uint32_t a = dst + static_cast<uint32_t>(kk * ROWS * 4 + ((rq ^ (kSw * ((kk >> 2) & 1))) * 16));
        const u32x4 v = {__float_as_uint(g[0]), __float_as_uint(g[1]), __float_as_uint(g[2]), __float_as_uint(g[3])};
        *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(static_cast<uintptr_t>(a)) = v;
      }
    }
  }

  // Unscaled stream elements (i0 .. i0 + 3, j), zero outside n x r.
  __device__ __forceinline__ void quad(int64_t i0, int64_t j, float (&g)[4]) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = 0.0f;
    if (j >= m.proj.r || i0 >= m.n) return;
    proj_quad(m.proj, m.key, i0, j, g);
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = i0 + e < m.n ? g[e] : 0.0f;
  }

  // The four values s = 0 .. 3 of MFMA steps (kk, s) of fragment f of the wave.
  __device__ __forceinline__ void frag(uint32_t stage, int f, int kk, float (&v)[4]) const {
    if constexpr (OP == OpF32::kKc) {
      const u32x4 w = *reinterpret_cast<const w4_lds_u32x4*>(static_cast<uintptr_t>(stage + foff[kk] + f * 4096));
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = __uint_as_float(w[s]);
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s)
        v[s] = *reinterpret_cast<const __attribute__((address_space(3))) float*>(
            static_cast<uintptr_t>(stage + foff[f] + (8 * kk + s) * ROWS * 4));
    }
  }
};

template <OpF32 OA, OpF32 OB, class Sh>
__device__ __forceinline__ void gemm_f32_tile(const JobF32& g, int tile) {
  constexpr int FM = Sh::kFm, FN = Sh::kFn, WK = Sh::kWk, S = Sh::kS, BM = Sh::kBM, BN = Sh::kBN;
  using TA = OperandTile<OA, BM, 4 / WK, FM>;
  using TB = OperandTile<OB, BN, 4 / WK, FN>;
  constexpr int CPW = TA::kCopies + TB::kCopies;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave % WK, wm = wave / WK / Sh::kWn, wn = wave / WK % Sh::kWn;
  const int64_t row0 = static_cast<int64_t>(tile / g.tiles_n) * BM, col0 = static_cast<int64_t>(tile % g.tiles_n) * BN;
  const uint32_t lbase = __builtin_amdgcn_groupstaticsize() + (WK > 1 ? wk * S * Sh::kStage : 0);
  const TA ta(g.A, row0, g.K, wm * FM * 32, tid);
  const TB tb(g.B, col0, g.K, wn * FN * 32, tid);
  auto stage = [&](int kt, int st) {
    ta.stage(kt, lbase + st * Sh::kStage, tid);
    tb.stage(kt, lbase + st * Sh::kStage + Sh::kAStage, tid);
  };
  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
#pragma unroll
  for (int s = 0; s < S - 1; ++s) stage(wk + s * WK, s);
  // The MFMAs of the stage at LDS address sa; `edge`: the step holds k >= K.
  auto compute = [&](uint32_t sa, auto edge) {
    float a[2][FM][4], b[2][FN][4];
    auto read = [&](int q) {
#pragma unroll
      for (int i = 0; i < FM; ++i) ta.frag(sa, i, q, a[q & 1][i]);
#pragma unroll
      for (int j = 0; j < FN; ++j) tb.frag(sa + Sh::kAStage, j, q, b[q & 1][j]);
    };
    read(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // the next fragments are read beside this part's MFMAs (left to itself the
      // compiler reads them right before their use and waits)
      if (q + 1 < 4) read(q + 1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (decltype(edge)::value) {
        const int left = static_cast<int>(g.K % kF32K) - 8 * q - 4 * (lane >> 5);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          if constexpr (OA == OpF32::kKc)
#pragma unroll
            for (int i = 0; i < FM; ++i) a[q & 1][i][s] = s < left ? a[q & 1][i][s] : 0.0f;
          if constexpr (OB == OpF32::kKc)
#pragma unroll
            for (int j = 0; j < FN; ++j) b[q & 1][j][s] = s < left ? b[q & 1][j][s] : 0.0f;
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) acc[i][j] = mfma32x32x2(a[q & 1][i][s], b[q & 1][j][s], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // this wave's part of a step is in LDS (the copies of the S - 2 steps after it
  // may be in flight) and its reads of the stage that is filled next have
  // returned; where the waves share the stages, the barrier says so for all
  auto arrive = [] {
    if constexpr (WK == 1)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((S - 2) * CPW) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * CPW) : "memory");
  };
  const int whole = static_cast<int>(g.K / kF32K);  // steps without k >= K
  int st = 0, kt = wk;
  for (; kt < whole; kt += WK) {
    arrive();
    stage(kt + (S - 1) * WK, st == 0 ? S - 1 : st - 1);
    compute(lbase + st * Sh::kStage, std::false_type{});
    st = st == S - 1 ? 0 : st + 1;
  }
  if (kt == whole && g.K % kF32K != 0) {  // (one wave's, with WK == 4)
    arrive();
    compute(lbase + st * Sh::kStage, std::true_type{});
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy may still be writing LDS when the workgroup ends
  // Modes 1 and 2 read all their elements of `out` before the first store: a load
  // behind a store that may alias it waits for a round trip to memory, 32 of them in
  // the update (768 x 3072, r = 384: 53 -> 46 us).
  auto inside = [&](int64_t gr, int64_t gc) { return gr < g.M && gc < g.N; };
  auto load = [&](int64_t gr, int64_t gc) { return inside(gr, gc) ? g.out[gr * g.ldo + gc] : 0.0f; };
  auto put = [&](int64_t gr, int64_t gc, float old, float v) {
    if (!inside(gr, gc)) return;
    const float d = g.scale * v;
    g.out[gr * g.ldo + gc] = g.mode == 0 ? d : g.mode == 2 ? old + v : old - d;
  };
  if constexpr (WK == 1) {
    const int64_t r0 = row0 + wm * FM * 32, c0 = col0 + wn * FN * 32;
    float old[FM * FN * 16] = {};
    int e = 0;
    if (g.mode != 0) for_each_acc(acc, lane, [&](int row, int col, float) { old[e++] = load(r0 + row, c0 + col); });
    e = 0;
    for_each_acc(acc, lane, [&](int row, int col, float v) { put(r0 + row, c0 + col, old[e++], v); });
  } else {
    // the four waves' sums of the 32 x 32 tile, added in wave order
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    float* part = reinterpret_cast<float*>(lds);
    __syncthreads();  // every read of the stages is done
    for_each_acc(acc, lane, [&](int row, int col, float v) { part[wave * 1024 + row * 32 + col] = v; });
    __syncthreads();
    float old[4] = {};
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (g.mode != 0) old[u] = load(row0 + ((tid + 256 * u) >> 5), col0 + (tid & 31));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = tid + 256 * u;
      put(row0 + (e >> 5), col0 + (e & 31), old[u], ((part[e] + part[1024 + e]) + part[2048 + e]) + part[3072 + e]);
    }
  }
}

// Large products: 64 x 64 tiles.  z takes 128 x 32 and the update 32 x 128,
// 256 or 384 (launch_update_f32), since a workgroup generates its tile of P itself (about
// 2000 clocks per quad of normals and wave, on the unit the MFMAs need): a taller
// tile of z, or a wider one of W, shares it among more MFMAs.  Other small products
// (64 x 64 tiles for less than three quarters of the CUs): 32 x 32 tiles whose
// waves split K, so that four times the CUs work, a wave has a quarter of the K
// steps in sequence and none waits for a barrier (256 x 256, K 512: 14 -> 6.5 us;
// 32 x 1024, K 2048: 36 -> 15 us).
using F32Big = F32Shape<2, 2, 1, 1, 1, 3>;
using F32Tall = F32Shape<4, 1, 1, 1, 1, 2>;
template <int FN>
using F32Update = F32Shape<1, 4, 1, 1, FN, 2>;
using F32Small = F32Shape<1, 1, 4, 1, 1, 3>;

// Workgroups of one launch: job 1's tiles first, then job 0's; each job's tiles keep
// the XCD-contiguous order.  (Job 1 is z in the forward, whose tiles generate P and
// take longer; in the backward it is G^ over K = tokens, the shorter job where tokens <
// m, so the longer tiles start last there: 2048 tokens, 768 -> 3072, r = 384: 672 tiles
// on 256 CUs take 157 us for 94 us of MFMA.)
__device__ __forceinline__ bool f32_pick(const PairF32& p, int& tile) {
  const uint32_t t1 = static_cast<uint32_t>(p.job[1].tiles), b = blockIdx.x;
  const bool second = b < t1;
  tile = static_cast<int>(second ? xcd_remap(b, t1) : xcd_remap(b - t1, gridDim.x - t1));
  return second;
}

// y = x W (job 0) and z = x P (job 1).
template <bool SMALL>
__global__ __launch_bounds__(256, 2) void k_fwd_f32(PairF32 p) {
  int tile;
  if (f32_pick(p, tile))
    gemm_f32_tile<OpF32::kKc, OpF32::kPk, std::conditional_t<SMALL, F32Small, F32Tall>>(p.job[1], tile);
  else
    gemm_f32_tile<OpF32::kKc, OpF32::kMn, std::conditional_t<SMALL, F32Small, F32Big>>(p.job[0], tile);
}

// dx = dL/do W^T (job 0) and G^ = z^T dL/do (job 1); either may have no tiles.
template <bool SMALL>
__global__ __launch_bounds__(256, 2) void k_bwd_f32(PairF32 p) {
  using Sh = std::conditional_t<SMALL, F32Small, F32Big>;
  int tile;
  if (f32_pick(p, tile))
    gemm_f32_tile<OpF32::kMn, OpF32::kMn, Sh>(p.job[1], tile);
  else
    gemm_f32_tile<OpF32::kKc, OpF32::kKc, Sh>(p.job[0], tile);
}

// W <- W - coef P N (job 0).
template <int FN>
__global__ __launch_bounds__(256, 2) void k_dec_f32(PairF32 p) {
  int tile;
  f32_pick(p, tile);
  gemm_f32_tile<OpF32::kPm, OpF32::kMn, F32Update<FN>>(p.job[0], tile);
}

}  // namespace compact
