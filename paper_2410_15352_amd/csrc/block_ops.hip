// The element-wise and row-wise parts of the LLaMA block and model around the
// CompAct layers (paper_2410_15352_amd/block.py), bf16 in and out, fp32 inside:
//
//   RMSNorm, alone or with the residual add before it, forward and backward
//   SwiGLU (silu(gate) * up) forward and backward
//   the mean cross-entropy of bf16 logits, forward and backward
//
// Every one is bound by HBM: each input is read once and each output written
// once, 16 bytes per lane, and sums over rows are formed in a fixed order
// (deterministic).  As chains of torch kernels (conversions to fp32, squares,
// products, slices, zero-filled gradients of slices) they moved 3 to 8 times the
// bytes.  LLaMA-350M widths, 8192 tokens, MI355X: RMSNorm with the residual forward
// 12 us, backward 16 + 5 us, SwiGLU 33 us (5.5 TB/s) and 44 us (6.1 TB/s), the
// gradients of q, k, v joined 16 us; the block's forward and backward 1825 -> 1094
// us.  Wider norms (forward and backward together, 65536 rows): d = 1024 131 us, 2048
// 249 (5.4 TB/s of the five tensors moved), 2056 321 (4.2), 4096 517 (5.2), 12, 12, 10
// and 12 times the torch expressions' rate; from 2056 on the backward has one wave per
// SIMD (365 registers).
// Cross-entropy over 32000 logits: 108 us forward alone (4.9 TB/s; one
// chunk at a time 141) and 140 us behind the GEMM that writes the logits (148),
// backward 187 us (5.6 TB/s), against 1.9 ms for both.
#include <hip/hip_runtime.h>

#include "block_ops.hpp"
#include "common.hpp"

namespace compact {
namespace {

constexpr int64_t kMaxBlocks = (int64_t(1) << 24) - 1;  // of 256 threads: a launch has under 2^32 threads
constexpr float kLog2e = 1.44269504088896340736f;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
  return v;
}

__device__ __forceinline__ void unpack8(const u32x4& w, float (&v)[8]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[2 * k] = __uint_as_float(w[k] << 16);
    v[2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ u32x4 pack8(const float (&v)[8]) {
  u32x4 w;
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = pack_bf16x2(v[2 * k], v[2 * k + 1]);
  return w;
}

// ------------------------------- RMSNorm -----------------------------------
// One wave per row of d = 8 dq elements, held in registers: NC 16-byte chunks per
// lane (dq <= 64 NC).
template <int NC, bool ADD>
__global__ __launch_bounds__(256) void k_rmsnorm_fwd(RmsNormArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= a.rows) return;
  const int dq = a.d / 8;
  const u32x4* xr = reinterpret_cast<const u32x4*>(a.x) + row * dq;
  float v[NC][8];
  float ss = 0.0f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int q = lane + 64 * c;
    u32x4 w = {0u, 0u, 0u, 0u};
    if (q < dq) w = xr[q];
    if constexpr (ADD) {
      if (q < dq) {
        float x[8], o[8];
        unpack8(w, x);
        unpack8(reinterpret_cast<const u32x4*>(a.add)[row * dq + q], o);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] += o[e];
        w = pack8(x);  // the residual stream is bf16: the norm sees the rounded sum
        reinterpret_cast<u32x4*>(a.sum)[row * dq + q] = w;
      }
    }
    unpack8(w, v[c]);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[c][e] * v[c][e];
  }
  ss = wave_sum(ss);
  const float rstd = 1.0f / __builtin_sqrtf(ss / static_cast<float>(a.d) + a.eps);
  if (lane == 0) a.rstd[row] = rstd;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int q = lane + 64 * c;
    if (q >= dq) continue;
    float g[8];
    unpack8(reinterpret_cast<const u32x4*>(a.g)[q], g);
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] = v[c][e] * rstd * g[e];
    reinterpret_cast<u32x4*>(a.y)[row * dq + q] = pack8(g);
  }
}

// dx = rstd (g dy - xhat mean(g dy xhat)) (+ the residual's own gradient), and this
// workgroup's sum over its rows of dy xhat into part[blockIdx.x].
template <int NC, bool RES, bool DX>
__global__ __launch_bounds__(256) void k_rmsnorm_bwd(RmsNormGradArgs a) {
  extern __shared__ float acc[];  // d sums
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, dq = a.d / 8;
  float g[NC][8], dg[NC][8];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int q = lane + 64 * c;
    u32x4 w = {0u, 0u, 0u, 0u};
    if (q < dq) w = reinterpret_cast<const u32x4*>(a.g)[q];
    unpack8(w, g[c]);
#pragma unroll
    for (int e = 0; e < 8; ++e) dg[c][e] = 0.0f;
  }
  for (int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + wave; row < a.rows; row += static_cast<int64_t>(gridDim.x) * 4) {
    const float rstd = a.rstd[row];
    float xh[NC][8], gd[NC][8];
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int q = lane + 64 * c;
      u32x4 wx = {0u, 0u, 0u, 0u}, wd = {0u, 0u, 0u, 0u};
      if (q < dq) {
        wx = reinterpret_cast<const u32x4*>(a.x)[row * dq + q];
        wd = reinterpret_cast<const u32x4*>(a.dy)[row * dq + q];
      }
      unpack8(wx, xh[c]);
      unpack8(wd, gd[c]);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xh[c][e] *= rstd;
        dg[c][e] += gd[c][e] * xh[c][e];
        gd[c][e] *= g[c][e];
        s += gd[c][e] * xh[c][e];
      }
    }
    if constexpr (DX) {
      const float mean = wave_sum(s) / static_cast<float>(a.d);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int q = lane + 64 * c;
        if (q >= dq) continue;
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = rstd * (gd[c][e] - xh[c][e] * mean);
        if constexpr (RES) {
          float r[8];
          unpack8(reinterpret_cast<const u32x4*>(a.dres)[row * dq + q], r);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] += r[e];
        }
        reinterpret_cast<u32x4*>(a.dx)[row * dq + q] = pack8(o);
      }
    }
  }
  // the four waves' sums, in wave order
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int q = lane + 64 * c;
        if (q >= dq) continue;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[8 * q + e] = w == 0 ? dg[c][e] : acc[8 * q + e] + dg[c][e];
      }
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < a.d; i += 256) a.part[static_cast<int64_t>(blockIdx.x) * a.d + i] = acc[i];
}

// dg[i] = the sum of part[0 .. parts - 1][i], rounded to bf16: 16 columns per
// workgroup, 16 threads per column with every 16th part each, their sums in order.
__global__ __launch_bounds__(256) void k_rmsnorm_dg(const float* part, int parts, int d, uint16_t* dg) {
  __shared__ float s[16][17];
  const int c = threadIdx.x & 15, k = threadIdx.x >> 4, i = static_cast<int>(blockIdx.x) * 16 + c;
  float v = 0.0f;
  if (i < d) {
    // eight loads in flight: few workgroups, so the loop is latency bound
    int p = k;
    for (; p + 7 * 16 < parts; p += 8 * 16) {
      float t[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = part[static_cast<int64_t>(p + 16 * j) * d + i];
#pragma unroll
      for (int j = 0; j < 8; ++j) v += t[j];
    }
    for (; p < parts; p += 16) v += part[static_cast<int64_t>(p) * d + i];
  }
  s[k][c] = v;
  __syncthreads();
  if (k == 0 && i < d) {
    float t = s[0][c];
#pragma unroll
    for (int j = 1; j < 16; ++j) t += s[j][c];
    dg[i] = f32_to_bf16(t);
  }
}

// -------------------------------- SwiGLU -----------------------------------
// gu [rows][2 f] = [gate | up]; s = silu(gate) and act = s up, both [rows][f]; one
// 8-element chunk per thread.  s is rounded to bf16 before the product, as the two
// separate operations do.
__global__ __launch_bounds__(256) void k_swiglu_fwd(const uint16_t* gu, uint16_t* s, uint16_t* act, int64_t rows, int fq) {
  const int64_t u = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (u >= rows * fq) return;
  const int64_t row = u / fq, q = u - row * fq;
  const u32x4* src = reinterpret_cast<const u32x4*>(gu) + row * 2 * fq + q;
  float g[8], up[8], sv[8];
  unpack8(src[0], g);
  unpack8(src[fq], up);
#pragma unroll
  for (int e = 0; e < 8; ++e) sv[e] = g[e] / (1.0f + expf(-g[e]));
  const u32x4 sw = pack8(sv);
  reinterpret_cast<u32x4*>(s)[u] = sw;
  unpack8(sw, sv);
#pragma unroll
  for (int e = 0; e < 8; ++e) sv[e] *= up[e];
  reinterpret_cast<u32x4*>(act)[u] = pack8(sv);
}

// dup = dact s;  dgate = dact up sigma (1 + gate (1 - sigma)), into dgu [rows][2 f].
__global__ __launch_bounds__(256) void k_swiglu_bwd(const uint16_t* gu, const uint16_t* s, const uint16_t* dact,
                                                    uint16_t* dgu, int64_t rows, int fq) {
  const int64_t u = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (u >= rows * fq) return;
  const int64_t row = u / fq, q = u - row * fq, o = row * 2 * fq + q;
  float g[8], up[8], sv[8], d[8], dg[8];
  unpack8(reinterpret_cast<const u32x4*>(gu)[o], g);
  unpack8(reinterpret_cast<const u32x4*>(gu)[o + fq], up);
  unpack8(reinterpret_cast<const u32x4*>(s)[u], sv);
  unpack8(reinterpret_cast<const u32x4*>(dact)[u], d);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float sg = 1.0f / (1.0f + expf(-g[e]));
    dg[e] = d[e] * up[e] * (sg * (1.0f + g[e] * (1.0f - sg)));
    sv[e] *= d[e];
  }
  reinterpret_cast<u32x4*>(dgu)[o] = pack8(dg);
  reinterpret_cast<u32x4*>(dgu)[o + fq] = pack8(sv);
}

// out [rows][3 dq chunks] = the rows of a, b and c side by side (the gradients of
// q, k and v joined into q|k|v's); one 16-byte chunk per thread.
__global__ __launch_bounds__(256) void k_join3(const u32x4* a, const u32x4* b, const u32x4* c, u32x4* out, int64_t rows,
                                               int dq) {
  const int64_t u = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (u >= rows * dq) return;
  const int64_t row = u / dq, q = u - row * dq;
  const u32x4 va = a[u], vb = b[u], vc = c[u];
  u32x4* o = out + row * 3 * dq + q;
  o[0] = va;
  o[dq] = vb;
  o[2 * dq] = vc;
}

// ----------------------------- cross-entropy --------------------------------
// A row of V logits starts at any 2-byte offset when V is odd: rows are walked in
// the 16-byte chunks of the whole buffer, elements outside the row (or past the
// buffer) left out.
struct Chunk {
  float v[8];
  int lo, hi;  // elements of the chunk inside the row
};

__device__ __forceinline__ Chunk ce_chunk(const uint16_t* x, int64_t q, int64_t begin, int64_t end, int64_t total) {
  Chunk c;
  const int64_t e0 = q * 8;
  c.lo = e0 < begin ? static_cast<int>(begin - e0) : 0;
  c.hi = e0 + 8 > end ? static_cast<int>(end - e0) : 8;
  if (e0 + 8 <= total) {
    unpack8(reinterpret_cast<const u32x4*>(x)[q], c.v);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) c.v[e] = e0 + e < total ? bf16_to_f32(x[e0 + e]) : 0.0f;
  }
  return c;
}

// exp(x), x <= 0 here; -inf gives 0, NaN stays NaN
__device__ __forceinline__ float ce_exp(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }

// One workgroup per row, one pass: running maximum and sum of exponentials per
// lane, merged over the workgroup.  loss = lse - x[target] and lse per row; a
// target of ignore_index (or outside 0 .. V - 1: NaN) has no part in the mean.
__global__ __launch_bounds__(256) void k_ce_fwd(CeArgs a) {
  __shared__ float sm[4], ssum[4];
  const int64_t row = blockIdx.x, begin = row * a.V, end = begin + a.V, total = a.rows * a.V;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float ninf = -__builtin_inff();
  float m = ninf, s = 0.0f;
  // NE elements into the running maximum and sum; `in(e)`: element e is the row's
  auto take = [&](const auto& v, auto in) {
    constexpr int NE = sizeof(v) / sizeof(float);
    float cm = ninf;
#pragma unroll
    for (int e = 0; e < NE; ++e) cm = in(e) ? fmaxf(cm, v[e]) : cm;
    const float nm = fmaxf(m, cm);
    // no element above -inf so far: their exponentials add nothing yet (the shift
    // 0 keeps exp(-inf) = 0 and lets a NaN through)
    const float sh = nm == ninf ? 0.0f : nm;
    float t = 0.0f;
#pragma unroll
    for (int e = 0; e < NE; ++e) t += in(e) ? ce_exp(v[e] - sh) : 0.0f;
    s = s * (m == ninf ? 1.0f : ce_exp(m - sh)) + t;
    m = nm;
  };
  // four chunks in flight while all of them lie inside the row (one at a time, each
  // load waited for the maximum of the one before), then one by one
  constexpr int U = 4;
  for (int64_t q = begin / 8 + threadIdx.x; q * 8 < end;) {
    if (q * 8 >= begin && (q + (U - 1) * 256) * 8 + 8 <= end) {
      u32x4 w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) w[u] = reinterpret_cast<const u32x4*>(a.x)[q + u * 256];
      float v[8 * U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float p[8];
        unpack8(w[u], p);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[8 * u + e] = p[e];
      }
      take(v, [](int) { return true; });
      q += U * 256;
    } else {
      const Chunk c = ce_chunk(a.x, q, begin, end, total);
      take(c.v, [&](int e) { return e >= c.lo && e < c.hi; });
      q += 256;
    }
  }
  const float wm = wave_max(m), wsh = wm == ninf ? 0.0f : wm;
  const float ws = wave_sum(s * (m == ninf ? 1.0f : ce_exp(m - wsh)));
  if (lane == 0) {
    sm[wave] = wm;
    ssum[wave] = ws;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float M = sm[0];
    for (int w = 1; w < 4; ++w) M = fmaxf(M, sm[w]);
    float S = 0.0f;
    for (int w = 0; w < 4; ++w) S += ssum[w] * (sm[w] == ninf ? 1.0f : ce_exp(sm[w] - (M == ninf ? 0.0f : M)));
    const float lse = M + logf(S);
    a.lse[row] = lse;
    const int64_t t = a.target[row];
    float loss = 0.0f;
    if (t != a.ignore_index)
      loss = t >= 0 && t < a.V ? lse - bf16_to_f32(a.x[begin + t]) : __builtin_nanf("");
    a.loss_row[row] = loss;
  }
}

// The mean of the rows' losses over the targets that count, their number, and whether
// every target is valid; one workgroup, fp64 sums in a fixed order.
__global__ __launch_bounds__(1024) void k_ce_mean(CeArgs a) {
  __shared__ double sl[1024], sc[1024];
  double l = 0.0, c = 0.0;
  int bad = 0;
  for (int64_t r = threadIdx.x; r < a.rows; r += 1024) {
    const int64_t t = a.target[r];
    if (t == a.ignore_index) continue;
    bad |= t < 0 || t >= a.V ? 1 : 0;
    l += a.loss_row[r];
    c += 1.0;
  }
  sl[threadIdx.x] = l;
  sc[threadIdx.x] = c;
  bad = __syncthreads_or(bad);
  for (int d = 512; d > 0; d >>= 1) {
    if (static_cast<int>(threadIdx.x) < d) {
      sl[threadIdx.x] += sl[threadIdx.x + d];
      sc[threadIdx.x] += sc[threadIdx.x + d];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.loss[0] = static_cast<float>(sl[0] / sc[0]);
    a.count[0] = static_cast<float>(sc[0]);
    a.valid[0] = bad != 0 ? 0.0f : 1.0f;
  }
}

// dx = (softmax(x) - onehot(target)) dloss / count; softmax(x) times zero for ignored
// rows (NaN where that is), NaN (as the loss) for a target outside 0 .. V - 1.
__global__ __launch_bounds__(256) void k_ce_bwd(CeGradArgs a) {
  const int64_t row = blockIdx.x, begin = row * a.V, end = begin + a.V, total = a.rows * a.V;
  const int64_t t = a.target[row];
  const bool ignored = t == a.ignore_index;
  const float lse = ignored || (t >= 0 && t < a.V) ? a.lse[row] : __builtin_nanf("");
  const float scale = ignored ? 0.0f : a.dloss[0] / a.count[0];
  for (int64_t q = begin / 8 + threadIdx.x; q * 8 < end; q += 256) {
    Chunk c = ce_chunk(a.x, q, begin, end, total);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float p = ce_exp(c.v[e] - lse) - (q * 8 + e == begin + t ? 1.0f : 0.0f);
      c.v[e] = p * scale;
    }
    if (c.lo == 0 && c.hi == 8) {
      reinterpret_cast<u32x4*>(a.dx)[q] = pack8(c.v);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (e >= c.lo && e < c.hi) a.dx[q * 8 + e] = f32_to_bf16(c.v[e]);
    }
  }
}

template <bool ADD>
void rmsnorm_fwd(const RmsNormArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<uint32_t>(ceil_div(a.rows, 4)));
  switch (ceil_div(a.d, 512)) {
    case 1: hipLaunchKernelGGL((k_rmsnorm_fwd<1, ADD>), grid, dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((k_rmsnorm_fwd<2, ADD>), grid, dim3(256), 0, s, a); break;
    case 3: case 4: hipLaunchKernelGGL((k_rmsnorm_fwd<4, ADD>), grid, dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_rmsnorm_fwd<8, ADD>), grid, dim3(256), 0, s, a); break;
  }
}

template <bool RES, bool DX>
void rmsnorm_bwd(const RmsNormGradArgs& a, int grid, hipStream_t s) {
  const size_t lds = size_t(a.d) * sizeof(float);
  switch (ceil_div(a.d, 512)) {
    case 1: hipLaunchKernelGGL((k_rmsnorm_bwd<1, RES, DX>), dim3(grid), dim3(256), lds, s, a); break;
    case 2: hipLaunchKernelGGL((k_rmsnorm_bwd<2, RES, DX>), dim3(grid), dim3(256), lds, s, a); break;
    case 3: case 4: hipLaunchKernelGGL((k_rmsnorm_bwd<4, RES, DX>), dim3(grid), dim3(256), lds, s, a); break;
    default: hipLaunchKernelGGL((k_rmsnorm_bwd<8, RES, DX>), dim3(grid), dim3(256), lds, s, a); break;
  }
}

int status() { return hipGetLastError() == hipSuccess ? 0 : -5; }

}  // namespace
}  // namespace compact

using namespace compact;

extern "C" {

int compact_block_rmsnorm_fwd(const RmsNormArgs* a, void* stream) {
  if (a->rows < 1 || a->rows > int64_t(1) << 31 || a->d < 8 || a->d % 8 != 0 || a->d > kRmsNormMaxD) return -1;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (a->add != nullptr) rmsnorm_fwd<true>(*a, s);
  else rmsnorm_fwd<false>(*a, s);
  return status();
}

// Rows of partial sums (fp32 [parts][d]) that the backward needs.
int compact_block_rmsnorm_parts(int64_t rows) {
  const int64_t b = ceil_div(rows, 4 * 4);  // at least four rows per wave, at most 1024 workgroups
  return static_cast<int>(b < 1 ? 1 : b > 1024 ? 1024 : b);
}

int compact_block_rmsnorm_bwd(const RmsNormGradArgs* a, void* stream) {
  if (a->rows < 1 || a->rows > int64_t(1) << 31 || a->d < 8 || a->d % 8 != 0 || a->d > kRmsNormMaxD) return -1;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int parts = compact_block_rmsnorm_parts(a->rows);
  if (a->dx == nullptr) rmsnorm_bwd<false, false>(*a, parts, s);
  else if (a->dres != nullptr) rmsnorm_bwd<true, true>(*a, parts, s);
  else rmsnorm_bwd<false, true>(*a, parts, s);
  hipLaunchKernelGGL(k_rmsnorm_dg, dim3(static_cast<uint32_t>(ceil_div(a->d, 16))), dim3(256), 0, s, a->part, parts,
                     a->d, a->dg);
  return status();
}

int compact_block_swiglu_fwd(const uint16_t* gu, uint16_t* s, uint16_t* act, int64_t rows, int64_t f, void* stream) {
  const int64_t blocks = ceil_div(rows * (f / 8), 256);
  if (rows < 1 || f < 8 || f % 8 != 0 || f > int64_t(1) << 30 || blocks > kMaxBlocks) return -1;
  hipLaunchKernelGGL(k_swiglu_fwd, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     gu, s, act, rows, static_cast<int>(f / 8));
  return status();
}

int compact_block_swiglu_bwd(const uint16_t* gu, const uint16_t* s, const uint16_t* dact, uint16_t* dgu, int64_t rows,
                             int64_t f, void* stream) {
  const int64_t blocks = ceil_div(rows * (f / 8), 256);
  if (rows < 1 || f < 8 || f % 8 != 0 || f > int64_t(1) << 30 || blocks > kMaxBlocks) return -1;
  hipLaunchKernelGGL(k_swiglu_bwd, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     gu, s, dact, dgu, rows, static_cast<int>(f / 8));
  return status();
}

int compact_block_join3(const void* a, const void* b, const void* c, void* out, int64_t rows, int64_t d, void* stream) {
  const int64_t blocks = ceil_div(rows * (d / 8), 256);
  if (rows < 1 || d < 8 || d % 8 != 0 || d > int64_t(1) << 30 || blocks > kMaxBlocks) return -1;
  hipLaunchKernelGGL(k_join3, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<const u32x4*>(a), static_cast<const u32x4*>(b), static_cast<const u32x4*>(c),
                     static_cast<u32x4*>(out), rows, static_cast<int>(d / 8));
  return status();
}

int compact_block_ce_fwd(const CeArgs* a, void* stream) {
  if (a->rows < 1 || a->rows > 0x7FFFFFFF || a->V < 1) return -1;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_ce_fwd, dim3(static_cast<uint32_t>(a->rows)), dim3(256), 0, s, *a);
  hipLaunchKernelGGL(k_ce_mean, dim3(1), dim3(1024), 0, s, *a);
  return status();
}

int compact_block_ce_bwd(const CeGradArgs* a, void* stream) {
  if (a->rows < 1 || a->rows > 0x7FFFFFFF || a->V < 1) return -1;
  hipLaunchKernelGGL(k_ce_bwd, dim3(static_cast<uint32_t>(a->rows)), dim3(256), 0, static_cast<hipStream_t>(stream), *a);
  return status();
}

}  // extern "C"
