// Shared device helpers: vector types, bf16 conversion, MFMA wrapper, grid
// mapping.  gfx950 (CDNA4) only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace compact {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kNumXcd = 8;  // MI355X: 8 XCDs, each with its own L2

// fp32 -> bf16 bits, round to nearest even (v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  const __bf16 b = static_cast<__bf16>(f);
  return __builtin_bit_cast(uint16_t, b);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}

// Two values, one v_cvt_pk_bf16_f32 (same rounding as f32_to_bf16).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// 32x32x16 bf16 MFMA, fp32 accumulate.  Operand lane layout: lane l holds
// row/column (l mod 32) and the 8 consecutive K values 8*(l/32) .. +7.
// Result: lane l, element v -> row 8*(v/4) + 4*(l/32) + (v mod 4), column l mod 32.
__device__ __forceinline__ f32x16 mfma32x32x16(const u32x4& a, const u32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Bijective remap of the linear workgroup id so that consecutive logical tiles
// run on the same XCD (workgroups are dealt round-robin over the 8 XCDs).
__device__ __forceinline__ uint32_t xcd_remap(uint32_t bid, uint32_t nblk) {
  const uint32_t q = nblk / kNumXcd, rem = nblk % kNumXcd;
  const uint32_t x = bid % kNumXcd, k = bid / kNumXcd;
  return x * q + (x < rem ? x : rem) + k;
}

// Several layers per launch: block b belongs to the layer l with
// begin[l] <= b < begin[l + 1] (begin[0] = 0, begin[count] = grid size).

__device__ __forceinline__ int batch_layer_of(const int* begin, int count, int b) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (begin[mid] <= b) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__host__ __device__ constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
__host__ __device__ constexpr int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

// Layer tables of Alg. 3's launches, by shape: sizes once per distinct shape.
constexpr int kStepShapes = 8;  // distinct shapes per launch
constexpr int kStepFew = 8;     // layers of the small table: a launch of few has 0.5 KB of arguments, not 4

struct StepShape {
  int n, m, r, ldw;
};

// Shape index of layer l, four to a word (a byte array would be read through the
// vector memory path, at the head of every workgroup).
__host__ __device__ inline int shape_index(const uint32_t* words, int l) {
  return static_cast<int>((words[l >> 2] >> (8 * (l & 3))) & 0xFFu);
}

// Scratch of a layer: N [r][round_up(m, 8)], then (bf16) P^T [r][round_up(n, 64)],
// each on a 256-byte boundary.
__host__ __device__ inline int64_t step_ldn(int64_t m) { return round_up(m, 8); }
__host__ __device__ inline int64_t step_ldpt(int64_t n) { return round_up(n, 64); }
__host__ __device__ inline int64_t step_n_bytes(int64_t m, int64_t r, int esz) {
  return round_up(r * step_ldn(m) * esz, int64_t(256));
}

}  // namespace compact
