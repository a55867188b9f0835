// Arguments of the block kernels (block_ops.hip), called by the PyTorch modules
// through _block_ops.py.  All pointers are device pointers; bf16 matrices are
// dense, 16-byte aligned, with row lengths that are multiples of 8 (the logits
// excepted: any V).  Entry points return 0, -1 (a size they do not take) or -5
// (HIP error).
#pragma once
#include <stdint.h>

namespace compact {

constexpr int kRmsNormMaxD = 4096;

// sum = x + add (when add is given), y = sum rstd g, rstd = 1 / sqrt(mean(sum^2) + eps)
struct RmsNormArgs {
  const uint16_t* x;
  const uint16_t* add;  // or NULL
  const uint16_t* g;
  uint16_t* sum;        // written when add is given
  uint16_t* y;
  float* rstd;
  int64_t rows;
  int d;
  float eps;
};

struct RmsNormGradArgs {
  const uint16_t* x;     // what was normalised
  const uint16_t* dy;
  const uint16_t* dres;  // gradient that reaches x past the norm, or NULL
  const uint16_t* g;
  const float* rstd;
  uint16_t* dx;          // or NULL
  float* part;           // [compact_block_rmsnorm_parts(rows)][d]
  uint16_t* dg;
  int64_t rows;
  int d;
};

struct CeArgs {
  const uint16_t* x;      // [rows][V]
  const int64_t* target;  // [rows]
  float* lse;             // [rows]
  float* loss_row;        // [rows] scratch
  float* loss;            // the mean
  float* count;           // number of targets that count
  float* valid;           // 1 if every target is ignore_index or in 0 .. V - 1, else 0
  int64_t rows, V, ignore_index;
};

struct CeGradArgs {
  const uint16_t* x;
  const int64_t* target;
  const float* lse;
  const float* count;     // of the forward
  const float* dloss;     // one value
  uint16_t* dx;
  int64_t rows, V, ignore_index;
};

}  // namespace compact
