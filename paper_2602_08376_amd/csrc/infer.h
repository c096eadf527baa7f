// Types shared by the kernels that use the quantized layer (infer.hip,
// infer_few.hip).
#pragma once

#include "device.h"
#include "kernels.h"
#include "x_piece.h"

namespace ojbkq {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

// Two float32 weights rounded to fp16 together (one packed convert, round to
// nearest even as for a single one).
__device__ __forceinline__ h2 to_f16x2(float lo, float hi) {
  return __builtin_convertvector(f2{lo, hi}, h2);
}
typedef float f4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));

struct DqArgs {
  const uint32_t* P;
  int64_t wpr;                 // words per packed row
  const float* S;
  const float* Z;
  int64_t n, m, g, G;
  const uint16_t* X;           // fp16 bits, [m, T] with row stride ldx
  int64_t T, ldx;
  const int32_t* perm;         // null, or X row of packed position k = perm[k]
  float* Y;
  int64_t ldy;
  int64_t tiles_n;
  const _Float16* Wh;          // W_hat [n, mw] fp16 formed beforehand (null: dequantize in the product)
  int64_t mw;                  // its row stride, m rounded up to a whole stage (zeros past m)
};

// Row of X that packed position k (< m) multiplies.
__device__ __forceinline__ int64_t x_row(const DqArgs& a, int64_t k) {
  if (!a.perm) return k;
  const int64_t r = a.perm[k];
  return r < 0 ? 0 : (r >= a.m ? a.m - 1 : r);
}

// The product for few tokens (infer_few.hip); needs no workspace.
hipError_t launch_dequant_few(const DqArgs& a, int bits, hipStream_t stream);

}  // namespace ojbkq
