// fp32 products on the bf16 matrix units (device part of gemm.hip).
//
// v_mfma_f32_16x16x4_f32 does 64 flops per cycle and SIMD, the bf16 MFMA 1024.
// An fp32 value is the exact sum of three bf16 values (h = x to nearest even,
// m = x - h to nearest even, l = the rest: 8 bits each and two signs), so
// a b = ah bh + (ah bm + am bh) + (am bm + ah bl + al bh) + terms below
// 2^-26 |a b|, which is under half the rounding of one fp32 product: six bf16
// MFMAs in place of eight fp32 ones of twice the cycles each, 2.7 times the
// fp32 rate at the peak.  The products are exact in fp32 and the sums are kept
// in fp32 accumulators.
#pragma once
#include "internal.hpp"
#include "wave.hpp"

namespace gnn {
namespace split {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = 256;
constexpr int BK = 32;  // k of a slab: one 16x16x32 MFMA

__device__ __forceinline__ uint32_t pack2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));  // nearest even
}

// eight fp32 values as three groups of eight bf16 values
__device__ __forceinline__ void split8(const float (&x)[8], uint4& h, uint4& m, uint4& l) {
  uint32_t ph[4], pm[4], pl[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
    ph[i] = pack2(a, b);
    a -= __uint_as_float(ph[i] << 16);
    b -= __uint_as_float(ph[i] & 0xFFFF0000u);
    pm[i] = pack2(a, b);
    a -= __uint_as_float(pm[i] << 16);
    b -= __uint_as_float(pm[i] & 0xFFFF0000u);
    pl[i] = pack2(a, b);
  }
  h = make_uint4(ph[0], ph[1], ph[2], ph[3]);
  m = make_uint4(pm[0], pm[1], pm[2], pm[3]);
  l = make_uint4(pl[0], pl[1], pl[2], pl[3]);
}

}  // namespace split
}  // namespace gnn
