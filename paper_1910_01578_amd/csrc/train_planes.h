// An fp32 value as three bf16 planes, for fp32 accuracy on the bf16 matrix cores.
#pragma once

#include "device_common.h"

namespace gdp {
namespace tr {

// Eight fp32 values as three bf16 planes each, v = p[0] + p[1] + p[2] exactly:
// each plane is the remainder rounded to nearest.  Exact for finite values that
// round to a finite bf16 (below 3.396e38); beyond, and for an infinity, p[0] is
// infinite and the rest its sign's opposite infinity or NaN, so a product of such
// planes is not finite.
struct Planes {
  bf16x8 p[3];
};
__device__ __forceinline__ Planes split8(const float (&v)[8]) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
  union P8 {
    bf16x2 h[4];
    bf16x8 q;
  } p1, p2, p3;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x2 a = {v[2 * i], v[2 * i + 1]};
    p1.h[i] = __builtin_convertvector(a, bf16x2);
    const f32x2 r = a - __builtin_convertvector(p1.h[i], f32x2);
    p2.h[i] = __builtin_convertvector(r, bf16x2);
    p3.h[i] = __builtin_convertvector(r - __builtin_convertvector(p2.h[i], f32x2), bf16x2);
  }
  Planes o;
  o.p[0] = p1.q;
  o.p[1] = p2.q;
  o.p[2] = p3.q;
  return o;
}

}  // namespace tr
}  // namespace gdp
