// The angles of the rotary embedding, for the kernels that tabulate them and those that take them on the way.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qp {

// cos_sin[t][i] = (cos, sin)(pos[axis(i)][t] * theta^(-i/64)) for the 64 rotation frequencies of head_dim 128;
// frequencies [0, s0) use position axis 0, [s0, s0+s1) axis 1, the rest axis 2. The angle (up to ~1e5 rad for long
// videos) and its sine/cosine are evaluated in f64 and rounded once, so the table is as exact as f32 holds.
struct RopeArgs {
  const int32_t* pos;
  long axis_stride;
  int n_tokens;
  float theta;
  int s0, s1;
  float2* cos_sin;  // [n_tokens][64], where a table is wanted
};
__device__ __forceinline__ float2 rope_cos_sin(const RopeArgs& a, int t, int i) {
  const int axis = i < a.s0 ? 0 : (i < a.s0 + a.s1 ? 1 : 2);
  const double ang = (double)a.pos[axis * a.axis_stride + t] * exp2(-(double)i / 64.0 * log2((double)a.theta));
  double sn, cs;
  sincos(ang, &sn, &cs);
  return make_float2((float)cs, (float)sn);
}

// A rotary pair turned by its angle. The roundings are spelled out, not left to the compiler's contraction: every store of
// the QKV projection (tiles, split product, weight streaming) rounds alike.
__device__ __forceinline__ void rotate_pair(float& lo, float& hi, float c, float s) {
  const float x0 = lo, x1 = hi;
  lo = fmaf(x0, c, -__fmul_rn(x1, s));
  hi = fmaf(x1, c, __fmul_rn(x0, s));
}

}  // namespace qp
