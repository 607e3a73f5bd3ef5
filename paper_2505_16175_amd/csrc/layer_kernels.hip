// Small HBM-bound kernels of the decoder layer around the path: RMSNorm and the table of rotary angles.
#include "qp_internal.h"

namespace qp {

// y[t][i] = x[t][i] / sqrt(mean_i x[t][i]^2 + eps) * w[i], f32 arithmetic, one rounding to bf16 at the store.
// One wavefront per token. Rows of up to RN_REG * 512 elements (8192 for RN_REG = 16) stay in registers between the
// sum of squares and the scaling, so the row is read once; longer rows are read a second time (from cache). With few
// tokens the kernel is one chain of latencies (8.3 us for one token when every chunk waited for its own weights), so the
// norm's weights are requested together with the row, and rows of up to 4096 elements take a variant of half the
// registers and loads. With the table below in the same launch as the first norm, a 7B layer takes 145.1 us for one
// token (154.5 before) and 260.7 for 64 (268.2).
constexpr int RN_WAVES = 4;
template <int RN_REG>  // 16-byte chunks per lane held in registers
__device__ __forceinline__ void rms_norm_token(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                               bf16_t* __restrict__ out, int t, int d_model, float eps) {
  const int lane = threadIdx.x & 63;
  const int chunks = d_model / 8;
  const uint4* xr = (const uint4*)(x + (size_t)t * d_model);
  const uint4* wr = (const uint4*)w;
  uint4* orow = (uint4*)(out + (size_t)t * d_model);
  const bool in_regs = chunks <= RN_REG * 64;
  uint4 held[RN_REG], wts[RN_REG];
  float ss = 0.f;
  if (in_regs) {
#pragma unroll
    for (int i = 0; i < RN_REG; ++i) held[i] = xr[min(lane + 64 * i, chunks - 1)];  // clamped, dropped below
#pragma unroll
    for (int i = 0; i < RN_REG; ++i) wts[i] = wr[min(lane + 64 * i, chunks - 1)];
#pragma unroll
    for (int i = 0; i < RN_REG; ++i) {
      float f[8];
      widen16<bf16_t>(lane + 64 * i < chunks ? held[i] : make_uint4(0u, 0u, 0u, 0u), f);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss = fmaf(f[e], f[e], ss);
    }
  } else {
    for (int c = lane; c < chunks; c += 64) {
      float f[8];
      widen16<bf16_t>(xr[c], f);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss = fmaf(f[e], f[e], ss);
    }
  }
  ss = wave_sum(ss);
  const float inv = 1.f / sqrtf(ss / (float)d_model + eps);
  auto scale_store = [&](int c, const uint4& raw, const uint4& wraw) {
    float f[8], g[8];
    widen16<bf16_t>(raw, f);
    widen16<bf16_t>(wraw, g);
    uint32_t p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      p[e] = (uint32_t)f32_to_bf16_rne(f[2 * e] * inv * g[2 * e]) | ((uint32_t)f32_to_bf16_rne(f[2 * e + 1] * inv * g[2 * e + 1]) << 16);
    orow[c] = make_uint4(p[0], p[1], p[2], p[3]);
  };
  if (in_regs) {
#pragma unroll
    for (int i = 0; i < RN_REG; ++i) {
      const int c = lane + 64 * i;
      if (c < chunks) scale_store(c, held[i], wts[i]);
    }
  } else {
    for (int c = lane; c < chunks; c += 64) scale_store(c, xr[c], wr[c]);
  }
}

// cos_sin[t][i] = (cos, sin)(pos[axis(i)][t] * theta^(-i/64)) for the 64 rotation frequencies of head_dim 128;
// frequencies [0, s0) use position axis 0, [s0, s0+s1) axis 1, the rest axis 2. The angle (up to ~1e5 rad for long
// videos) and its sine/cosine are evaluated in f64 and rounded once, so the table is as exact as f32 holds.
struct RopeArgs {
  const int32_t* pos;
  long axis_stride;
  int n_tokens;
  float theta;
  int s0, s1;
  float2* cos_sin;
};
__device__ __forceinline__ void rope_entry(const RopeArgs& a, int id) {
  if (id >= a.n_tokens * 64) return;
  const int t = id >> 6, i = id & 63;
  const int axis = i < a.s0 ? 0 : (i < a.s0 + a.s1 ? 1 : 2);
  const double ang = (double)a.pos[axis * a.axis_stride + t] * exp2(-(double)i / 64.0 * log2((double)a.theta));
  double sn, cs;
  sincos(ang, &sn, &cs);
  a.cos_sin[id] = make_float2((float)cs, (float)sn);
}

template <int RN_REG>
__global__ __launch_bounds__(RN_WAVES * 64) void rms_norm_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                                 bf16_t* __restrict__ out, int n_tokens, int d_model,
                                                                 float eps) {
  const int t = blockIdx.x * RN_WAVES + (threadIdx.x >> 6);
  if (t < n_tokens) rms_norm_token<RN_REG>(x, w, out, t, d_model, eps);
}

__global__ __launch_bounds__(256) void rope_table_kernel(RopeArgs a) { rope_entry(a, blockIdx.x * 256 + threadIdx.x); }

// The layer's norm and its rotary table in one launch: they share nothing, and on one stream the table's launch (4 us
// at any small token count, most of it the latency of an f64 sincos) would stand between the norm and the projection.
// Workgroups [0, n_rope) fill the table, the others norm RN_WAVES tokens each.
template <int RN_REG>
__global__ __launch_bounds__(RN_WAVES * 64) void norm_rope_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                                  bf16_t* __restrict__ out, int n_tokens, int d_model,
                                                                  float eps, RopeArgs a, int n_rope) {
  if ((int)blockIdx.x < n_rope) {
    rope_entry(a, blockIdx.x * 256 + threadIdx.x);
    return;
  }
  const int t = (blockIdx.x - n_rope) * RN_WAVES + (threadIdx.x >> 6);
  if (t < n_tokens) rms_norm_token<RN_REG>(x, w, out, t, d_model, eps);
}

void launch_rms_norm(const void* x, const void* w, void* out, int n_tokens, int d_model, float eps, hipStream_t s) {
  const dim3 grid((n_tokens + RN_WAVES - 1) / RN_WAVES), block(RN_WAVES * 64);
  if (d_model <= 8 * 512)
    hipLaunchKernelGGL(rms_norm_kernel<8>, grid, block, 0, s, (const bf16_t*)x, (const bf16_t*)w, (bf16_t*)out, n_tokens, d_model, eps);
  else
    hipLaunchKernelGGL(rms_norm_kernel<16>, grid, block, 0, s, (const bf16_t*)x, (const bf16_t*)w, (bf16_t*)out, n_tokens, d_model, eps);
}

void launch_rope_table(const int32_t* pos, long axis_stride, int n_tokens, float theta, int s0, int s1, float* cos_sin,
                       hipStream_t s) {
  const RopeArgs a{pos, axis_stride, n_tokens, theta, s0, s1, (float2*)cos_sin};
  hipLaunchKernelGGL(rope_table_kernel, dim3((n_tokens * 64 + 255) / 256), dim3(256), 0, s, a);
}

void launch_norm_rope(const void* x, const void* w, void* out, int n_tokens, int d_model, float eps, const int32_t* pos,
                      long axis_stride, float theta, int s0, int s1, float* cos_sin, hipStream_t s) {
  const RopeArgs a{pos, axis_stride, n_tokens, theta, s0, s1, (float2*)cos_sin};
  const int n_rope = (n_tokens * 64 + 255) / 256;
  const dim3 grid(n_rope + (n_tokens + RN_WAVES - 1) / RN_WAVES), block(RN_WAVES * 64);
  if (d_model <= 8 * 512)
    hipLaunchKernelGGL(norm_rope_kernel<8>, grid, block, 0, s, (const bf16_t*)x, (const bf16_t*)w, (bf16_t*)out, n_tokens,
                       d_model, eps, a, n_rope);
  else
    hipLaunchKernelGGL(norm_rope_kernel<16>, grid, block, 0, s, (const bf16_t*)x, (const bf16_t*)w, (bf16_t*)out, n_tokens,
                       d_model, eps, a, n_rope);
}

}  // namespace qp
