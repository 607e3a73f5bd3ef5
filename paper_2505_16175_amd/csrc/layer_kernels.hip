// Small HBM-bound kernels of the decoder layer around the path: RMSNorm and the table of rotary angles.
#include "qp_internal.h"

#include <type_traits>

namespace qp {

// y[t][i] = x[t][i] / sqrt(mean_i x[t][i]^2 + eps) * w[i], f32 arithmetic, one rounding to bf16 at the store.
// One wavefront per token. Rows of up to RN_REG * 512 elements (8192 for RN_REG = 16) stay in registers between the
// sum of squares and the scaling, so the row is read once; longer rows are read a second time (from cache). With few
// tokens the kernel is one chain of latencies (8.3 us for one token when every chunk waited for its own weights), so the
// norm's weights are requested together with the row (AHEAD), and rows of up to 4096 elements take a variant of half the
// registers and loads. With the table below in the same launch as the first norm, a 7B layer takes 145.1 us for one
// token (154.5 before) and 260.7 for 64 (268.2).
// AHEAD doubles the registers of the 16-chunk variant: 3 wavefronts share a SIMD, 5 without (rows of up to 4096: 5 either
// way). It is the faster one while its wavefronts are all resident at once, 12 tokens per CU. us without / with, 8192
// elements: 1 token 9.2 / 7.6, 1024 15.2 / 11.7, 3072 23.8 / 22.9, 4096 26.9 / 31.5; 5120 elements: 20.5 / 23.5 at 4096.
// Rows beyond 8192 have nothing in registers to gain.
constexpr int RN_WAVES = 4;
constexpr int RN_AHEAD_PER_CU = 12;
template <int RN_REG, bool AHEAD>  // 16-byte chunks per lane held in registers; their weights requested with them
__device__ __forceinline__ void rms_norm_token(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                               bf16_t* __restrict__ out, int t, int d_model, float eps) {
  const int lane = threadIdx.x & 63;
  const int chunks = d_model / 8;
  const uint4* xr = (const uint4*)(x + (size_t)t * d_model);
  const uint4* wr = (const uint4*)w;
  uint4* orow = (uint4*)(out + (size_t)t * d_model);
  const bool in_regs = chunks <= RN_REG * 64;
  uint4 held[RN_REG], wts[AHEAD ? RN_REG : 1];
  float ss = 0.f;
  if (in_regs) {
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    if constexpr (AHEAD) {
#pragma unroll
      for (int i = 0; i < RN_REG; ++i) held[i] = xr[min(lane + 64 * i, chunks - 1)];  // clamped, dropped below
#pragma unroll
      for (int i = 0; i < RN_REG; ++i) wts[i] = wr[min(lane + 64 * i, chunks - 1)];
    } else {
#pragma unroll
      for (int i = 0; i < RN_REG; ++i) {
        const int c = lane + 64 * i;
        held[i] = c < chunks ? xr[c] : make_uint4(0u, 0u, 0u, 0u);
      }
    }
#pragma unroll
    for (int i = 0; i < RN_REG; ++i) {
      float f[8];
      if constexpr (AHEAD) widen16<bf16_t>(lane + 64 * i < chunks ? held[i] : zero, f);
      else widen16<bf16_t>(held[i], f);
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
  auto scale_store = [&](int c, const uint4& raw, const uint4* ahead) {
    float f[8], g[8];
    widen16<bf16_t>(raw, f);
    widen16<bf16_t>(ahead != nullptr ? *ahead : wr[c], g);
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
      if (c < chunks) scale_store(c, held[i], AHEAD ? &wts[AHEAD ? i : 0] : nullptr);
    }
  } else {
    for (int c = lane; c < chunks; c += 64) scale_store(c, xr[c], nullptr);
  }
}

template <int RN_REG, bool AHEAD>
__global__ __launch_bounds__(RN_WAVES * 64) void rms_norm_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                                 bf16_t* __restrict__ out, int n_tokens, int d_model,
                                                                 float eps) {
  const int t = blockIdx.x * RN_WAVES + (threadIdx.x >> 6);
  if (t < n_tokens) rms_norm_token<RN_REG, AHEAD>(x, w, out, t, d_model, eps);
}

__device__ __forceinline__ void rope_entry(const RopeArgs& a, int id) {
  if (id < a.n_tokens * 64) a.cos_sin[id] = rope_cos_sin(a, id >> 6, id & 63);
}

__global__ __launch_bounds__(256) void rope_table_kernel(RopeArgs a) { rope_entry(a, blockIdx.x * 256 + threadIdx.x); }

// The layer's norm and its rotary table in one launch: they share nothing, and on one stream the table's launch (4 us
// at any small token count, most of it the latency of an f64 sincos) would stand between the norm and the projection.
// Workgroups [0, n_rope) fill the table, the others norm RN_WAVES tokens each.
template <int RN_REG, bool AHEAD>
__global__ __launch_bounds__(RN_WAVES * 64) void norm_rope_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                                  bf16_t* __restrict__ out, int n_tokens, int d_model,
                                                                  float eps, RopeArgs a, int n_rope) {
  if ((int)blockIdx.x < n_rope) {
    rope_entry(a, blockIdx.x * 256 + threadIdx.x);
    return;
  }
  const int t = (blockIdx.x - n_rope) * RN_WAVES + (threadIdx.x >> 6);
  if (t < n_tokens) rms_norm_token<RN_REG, AHEAD>(x, w, out, t, d_model, eps);
}

template <typename F>
static void with_norm_variant(int n_tokens, int d_model, F launch) {
  typedef std::true_type Yes;
  typedef std::false_type No;
  if (d_model <= 8 * 512) launch(std::integral_constant<int, 8>(), Yes());
  else if (d_model <= 16 * 512 && n_tokens <= RN_AHEAD_PER_CU * device_cu_count()) launch(std::integral_constant<int, 16>(), Yes());
  else launch(std::integral_constant<int, 16>(), No());
}

void launch_rms_norm(const void* x, const void* w, void* out, int n_tokens, int d_model, float eps, hipStream_t s) {
  with_norm_variant(n_tokens, d_model, [&](auto reg, auto ahead) {
    hipLaunchKernelGGL((rms_norm_kernel<reg.value, ahead.value>), dim3((n_tokens + RN_WAVES - 1) / RN_WAVES), dim3(RN_WAVES * 64),
                       0, s, (const bf16_t*)x, (const bf16_t*)w, (bf16_t*)out, n_tokens, d_model, eps);
  });
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
  with_norm_variant(n_tokens, d_model, [&](auto reg, auto ahead) {
    hipLaunchKernelGGL((norm_rope_kernel<reg.value, ahead.value>), dim3(n_rope + (n_tokens + RN_WAVES - 1) / RN_WAVES),
                       dim3(RN_WAVES * 64), 0, s, (const bf16_t*)x, (const bf16_t*)w, (bf16_t*)out, n_tokens, d_model, eps, a,
                       n_rope);
  });
}

}  // namespace qp
