// The projections of the decoder layer for a handful of tokens (Sec. 2.1's last stage: decoding one token at a time
// through the layer, over the pruned cache), gfx950:
//   Y[m][n] = sum_k X[m][k] W[n][k],   m <= 2 tokens, W [N][K] bf16 weights ([out][in]), f32 accumulation,
// with the same three stores as the matrix-pipe kernel of gemm_bf16.hip (PLAIN: bias / residual; QKV_ROPE: bias,
// rotary embedding, scatter to Q / K / V; SWIGLU: SiLU(gate) * up; Appendix D.1 for the latter).
//
// With so few tokens the product is a stream of the weights: every weight byte is read once and meets m activations,
// so HBM is the bound and the matrix pipe has nothing to offer (a 256-row tile would hold one or two useful rows). The
// matrix-pipe kernel serves such calls by dealing the contraction to k chunks and summing their partial tiles in a
// second launch; this kernel does it in one launch and without partials in memory:
//   * a workgroup of 4 wavefronts owns 4 weight rows, chosen so that the values a store combines belong to the same
//     workgroup: 4 consecutive outputs (PLAIN), 2 dims of a head and their rotary partners (QKV_ROPE), 2 gate rows and
//     the up rows of the same outputs (SWIGLU);
//   * the wavefronts walk k side by side, 16 bytes per lane and row (1 KB runs of each row per wavefront, 4 KB per
//     workgroup), two steps per loop trip, all loads of a trip issued before its first product: 8 KB of weights in
//     flight per wavefront, and a compute unit (up to 32 wavefronts) well over the ~40 KB that 8 TB/s need at ~2 us of
//     latency. A step past the end loads the first one again and is dropped: as a conditional load it was a branch that
//     waited for the loads before it, and the weights came at 4.1-5.6 TB/s. us at one token, conditional / not, 7B sizes:
//     gate/up 48.9 / 43.4 (6.3 TB/s), down 32.8 / 26.4, all four 102 / 89; 72B sizes 343 / 287, of which 9 by the
//     wavefronts' places (a quarter of k each: 296). Requesting the next trip's weights before the products of this one
//     gained nothing on top (89 and 291; at k <= 4096 there is one trip). The activations (a few KB per token) come from
//     L2 alongside;
//   * products are v_dot2_f32_bf16 (two multiply-adds per lane and instruction, f32 accumulation);
//   * the 64 lanes' sums are added by shuffles, the 4 wavefronts' sums meet in LDS and are added in wavefront order
//     (deterministic), and one lane per token applies the store.
//
// Inside a layer the QKV launch appends to the cache, and for one token (launch_gemv_fused) it also takes the RMSNorm of the
// row and the rotary angles, which as a launch of their own are latency and nothing else (6.1 us). Every workgroup repeats
// the norm: a wavefront takes the row's sum of squares, over its chunks and lanes in the order of rms_norm_kernel, so that the
// factor's bits are the same, while the first weights are on their way; another takes the workgroup's angles in double
// precision. It costs registers, and with them wavefronts in flight: for two tokens, and for the large gate/up launch
// (43.7 -> 52 us), more than the launch it saves. us with norms in both launches / in QKV at one or two tokens / QKV at one
// / nowhere: 7B layer, one token over 46,125 entries 117.5 / 115.5 / 115.5 / 117.8, two over 9,000 154 / 124 / 113.6 /
// 113.7; 72B layer, one 311 / 313 / 314 / 320, two 375 / 333 / 322 / 322.
#include "append.h"
#include "qp_internal.h"

#include <type_traits>

namespace qp {

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

constexpr int GV_WAVES = 4;
constexpr int GV_MAX_M = 2;  // tokens this kernel takes: every workgroup re-reads the activations, m / 4 of its weight bytes,
                             // and from 4 tokens on the tiled kernel with its split contraction is as fast or faster
constexpr int GV_NORM = 8;   // 16-byte chunks per lane of a row being normed that are in flight together

__device__ __forceinline__ float dot8(const uint4& w, const uint4& x, float acc) {
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.x), __builtin_bit_cast(bf16x2, x.x), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.y), __builtin_bit_cast(bf16x2, x.y), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.z), __builtin_bit_cast(bf16x2, x.z), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.w), __builtin_bit_cast(bf16x2, x.w), acc, false);
  return acc;
}

// 1 / rms of a row, as one wavefront of rms_norm_kernel takes it: the same sums in the same order
template <typename First>
__device__ __forceinline__ float gemv_inv_rms(const uint4* x, int chunks, int k, float eps, int lane, const First& first) {
  float ss = 0.f;
  auto add = [&](const uint4& raw) {
    float f[8];
    widen16<bf16_t>(raw, f);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(f[e], f[e], ss);
  };
#pragma unroll
  for (int i = 0; i < GV_NORM; ++i)
    if (lane + 64 * i < chunks) add(first[i]);
  for (int c0 = lane + 64 * GV_NORM; c0 < chunks; c0 += 64 * GV_NORM) {
    uint4 raw[GV_NORM];
#pragma unroll
    for (int i = 0; i < GV_NORM; ++i) raw[i] = x[min(c0 + 64 * i, chunks - 1)];
#pragma unroll
    for (int i = 0; i < GV_NORM; ++i)
      if (c0 + 64 * i < chunks) add(raw[i]);
  }
  return 1.f / sqrtf(wave_sum(ss) / (float)k + eps);
}
__device__ __forceinline__ uint4 scale8(const uint4& raw, const uint4& w, float inv) {  // as rms_norm_kernel stores it
  float f[8], g[8];
  widen16<bf16_t>(raw, f);
  widen16<bf16_t>(w, g);
  uint32_t p[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    p[e] = (uint32_t)f32_to_bf16_rne(f[2 * e] * inv * g[2 * e]) | ((uint32_t)f32_to_bf16_rne(f[2 * e + 1] * inv * g[2 * e + 1]) << 16);
  return make_uint4(p[0], p[1], p[2], p[3]);
}

struct NoFusion {};
struct AppendFusion {};

// M: tokens computed (1 or 2). F: NoFusion, AppendFusion (QKV_ROPE, the tokens are appended to the cache) or GemvFusion (that,
// the norm and the angles)
template <int MODE, int M, typename F>
__global__ __launch_bounds__(GV_WAVES * 64) void gemv_bf16_kernel(GemmArgs a, F fuse) {
  constexpr bool FUSED = std::is_same<F, GemvFusion>::value, APPEND = FUSED || std::is_same<F, AppendFusion>::value;
  static_assert(!APPEND || MODE == GEMM_QKV_ROPE, "keys and values are appended");
  static_assert(!FUSED || M == 1, "one wavefront takes the norm of the one row");
  __shared__ float part[GV_WAVES][4][M];
  __shared__ float inv_rms;
  __shared__ float2 angles[2];  // FUSED: (cos, sin) of this workgroup's two frequencies
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int quad = blockIdx.x;  // < n / 4
  const int d_ff = a.n >> 1;
  // the 4 weight rows of this workgroup: y[0], y[1] and their partners y[2], y[3] in the store below
  int row[4];
  if (MODE == GEMM_QKV_ROPE) {
    const int head = quad >> 5, f0 = 2 * (quad & 31);
    row[0] = head * 128 + f0, row[1] = row[0] + 1, row[2] = row[0] + 64, row[3] = row[0] + 65;
  } else if (MODE == GEMM_SWIGLU) {
    row[0] = 2 * quad, row[1] = row[0] + 1, row[2] = d_ff + row[0], row[3] = d_ff + row[0] + 1;
  } else {
    row[0] = 4 * quad, row[1] = row[0] + 1, row[2] = row[0] + 2, row[3] = row[0] + 3;
  }
  const int chunks = a.k / 8;
  const uint4* w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = (const uint4*)((const bf16_t*)a.w + (size_t)row[e] * a.k);
  const uint4* x[M];
#pragma unroll
  for (int t = 0; t < M; ++t) x[t] = (const uint4*)((const bf16_t*)a.x + (size_t)min(t, a.m - 1) * a.k);

  float acc[4][M];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int t = 0; t < M; ++t) acc[e][t] = 0.f;
  constexpr int STEP = GV_WAVES * 64;
  uint4 ahead[GV_NORM];  // FUSED: wavefront 0 takes the norm; the row is requested before anything else
  if constexpr (FUSED) {
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < GV_NORM; ++i) ahead[i] = x[0][min(lane + 64 * i, chunks - 1)];
    }
  }
  uint4 w0[4], w1[4], x0[M], x1[M], n0, n1;
  auto request = [&](int c) {
    const int c1 = c + STEP < chunks ? c + STEP : c;
#pragma unroll
    for (int e = 0; e < 4; ++e) w0[e] = w[e][c];
#pragma unroll
    for (int t = 0; t < M; ++t) x0[t] = x[t][c];
#pragma unroll
    for (int e = 0; e < 4; ++e) w1[e] = w[e][c1];
#pragma unroll
    for (int t = 0; t < M; ++t) x1[t] = x[t][c1];
    if constexpr (FUSED) n0 = ((const uint4*)fuse.norm_w)[c], n1 = ((const uint4*)fuse.norm_w)[c1];
  };
  int c = wave * 64 + lane;
  float inv = 0.f;
  if constexpr (FUSED) {
    request(min(c, chunks - 1));
    if (wave == 0) {
      const float v = gemv_inv_rms(x[0], chunks, a.k, fuse.eps, lane, ahead);
      if (lane == 0) inv_rms = v;
    } else if (wave == 1 + quad % (GV_WAVES - 1)) {
      // the double-precision chain goes to another SIMD from workgroup to workgroup
      const float2 cs = rope_cos_sin(fuse.rope, 0, 2 * (quad & 31) + (lane & 1));
      if (lane < 2) angles[lane] = cs;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // not for the weights under way
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    inv = inv_rms;
  }
  for (; c < chunks; c += 2 * STEP) {
    const bool has1 = c + STEP < chunks;
    if constexpr (!FUSED) {
      request(c);  // not at the end of the trip before, as below: 72B QKV of two tokens 32.3 us so, 31.3 here
    } else {
      x0[0] = scale8(x0[0], n0, inv), x1[0] = scale8(x1[0], n1, inv);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int t = 0; t < M; ++t) {
        const float s0 = dot8(w0[e], x0[t], acc[e][t]), s1 = dot8(w1[e], x1[t], s0);
        acc[e][t] = has1 ? s1 : s0;
      }
    if constexpr (FUSED)
      if (c + 2 * STEP < chunks) request(c + 2 * STEP);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int t = 0; t < M; ++t) {
      const float s = wave_sum(acc[e][t]);
      if (lane == 0) part[wave][e][t] = s;
    }
  __syncthreads();
  const int t = threadIdx.x;
  if (t >= M || t >= a.m) return;
  float y[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = ((part[0][e][t] + part[1][e][t]) + part[2][e][t]) + part[3][e][t];

  if (MODE == GEMM_PLAIN) {
    const int n = row[0];
    if (a.bias != nullptr) {
      const uint2 raw = *(const uint2*)((const bf16_t*)a.bias + n);
      y[0] += bf16lo_to_f32(raw.x), y[1] += bf16hi_to_f32(raw.x), y[2] += bf16lo_to_f32(raw.y), y[3] += bf16hi_to_f32(raw.y);
    }
    if (a.residual != nullptr) {
      const uint2 raw = *(const uint2*)((const bf16_t*)a.residual + (size_t)t * a.n + n);
      y[0] += bf16lo_to_f32(raw.x), y[1] += bf16hi_to_f32(raw.x), y[2] += bf16lo_to_f32(raw.y), y[3] += bf16hi_to_f32(raw.y);
    }
    uint2 pk;
    pk.x = (uint32_t)f32_to_bf16_rne(y[0]) | ((uint32_t)f32_to_bf16_rne(y[1]) << 16);
    pk.y = (uint32_t)f32_to_bf16_rne(y[2]) | ((uint32_t)f32_to_bf16_rne(y[3]) << 16);
    *(uint2*)((bf16_t*)a.out + (size_t)t * a.n + n) = pk;
  } else if (MODE == GEMM_QKV_ROPE) {
    const int head = quad >> 5, f0 = 2 * (quad & 31);  // f0: first of 2 rotary frequencies
    const bf16_t* bias = (const bf16_t*)a.bias + (size_t)head * 128;
    const uint32_t b0 = *(const uint32_t*)(bias + f0), b1 = *(const uint32_t*)(bias + 64 + f0);
    float lo[2] = {y[0] + bf16lo_to_f32(b0), y[1] + bf16hi_to_f32(b0)};
    float hi[2] = {y[2] + bf16lo_to_f32(b1), y[3] + bf16hi_to_f32(b1)};
    bf16_t* dst;
    int heads_dst, head_dst;
    if (head < a.h_q) dst = (bf16_t*)a.q, heads_dst = a.h_q, head_dst = head;
    else if (head < a.h_q + a.h_kv) dst = (bf16_t*)a.k_out, heads_dst = a.h_kv, head_dst = head - a.h_q;
    else dst = (bf16_t*)a.v_out, heads_dst = a.h_kv, head_dst = head - a.h_q - a.h_kv;
    if (head < a.h_q + a.h_kv) {
      float4 cs;  // (cos, sin) of f0 and f0 + 1
      if constexpr (FUSED) cs = make_float4(angles[0].x, angles[0].y, angles[1].x, angles[1].y);
      else cs = *(const float4*)(a.cos_sin + ((size_t)t * 64 + f0) * 2);
      const float c[2] = {cs.x, cs.z}, sn[2] = {cs.y, cs.w};
#pragma unroll
      for (int e = 0; e < 2; ++e) rotate_pair(lo[e], hi[e], c[e], sn[e]);
    }
    bf16_t* out_row = dst + ((size_t)t * heads_dst + head_dst) * 128;
    const uint32_t p0 = (uint32_t)f32_to_bf16_rne(lo[0]) | ((uint32_t)f32_to_bf16_rne(lo[1]) << 16);
    const uint32_t p1 = (uint32_t)f32_to_bf16_rne(hi[0]) | ((uint32_t)f32_to_bf16_rne(hi[1]) << 16);
    *(uint32_t*)(out_row + f0) = p0;
    *(uint32_t*)(out_row + 64 + f0) = p1;
    if (APPEND && head >= a.h_q) {
      const size_t row = append_row(a.append, head_dst, t);
      unsigned char* const cache = (unsigned char*)(head < a.h_q + a.h_kv ? a.append.k : a.append.v);
      if (a.append.fp8) {
        *(uint16_t*)(cache + row * 128 + f0) = (uint16_t)(bf16_to_e4m3(p0 & 0xffffu) | (bf16_to_e4m3(p0 >> 16) << 8));
        *(uint16_t*)(cache + row * 128 + 64 + f0) = (uint16_t)(bf16_to_e4m3(p1 & 0xffffu) | (bf16_to_e4m3(p1 >> 16) << 8));
      } else {
        *(uint32_t*)((bf16_t*)cache + row * 128 + f0) = p0;
        *(uint32_t*)((bf16_t*)cache + row * 128 + 64 + f0) = p1;
      }
      if (f0 == 0 && head < a.h_q + a.h_kv) append_index(a.append, head_dst, t, a.m);
    }
  } else {  // GEMM_SWIGLU: y[0], y[1] gate and y[2], y[3] up of outputs row[0], row[0] + 1
    const float o0 = y[0] / (1.f + __expf(-y[0])) * y[2], o1 = y[1] / (1.f + __expf(-y[1])) * y[3];
    *(uint32_t*)((bf16_t*)a.out + (size_t)t * d_ff + row[0]) =
        (uint32_t)f32_to_bf16_rne(o0) | ((uint32_t)f32_to_bf16_rne(o1) << 16);
  }
}

// The shapes gemm_supported admits all fit: k is a multiple of 64 (a whole number of 16-byte chunks), n a multiple of 8
// (PLAIN), of 128 per head (QKV_ROPE) or of 256 (SWIGLU), hence of 4.
bool gemv_applies(const GemmArgs& a) { return a.m <= GV_MAX_M; }

template <int MODE>
static hipError_t launch_gemv_mode(const GemmArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)(a.n / 4)), block(GV_WAVES * 64);
  if (a.m == 1) hipLaunchKernelGGL((gemv_bf16_kernel<MODE, 1, NoFusion>), grid, block, 0, s, a, NoFusion());
  else hipLaunchKernelGGL((gemv_bf16_kernel<MODE, 2, NoFusion>), grid, block, 0, s, a, NoFusion());
  return hipSuccess;
}

hipError_t launch_gemv_bf16(const GemmArgs& a, int mode, hipStream_t s) {
  if (!gemv_applies(a) || !gemm_supported(a, mode)) return hipErrorInvalidValue;
  if (a.append.k != nullptr) {  // two tokens: one is launch_gemv_fused's
    if (a.m != 2 || mode != GEMM_QKV_ROPE) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemv_bf16_kernel<GEMM_QKV_ROPE, 2, AppendFusion>), dim3((unsigned)(a.n / 4)), dim3(GV_WAVES * 64), 0, s, a,
                       AppendFusion());
    return hipSuccess;
  }
  switch (mode) {
    case GEMM_PLAIN: return launch_gemv_mode<GEMM_PLAIN>(a, s);
    case GEMM_QKV_ROPE: return launch_gemv_mode<GEMM_QKV_ROPE>(a, s);
    case GEMM_SWIGLU: return launch_gemv_mode<GEMM_SWIGLU>(a, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemv_fused(const GemmArgs& a, const GemvFusion& f, hipStream_t s) {
  if (a.m != 1 || a.append.k == nullptr || !gemm_supported(a, GEMM_QKV_ROPE)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemv_bf16_kernel<GEMM_QKV_ROPE, 1, GemvFusion>), dim3((unsigned)(a.n / 4)), dim3(GV_WAVES * 64), 0, s, a, f);
  return hipSuccess;
}

}  // namespace qp
