// Group attention without the matrix pipe: f32 and bf16 inputs, f32 arithmetic. It serves f32 (the tiny clips) and the
// layouts that the MFMA kernel does not take.
//
// A wavefront, or with few rows over a long cache the workgroup's four (SPLIT, attend_scalar_chunks), batch by batch in turn,
// own one query row (token i of query head qh). The visible keys of a row are the C cache entries of its
// KV head followed by group tokens 0..i (Sec. 3.2: pruned cache + own group, causal). A key row is spread over LPR lanes of
// 16 bytes each, so that a load instruction reads 64 / LPR whole rows; each of these lane groups runs its own online
// softmax (running max m, denominator l, this lane's slice of the weighted sum), and the groups are merged once at the end.
//
// Such calls are small: what they cost is latency, one memory round trip per batch of keys. A batch is UNROLL keys per
// lane group (32 keys at d = 64, 16 at d = 128), its K and V are requested together and one batch ahead. With one key per lane
// (every load instruction touching 64 rows, both tensors of a key one after the other, and the merge of 64 states by shuffles) the
// video of eight f32 frames of 16 tokens, 4 heads of 64, took 21.8 us, 15.3 with this kernel; 48 frames of 32 in groups of 8, 217 and 96;
// 2048 tokens of 28 heads over 10,000 entries 34.3 and 13.4 ms; 512 bf16 ones over 4,000 1762 and 896 us.
#include "qp_internal.h"

namespace qp {

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {  // x + the value of the lane that CTRL names
  return x + __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}
// Sum over aligned groups of LANES lanes, in every lane. The mirrors pair equal partial sums of the halves.
template <int LANES>
__device__ __forceinline__ float group_sum(float x) {
  static_assert(LANES == 8 || LANES == 16 || LANES == 32, "lanes per row");
  x = dpp_add<0xB1>(x);                    // quad_perm 1,0,3,2
  x = dpp_add<0x4E>(x);                    // quad_perm 2,3,0,1
  x = dpp_add<0x141>(x);                   // row_half_mirror
  if (LANES >= 16) x = dpp_add<0x140>(x);  // row_mirror
  if (LANES >= 32) x += __shfl_xor(x, 16, 64);
  return x;
}

constexpr int WAVES = 4;

// wavefronts per SIMD: with two instead of three (two registers more) the f32 kernel took 11-14 % longer
template <typename T, int D, bool SPLIT>
__global__ __launch_bounds__(WAVES * 64, sizeof(T) == 4 ? 3 : 4) void attend_scalar_kernel(AttendArgs a) {
  constexpr int PER = Elem<T>::kPer16B;  // elements per 16-byte chunk
  constexpr int LPR = D / PER;           // lanes per key row
  constexpr int GROUPS = 64 / LPR;       // keys per load instruction
  constexpr int UNROLL = 32 / PER;       // keys per lane group and batch
  constexpr int BATCH = GROUPS * UNROLL;
  constexpr int STRIDE = SPLIT ? WAVES * BATCH : BATCH;
  constexpr int FOLD = 16;               // batches

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int sub = lane % LPR, lg = lane / LPR;
  const int qh = blockIdx.y;
  const int r = a.h_q / a.h_kv;
  const int h = qh / r;
  if (a.groups > 1) {  // this workgroup's group of a run (grid.z)
    const size_t t0 = (size_t)blockIdx.z * a.n_g;
    a.q = (const T*)a.q + t0 * a.h_q * D;
    a.k = (const T*)a.k + t0 * a.h_kv * D;
    a.v = (const T*)a.v + t0 * a.h_kv * D;
    a.out = (T*)a.out + t0 * a.h_q * D;
    a.c += blockIdx.z * a.keep;
    if ((int)blockIdx.z == a.groups - 1) a.n_g = a.n_last;
  }
  const int part = SPLIT ? wave : 0;                            // this wavefront's share of the row's batches
  const int i = SPLIT ? blockIdx.x : blockIdx.x * WAVES + wave;  // group token (query row)
  if (i >= a.n_g) return;  // whole wavefront; the whole workgroup if SPLIT

  const int n_keys = a.c + i + 1;
  const T* ck = (const T*)a.ck + (size_t)h * a.cap * D + sub * PER;
  const T* cv = (const T*)a.cv + (size_t)h * a.cap * D + sub * PER;
  const T* gk = (const T*)a.k + (size_t)h * D + sub * PER;
  const T* gv = (const T*)a.v + (size_t)h * D + sub * PER;
  const size_t gstride = (size_t)a.h_kv * D;

  uint4 kr[UNROLL], vr[UNROLL];
  auto request = [&](int j0) {  // this lane's chunks of the batch of keys from j0; keys past the end: the last one again
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int j = min(j0 + u * GROUPS + lg, n_keys - 1);
      const bool cached = j < a.c;
      kr[u] = *(const uint4*)(cached ? ck + (size_t)j * D : gk + (size_t)(j - a.c) * gstride);
      vr[u] = *(const uint4*)(cached ? cv + (size_t)j * D : gv + (size_t)(j - a.c) * gstride);
    }
  };
  request(part * BATCH);
  float q[PER];
  widen16<T>(*(const uint4*)((const T*)a.q + ((size_t)i * a.h_q + qh) * D + sub * PER), q);

  float m = -INFINITY, l = 0.f;
  float acc[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.f;

  // The running sums take at most FOLD batches before they are folded into outer ones: a lane group walks 1/GROUPS of the
  // row, and one chain of that length would round more often than it did with a key per lane (32-bit rows, d = 128, unit
  // normal: relative error over 4000 / 32,000 / 128,000 entries 3.7e-7 / 9.4e-7 / 1.8e-6 in one chain, 4.5e-7 / 6.1e-7 /
  // 8.9e-7 with a key per lane, 2.0e-7 / 3.1e-7 / 4.9e-7 folded; 2000 tokens of 8 heads 767 us, 765 folded).
  float m_out = -INFINITY, l_out = 0.f, acc_out[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc_out[e] = 0.f;
  auto fold = [&]() {
    const float f = exp2f(m_out - (m == -INFINITY ? 0.f : m));
    l_out = fmaf(l_out, f, l);
#pragma unroll
    for (int e = 0; e < PER; ++e) acc_out[e] = fmaf(acc_out[e], f, acc[e]), acc[e] = 0.f;
    m_out = m;
    l = 0.f;
  };

  int batches = 0;
  for (int j0 = part * BATCH; j0 < n_keys; j0 += STRIDE) {
    uint4 vc[UNROLL];
    float s[UNROLL], mb = -INFINITY;
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      float kv[PER], dot = 0.f;
      widen16<T>(kr[u], kv);
#pragma unroll
      for (int e = 0; e < PER; ++e) dot = fmaf(q[e], kv[e], dot);
      s[u] = dot;
      vc[u] = vr[u];
    }
    if (j0 + STRIDE < n_keys) request(j0 + STRIDE);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      s[u] = group_sum<LPR>(s[u]);
      mb = fmaxf(mb, s[u] * a.scale_log2);  // a key past the end is the last one again: its logit may set the reference
    }
    const float m_new = fmaxf(m, mb);
    const float ref = m_new == -INFINITY ? 0.f : m_new;  // a lane group without a key so far: all its weights are 0
    const float alpha = exp2f(m - ref);                  // exp2(-inf) = 0 on the first keys
    m = m_new;
    // the batch is summed by itself, in pairs, so that the running sums take one addition per batch and their rounding
    // stays what it was with a key per lane
    float p[UNROLL], t[UNROLL][PER];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      // the scaled logit is not rounded before the reference is taken off
      p[u] = exp2f(fmaf(s[u], a.scale_log2, -ref));
      widen16<T>(vc[u], t[u]);
    }
    if (j0 + BATCH > n_keys) {  // the row's last batch: keys past the end weigh nothing, whatever the last one holds
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (j0 + u * GROUPS + lg >= n_keys) {
          p[u] = 0.f;
#pragma unroll
          for (int e = 0; e < PER; ++e) t[u][e] = 0.f;
        }
    }
#pragma unroll
    for (int u = 0; u < UNROLL; u += 2)
#pragma unroll
      for (int e = 0; e < PER; ++e) t[u][e] = fmaf(p[u + 1], t[u + 1][e], p[u] * t[u][e]);
#pragma unroll
    for (int w = 1; w < UNROLL; w *= 2)
#pragma unroll
      for (int u = 0; u < UNROLL; u += 2 * w) {
        p[u] += p[u + w];
        if (w > 1)
#pragma unroll
          for (int e = 0; e < PER; ++e) t[u][e] += t[u + w][e];
      }
    l = fmaf(l, alpha, p[0]);
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = fmaf(acc[e], alpha, t[0][e]);
    if (++batches % FOLD == 0) fold();
  }
  if (batches >= FOLD) {
    fold();
    l = l_out;
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = acc_out[e];
  }

  // merge the lane groups' states
  float mw = m;
#pragma unroll
  for (int o = LPR; o < 64; o <<= 1) mw = fmaxf(mw, __shfl_xor(mw, o, 64));
  const float ref = mw == -INFINITY ? 0.f : mw;  // a wavefront without keys (only beside others of its row)
  const float f = exp2f(m - ref);                // lane groups without keys: exp2(-inf) = 0
  l *= f;
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] *= f;
#pragma unroll
  for (int o = LPR; o < 64; o <<= 1) {
    l += __shfl_xor(l, o, 64);
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
  }
  T* orow = (T*)a.out + ((size_t)i * a.h_q + qh) * D;
  if constexpr (!SPLIT) {
    if (lg == 0)
#pragma unroll
      for (int e = 0; e < PER; ++e) store_elem<T>(orow + sub * PER + e, acc[e] / l);
  } else {  // and those of the row's wavefronts
    __shared__ float part_acc[WAVES][D], part_m[WAVES], part_l[WAVES];
    if (lg == 0)
#pragma unroll
      for (int e = 0; e < PER; ++e) part_acc[wave][sub * PER + e] = acc[e];
    if (lane == 0) part_m[wave] = mw, part_l[wave] = l;
    __syncthreads();
    mw = part_m[0];  // finite: the first batch has a key
#pragma unroll
    for (int w = 1; w < WAVES; ++w) mw = fmaxf(mw, part_m[w]);
    float o = 0.f;
    l = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float wgt = exp2f(part_m[w] - mw);  // 0 for a wavefront without keys
      l = fmaf(wgt, part_l[w], l);
      o = fmaf(wgt, part_acc[w][threadIdx.x % D], o);
    }
    if (threadIdx.x < D) store_elem<T>(orow + threadIdx.x, o / l);
  }
  if (a.lse != nullptr && lane == 0 && part == 0) a.lse[(size_t)qh * a.n_g + i] = (mw + log2f(l)) * 0.6931471805599453f;
}

// Rows that would leave SIMDs idle are split over a workgroup, for caches of several batches: us unsplit / split, f32 d=64,
// 4 rows over 300 entries 14.7 / 7.6, 256 over 1000 47 / 13, 800 over 1000 54 / 39, 1600 over 1000 70 / 68; with rows
// enough the wavefronts of a workgroup are better off reading the same keys: 57,344 over 10,000 12.7 / 17.4 ms.
// The split needs no scratch, but its merge changes a row's last bits, so it keeps to the rule of every key split: a call
// without scratch is not split, and a launch of qp_prefill_video's runs never is, even of one group, because there the
// groups that share a launch follow from the workspace and from the length of the video.
constexpr int SPLIT_FROM = 256;

int attend_scalar_chunks(const AttendArgs& a, size_t scratch_bytes) {
  return scratch_bytes > 0 && a.c >= SPLIT_FROM && (long)a.n_g * a.h_q <= 4 * device_cu_count() ? WAVES : 1;
}

template <typename T, int D>
static void launch_scalar(const AttendArgs& a, int chunks, hipStream_t s) {
  const unsigned groups = a.groups > 1 ? a.groups : 1;
  if (chunks > 1)
    hipLaunchKernelGGL((attend_scalar_kernel<T, D, true>), dim3(a.n_g, a.h_q), dim3(WAVES * 64), 0, s, a);
  else
    hipLaunchKernelGGL((attend_scalar_kernel<T, D, false>), dim3((a.n_g + WAVES - 1) / WAVES, a.h_q, groups), dim3(WAVES * 64), 0,
                       s, a);
}

void launch_attend_scalar(const AttendArgs& a, int dtype, int chunks, hipStream_t s) {
  if (dtype == QP_F32) a.d == 64 ? launch_scalar<float, 64>(a, chunks, s) : launch_scalar<float, 128>(a, chunks, s);
  else a.d == 64 ? launch_scalar<bf16_t, 64>(a, chunks, s) : launch_scalar<bf16_t, 128>(a, chunks, s);
}

}  // namespace qp
