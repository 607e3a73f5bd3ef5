// Rows of the cache as the kernels that append to it write them.
#pragma once
#include "fp8_e4m3.h"
#include "qp_internal.h"

namespace qp {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 8 bf16 values (16 bytes) as 8 E4M3 codes (the 8-bit cache's rows)
__device__ __forceinline__ uint2 pack8_e4m3(const u32x4& b) {
  uint2 r;
  r.x = bf16_to_e4m3(b.x & 0xffffu) | (bf16_to_e4m3(b.x >> 16) << 8) | (bf16_to_e4m3(b.y & 0xffffu) << 16) |
        (bf16_to_e4m3(b.y >> 16) << 24);
  r.y = bf16_to_e4m3(b.z & 0xffffu) | (bf16_to_e4m3(b.z >> 16) << 8) | (bf16_to_e4m3(b.w & 0xffffu) << 16) |
        (bf16_to_e4m3(b.w >> 16) << 24);
  return r;
}

// Token t of KV head h in the cache: its row, and what goes with it
__device__ __forceinline__ size_t append_row(const CacheAppend& a, int h, int t) { return (size_t)h * a.cap + a.len + t; }
__device__ __forceinline__ void append_index(const CacheAppend& a, int h, int t, int n) {
  a.pos[append_row(a, h, t)] = a.base + t;
  if (a.kept != nullptr) a.kept[(size_t)h * n + t] = t;
}
// 8 (4) elements of it, at dimension dim of a key (or value)
__device__ __forceinline__ void append_chunk(const CacheAppend& a, bool is_v, int h, int t, int dim, const u32x4& b) {
  const size_t at = append_row(a, h, t) * 128 + dim;
  void* const cache = is_v ? a.v : a.k;
  if (a.fp8) *(uint2*)((unsigned char*)cache + at) = pack8_e4m3(b);
  else *(u32x4*)((bf16_t*)cache + at) = b;
}
__device__ __forceinline__ void append_run(const CacheAppend& a, bool is_v, int h, int t, int dim, const uint2& b) {
  const size_t at = append_row(a, h, t) * 128 + dim;
  void* const cache = is_v ? a.v : a.k;
  if (a.fp8) *(uint32_t*)((unsigned char*)cache + at) = pack8_e4m3(u32x4{b.x, b.y, 0u, 0u}).x;
  else *(uint2*)((bf16_t*)cache + at) = b;
}

}  // namespace qp
