// bf16 MFMA group attention for gfx950 (head_dim 128), flash-style.
//
// What it computes (Sec. 3.2 of the paper, group-based prefill): for query head qh of KV head
// h = qh / R and group token t, softmax over {cache entries 0..C-1 of h} U {group tokens 0..t}
// of scale * q.k, times V.
//
// Mapping. The R query heads that share a KV head are stacked into one row space per KV head:
// row r = t * R + j (j = query head inside the KV group), which is also the memory order of
// Q_g[t][h*R + j][:]. A workgroup of 8 wavefronts owns 256 rows of one KV head; every K/V tile it
// stages in LDS is shared by all R query heads (GQA). Two row mappings, chosen by the launcher:
//   * more workgroups than CUs: 256 consecutive rows each, latest tokens (longest key range) first,
//     so that the short workgroups fill the tail of the launch;
//   * at most one workgroup per CU (all resident at once, the launch lasts as long as its longest
//     workgroup): two half blocks of 128 consecutive rows each, one from the early end of the group
//     and its mirror from the late end, so that all workgroups carry the same causal work.
// The keys are walked as two segments, cache tiles first and then group tiles starting
// at group token 0, so a tile never straddles the two sources; only the cache's last tile and the
// group's diagonal tiles are masked, and a wavefront skips group tiles beyond its causal horizon.
// Key split: the cache tiles of a row block can be dealt to several workgroups (chunks), each leaving a normalised
// partial output and its log-sum-exp for a merge launch. The planner splits every row block when few rows meet a
// long cache (so that the launch covers the chip), and, in launches of several rounds of workgroups, only the row
// blocks of a partly filled last round (so that their chunks fill the compute units evenly); see plan_attend_mfma.
//
// Per wavefront (32 rows), per block of 32 keys, with v_mfma_f32_32x32x16_bf16:
//   S^T[key][row] = K_block . Q^T     (A = K from LDS, 16-byte reads; B = Q held in registers)
//     -> a lane holds ONE row (column of S^T) and 16 of the block's keys, lane l + 32 the other 16.
//   P^T = exp2(c*S^T - c*m) rounded to bf16, fed straight back as the B operand of
//   O^T[d][row] += V^T . P^T         (A = V^T read from the row-major V tile in LDS with the
//                                      transposing ds_read_tr16_b64, 4 keys x 16 d per 16 lanes)
//     -> O^T keeps the lane <-> row association, so a rescale is a per-lane scalar multiply.
// The contraction index of the second product is permuted (keys 4g..4g+3 and 8+4g..8+4g+3 of
// each 16-key step go to lane half g) so that the accumulator layout of S^T is already the
// operand layout of P^T; V^T is read with the same permutation.
//
// Schedule. What bounds the loop is the matrix pipe (64 products of 32 cycles per SIMD and tile, and 16 small ones of 8 for the
// row sums, 6 % more) and, at full occupancy, the power that the products and their operands cost: the chip lowers its clock. The loop is software-pipelined over three
// consecutive blocks: one step issues S^T of block j+1, the numerators of block j and O^T += V^T P^T of block j-1, none
// of which waits for another, in a fixed order of 16 products with two vector operations and an exponential or so behind
// each, and fragments read three products ahead. For that the numerators must not wait for the block's max:
//   * The reference m of a row is not the running max. It moves only when a block's numerators outgrow it (a lane's sum of
//     16 beyond 2^6, infinity included), checked after they are formed and before they are used; the block's numerators are
//     then formed again around the new max, of both blocks of a tile if it is the first. The row's first tile sets it. The
//     range of bf16 and f32 would allow a reference far below the max, but the max itself is then rounded to bf16, where
//     around itself it is an exact 1, and of a sharp row it is most of the sum: see MF_RESCALE.
//   * The row sum of the bf16-rounded numerators is taken by four small products with ones (add_four).
// 8192 tokens of the 7B heads over 24,576 entries, random (all-zero, which leaves the clock alone) inputs: 2727 us (1967), with
// the row sums by vector adds on the same card 2764 (1952). With those, on an earlier card: 2945 us (2000);
// one tile after the other with max, numerators and v_dot2 sum between the two products 3240 (2590); that pipeline with the
// v_dot2 sum and all requests behind the barrier 3220 (2500). Products in fours per kind: alternating one by one costs 1 %.
//   * K/V tiles go global -> LDS with global_load_lds_dwordx4 (no staging registers, no ds_write):
//     one instruction moves 64 lanes x 16 bytes into 1 KB of LDS, lane L landing at base + 16 L.
//     Rows are 256 bytes, unpadded; bank conflicts are avoided by an XOR swizzle of the 16-byte
//     chunk index: K chunk c of key k sits at position c ^ (k & 15), V chunk c at position
//     c ^ ((k & 7) << 1); each lane fetches the global chunk that belongs at its LDS position.
//   * Tiles of 64 keys sit in rings of four LDS slots and are requested more than two tiles ahead, one barrier per tile, the
//     wavefront's four requests spread over a step (issued together behind the barrier they cost 10 %, all-zero 15 %).
//   * Workgroup ids are mapped so that the workgroups of one KV head run on the same XCDs (ids are
//     dealt round-robin over the 8 XCDs, each with its own L2): with 4 KV heads, XCDs 2h and 2h+1
//     serve head h, so every L2 streams one head's K/V instead of all of them.
#include "qp_internal.h"

#include <float.h>

#include <algorithm>

namespace qp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

constexpr int MF_D = 128;               // head_dim
constexpr int MF_BN = 64;               // keys per tile
constexpr int MF_NW = 8;                // wavefronts per workgroup
constexpr int MF_NT = MF_NW * 64;
constexpr int MF_HB = MF_NW / 2 * 32;   // rows per half block (4 wavefronts); a workgroup owns two half blocks
constexpr int MF_TILE = MF_BN * 256;    // bytes of one K or V tile (unpadded, swizzled)
constexpr int MF_STAGES = 4;            // ring slots of K and of V tiles
constexpr int MF_V0 = MF_STAGES * MF_TILE;  // LDS offset of the V ring
constexpr int MF_LDS = 2 * MF_STAGES * MF_TILE;
// Move the reference when a lane's 16 numerators of a block sum to more. Relative error against 64 bits (512 tokens of the
// 7B heads over 8192 entries, unit-normal keys, queries scaled by 1 / 2 / 4 / 8), by the limit: 2^12 2.34e-3 / 2.26 / 1.91 /
// 1.73, 2^8 2.34 / 2.23 / 1.85 / 1.70, 2^6 2.34 / 2.16 / 1.81 / 1.69; a max per tile that moves it by 2^8 and more 2.34 /
// 2.23 / 1.82 / 1.71. What it costs: 4096 tokens over 24,576 entries 1293 / 1328 / 1384 / 1420 us, with 2^12 1294 / 1316 /
// 1348 / 1388; 77 tokens over 9840 29.0 / 30.2 / 32.3 / 33.0 and 29.1 / 28.9 / 30.2 / 32.9.
constexpr float MF_RESCALE = 64.f;
// Up to so many rows of a KV head a chunk's partial rows are stored from the accumulators: for one to three live wavefronts the
// barrier and the way through LDS take longer than what whole rows save. us of the call from the accumulators / through LDS:
// 7B heads, 5 tokens (35 rows) over 600, 5,000 and 20,000 entries 11.9 / 12.6, 12.5 / 13.1, 16.4 / 17.1; 9 tokens over 5,000
// 13.8 / 14.1, 11 tokens 15.2 / 15.4, 14 (98 rows) 16.4 / 16.2, 18 17.5 / 17.1; 72B heads, 5 tokens (40 rows) over 5,000 14.4 / 15.0.
// With more than a tile of tokens, which so few rows have only where every query head has keys of its own, four live wavefronts
// are stored so too: of the last chunk they end at their horizons, and the barrier would hold them until the last has ended. 16 such
// heads, 100 tokens over 600 and 5,000 entries 14.7 / 15.5, 21.0 / 21.7, 128 over 600 15.3 / 15.7, over 20,000 39.1 / 38.7.
constexpr int MF_DIRECT_ROWS = 96;
constexpr int MF_VMCNT0 = 0x0f70;       // s_waitcnt vmcnt(0), other counters untouched
constexpr int MF_VMCNT4 = 0x0f74;       // s_waitcnt vmcnt(4)
constexpr int MF_LGKM0 = 0xc07f;        // s_waitcnt lgkmcnt(0)
constexpr int MF_SPLIT_BELOW = 128;     // launches of fewer workgroups split the cache over chunks
constexpr int MF_MAX_SPLIT = 128;       // chunks at most
constexpr size_t MF_SPLIT_ALL_BYTES = (size_t)32 << 20;  // scratch that a split of every row block takes at most
constexpr int MF_TAIL_SPLIT_MAX = 8;    // chunks per row block when only the last round's row blocks are split
constexpr int MF_TAIL_MIN_TILES = 16;   // ... whose chunks hold at least this many cache tiles

// Masks S^T of one 32-key block: this lane's keys beyond `lim` (block-local, minus 4 g) become -inf.
__device__ __forceinline__ void mask_block(f32x16& st, int lim) {
#pragma unroll
  for (int r = 0; r < 16; ++r) st[r] = 8 * (r >> 2) + (r & 3) > lim ? -INFINITY : st[r];
}

// Two numerators, rounded to bf16, as elements i and i + 1 of a P^T operand.
__device__ __forceinline__ void pack_pair(float e0, float e1, bf16x8& p, int i) {
  p[i] = (__bf16)e0;
  p[i + 1] = (__bf16)e1;
}
// Adds four rounded numerators of this lane (elements 4 hi .. 4 hi + 3 of a P^T operand) to sum, in every element of it. Of
// the 4x4x4 product's 16 independent blocks, lane l holds all four contraction elements of column l & 3 of block l >> 2 and
// gets that column of the result: with ones as the other operand, its own sum. It takes the matrix pipe 8 cycles; shifts
// and adds took 16 of the vector pipe for each pair of numerators, and 44 % of a step's vector instructions. At full
// occupancy the kernel is bound by power, so instructions that are gone are time: 512 frames of 256 tokens through the 72B heads
// 62150 -> 60920 us, 1024 of 128 through the 7B heads 22580 -> 22080, 256 of them 2348 -> 2294, 99 of 121 tokens over an 8-bit
// cache 520 -> 503; but 77 tokens of 32 heads (8 of keys) over 46,000 and 100,000 entries, three half blocks of rows, 77.8 -> 78.8 and
// 168 -> 173: the lone one runs further ahead of its partner than the L2 holds. (v_dot2_f32_bf16, two numerators each, holds the matrix pipe for 16 cycles.)
__device__ __forceinline__ f32x4 add_four(const bf16x8& p, int hi, f32x4 sum) {
  const s16x8 all = __builtin_bit_cast(s16x8, p);
  const s16x4 part = hi ? __builtin_shufflevector(all, all, 4, 5, 6, 7) : __builtin_shufflevector(all, all, 0, 1, 2, 3);
  const s16x4 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
  return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, part, sum, 0, 0, 0);
}

struct Pieces {
  uint2 p[4];
};
// 8 E4M3 bytes -> 8 bf16 (exact)
__device__ __forceinline__ u32x4 widen8(uint2 p) {
  u32x4 o;
  o.x = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(p.x, 1.f, false));
  o.y = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(p.x, 1.f, true));
  o.z = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(p.y, 1.f, false));
  o.w = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(p.y, 1.f, true));
  return o;
}

struct true_type { static constexpr bool value = true; };
struct false_type { static constexpr bool value = false; };

// F8: the cache's K~ and V~ hold one E4M3 byte per element (the pruned cache's 8-bit format). Their tiles cannot go
// global -> LDS directly: every wavefront loads its share of a tile into registers one tile ahead (8 bytes per lane
// and row), widens it exactly to bf16 and writes it to the ring slot in the same swizzled layout, so that everything
// after the staging is the same code. The group's own tiles are bf16 and staged as usual.
template <bool F8>
__global__ __launch_bounds__(MF_NT, 2) void attend_mfma_kernel(AttendArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform for the compiler too: scalar address and branch work
  const int l32 = lane & 31, g = lane >> 5;
  const int r_heads = a.h_q / a.h_kv;
  int n_rows = a.n_g * r_heads;
  int n_hb = (n_rows + MF_HB - 1) / MF_HB;  // half blocks of 128 rows
  int n_rb = (n_hb + 1) / 2;                // workgroups per KV head (256 rows or a pair of half blocks)
  // Work items of a KV head: the row blocks that one workgroup serves whole (longest first), then the chunks of the
  // split row blocks (the shortest ones), chunk by chunk.
  const int n_whole = n_rb - (a.n_split > 1 ? a.split_rb : 0);
  int n_items = n_whole + (n_rb - n_whole) * a.n_split;
  // A run of groups is never split: its items are the row blocks of the last group (longest key range), then those of
  // the group before it, and so on.
  const int n_rb_last = a.groups > 1 ? ((a.n_last * r_heads + MF_HB - 1) / MF_HB + 1) / 2 : 0;
  if (a.groups > 1) n_items = n_rb_last + (a.groups - 1) * n_rb;
  // workgroup id -> (KV head, item): ids go round-robin over the 8 XCDs
  int h, item;
  {
    const int wg = blockIdx.x, xcd = wg & 7, idx = wg >> 3;
    if (8 % a.h_kv == 0) {
      const int per = 8 / a.h_kv;  // XCDs per KV head
      h = xcd / per;
      item = idx * per + (xcd % per);
      // Dealt one by one, the two row blocks of a text chunk each took a copy of the cache through an L2 of their own: both
      // of a key chunk go to one XCD, whose L2 then fetches its keys once. us before / after, 7B heads: 64 tokens over 60,000
      // entries 69.6 / 66.5, 50 tokens 64.8 / 60.1, 64 over 30,000 45.0 / 43.6, over 20,000 (chunks of 10 tiles) 36.5 / 34.8.
      // Shorter chunks are not bound by the fetch (64 over 9,840, 5 tiles: 28.6 / 28.8), nor are those of an 8-bit cache, half
      // as large, up to 13 tiles (40 and 50 tokens over 20,000, 10 tiles: 31.4 / 33.0 and 33.7 / 34.4; 50 over 25,000, 13 tiles:
      // 37.5 / 37.5; 50 over 30,000 and 46,125: 40.7 / 40.0 and 51.3 / 50.3), and of three row blocks and more,
      // side by side, chunks got slower (200 over 5,000 31.4 / 34.1, 128 over 9,840 33.5 / 34.2).
      // Chunks that do not divide among the head's XCDs would need a larger grid, which has not been tried: one by one, as before.
      if (n_whole == 0 && n_rb == 2 && a.split_tiles >= (F8 ? 14 : 10) && a.n_split % per == 0) item = (idx / 2 * per + xcd % per) * 2 + idx % 2;
    } else if (a.h_kv % 8 == 0) {
      const int hp = a.h_kv / 8;  // KV heads per XCD
      h = (idx % hp) * 8 + xcd;
      item = idx / hp;
    } else {
      h = wg % a.h_kv;
      item = wg / a.h_kv;
    }
  }
  if (item >= n_items) return;    // padding workgroups of the XCD mapping (whole workgroup, before any barrier)
  const int tokens = a.n_g;  // of a full group
  size_t t0 = 0;             // first token of this item's group
  int rbi = item, chunk = 0, my_split = 1;  // row block (0 = latest tokens), key chunk, chunks of this row block
  if (a.groups > 1) {  // from here on: this item's group
    int grp = a.groups - 1;
    if (item < n_rb_last) {
      a.n_g = a.n_last;
      n_rows = a.n_g * r_heads;
      n_hb = (n_rows + MF_HB - 1) / MF_HB;
      n_rb = n_rb_last;
    } else {
      const int e = item - n_rb_last, back = e / n_rb;
      grp -= 1 + back;
      rbi = e - back * n_rb;
    }
    a.c += grp * a.keep;
    t0 += (size_t)grp * tokens;
  } else if (item >= n_whole) {
    const int e = item - n_whole, n_sp = n_rb - n_whole;
    chunk = e / n_sp;
    rbi = n_whole + (e - chunk * n_sp);
    my_split = a.n_split;
  }
  // Mirrored mapping: the workgroup owns half block rbi (early tokens, short key range) and its mirror
  // n_hb-1-rbi (late tokens, long key range). Wavefronts 0..3 take the early half block and 4..7 the late one:
  // wavefronts w and w+4 share a SIMD, so each SIMD keeps one wavefront busy after the early rows have reached
  // their causal horizon. Consecutive mapping: half blocks 2 rb and 2 rb + 1 with rb counted from the late end.
  const int half = wave >> 2;
  const int hb_late = a.mirrored ? n_hb - 1 - rbi : min(2 * (n_rb - 1 - rbi) + 1, n_hb - 1);
  const int hb_early = a.mirrored ? rbi : 2 * (n_rb - 1 - rbi);
  const int hb = half ? hb_late : hb_early;
  const bool unpaired = half == 0 && hb_early == hb_late;  // odd count: that half block is served as "late" only
  const int row0 = hb * MF_HB + (wave & 3) * 32;
  const int row = row0 + l32;
  const bool row_ok = row < n_rows;
  const int rowc = row_ok ? row : n_rows - 1;
  const int t_lane = rowc / r_heads;
  const int j_lane = rowc - t_lane * r_heads;
  const bf16_t* qrow = (const bf16_t*)a.q + ((t0 + t_lane) * a.h_q + (size_t)h * r_heads + j_lane) * MF_D;
  // wave-uniform token horizons
  const int t_w_max = min(row0 + 31, n_rows - 1) / r_heads;
  const int t_w_min = min(row0, n_rows - 1) / r_heads;
  const int t_wg_max = min(hb_late * MF_HB + MF_HB - 1, n_rows - 1) / r_heads;
  const bool wave_live = row0 < n_rows && !unpaired;
  const int n_ct = (a.c + MF_BN - 1) / MF_BN;       // cache tiles
  const int n_tiles = n_ct + t_wg_max / MF_BN + 1;  // + group tiles
  // key split: a chunk walks cache tiles [t_begin, t_end); the last chunk goes on through the group tiles
  const int t_begin = chunk * a.split_tiles;
  const int t_end = chunk == my_split - 1 ? n_tiles : t_begin + a.split_tiles;

  constexpr int CROW = F8 ? MF_D : MF_D * 2;  // bytes of one cached row
  const unsigned char* ck = (const unsigned char*)a.ck + (size_t)h * a.cap * CROW;
  const unsigned char* cv = (const unsigned char*)a.cv + (size_t)h * a.cap * CROW;
  const unsigned char* gk = (const unsigned char*)a.k + (t0 * a.h_kv + h) * (MF_D * 2);
  const unsigned char* gv = (const unsigned char*)a.v + (t0 * a.h_kv + h) * (MF_D * 2);
  const unsigned gstride_b = (unsigned)a.h_kv * (MF_D * 2);

  // staging: this wavefront's two load instructions per tensor cover keys 8*wave .. 8*wave+7 of the tile;
  // LDS position (lane & 15) of key row (lane >> 4) <- the global chunk position ^ swizzle(key)
  const int st_key0 = 8 * wave + (lane >> 4), st_key1 = st_key0 + 4;
  const int st_pos = lane & 15;
  const unsigned st_kc0 = (unsigned)((st_pos ^ (st_key0 & 15)) * 16), st_kc1 = (unsigned)((st_pos ^ (st_key1 & 15)) * 16);
  const unsigned st_vc0 = (unsigned)((st_pos ^ ((st_key0 & 7) << 1)) * 16),
                 st_vc1 = (unsigned)((st_pos ^ ((st_key1 & 7) << 1)) * 16);
  const unsigned st_lds = lds_address(smem) + wave * 2048;  // this wavefront's 2 x 1 KB inside a tile

  // One tensor's tile requests, in order: the next tile, its address, and this lane's byte offsets of its two rows in it.
  // The offsets change only where a segment starts or a tile is cut off by its segment's end (rows past the end are
  // clamped: masked, never used); `event` is the next such tile.
  struct Stream {
    const unsigned char* src;
    unsigned o0, o1, step;
    int tile, event;
  };
  const int cache_tail = a.c % MF_BN != 0 ? n_ct - 1 : -1;
  const int group_tail = a.n_g % MF_BN != 0 ? n_ct + a.n_g / MF_BN : -1;
  auto settle = [&](Stream& s, const unsigned char* cache, const unsigned char* group, unsigned c0, unsigned c1) {
    const bool in_cache = s.tile < n_ct;
    const int first = (in_cache ? s.tile : s.tile - n_ct) * MF_BN;
    const int left = (in_cache ? a.c : a.n_g) - first - 1;  // last valid row of the tile
    const unsigned stride = in_cache ? (unsigned)CROW : gstride_b;
    const int sh = F8 && in_cache ? 1 : 0;  // 8 bytes of an 8-bit row where a bf16 row has 16
    s.src = (in_cache ? cache : group) + (size_t)first * stride;
    s.step = MF_BN * stride;
    s.o0 = __umul24((unsigned)min(st_key0, left), stride) + (c0 >> sh);
    s.o1 = __umul24((unsigned)min(st_key1, left), stride) + (c1 >> sh);
    const int tail = in_cache ? cache_tail : group_tail;
    s.event = s.tile < tail ? tail : in_cache ? n_ct : 0x7fffffff;
  };
  auto advance = [&](Stream& s, const unsigned char* cache, const unsigned char* group, unsigned c0, unsigned c1) {
    s.src += s.step;
    if (++s.tile >= s.event && s.tile < t_end) settle(s, cache, group, c0, c1);
  };
  Stream sk, sv;
  sk.tile = sv.tile = t_begin;
  settle(sk, ck, gk, st_kc0, st_kc1);
  settle(sv, cv, gv, st_vc0, st_vc1);
  // A pair's four requests: halves of its K tile (0, 1) and of its V tile (2, 3). Tiles of an 8-bit cache cannot go to LDS
  // directly: this lane's 8 bytes of each half are pending in registers until they are stored, widened.
  Pieces pend;
  auto load_piece = [&](int i) {
    const Stream& s = i < 2 ? sk : sv;
    return *(const uint2*)(s.src + ((i & 1) ? s.o1 : s.o0));
  };
  auto request_half = [&](int i, unsigned dst) {  // dst: LDS address of the slot's K tile
    const Stream& s = i < 2 ? sk : sv;
    lds_dma16_to(s.src, (i & 1) ? s.o1 : s.o0, dst + (i < 2 ? 0 : MF_V0) + (i & 1) * 1024);
  };
  auto store_piece = [&](int i, uint2 p, int slot) {
    *(u32x4*)(smem + slot * MF_TILE + (i < 2 ? 0 : MF_V0) + (i & 1) * 1024 + wave * 2048 + lane * 16) = widen8(p);
  };
  auto request_k = [&](int slot) {
    if (F8 && sk.tile < n_ct) pend.p[0] = load_piece(0), pend.p[1] = load_piece(1);
    else request_half(0, st_lds + slot * MF_TILE), request_half(1, st_lds + slot * MF_TILE);
  };
  auto request_v = [&](int slot) {
    if (F8 && sv.tile < n_ct) pend.p[2] = load_piece(2), pend.p[3] = load_piece(3);
    else request_half(2, st_lds + slot * MF_TILE), request_half(3, st_lds + slot * MF_TILE);
  };
  auto store_k = [&](int tile, const Pieces& p, int slot) {  // if `tile` is a tile of an 8-bit cache
    if (F8 && tile < n_ct) store_piece(0, p.p[0], slot), store_piece(1, p.p[1], slot);
  };
  auto store_v = [&](int tile, const Pieces& p, int slot) {
    if (F8 && tile < n_ct) store_piece(2, p.p[2], slot), store_piece(3, p.p[3], slot);
  };

  // fragment read addresses (bytes inside a tile)
  const unsigned lds0 = lds_address(smem);
  unsigned k_addr[8];  // K fragment of d-step s: key l32 (+32 per block), chunk 2s+g at position (2s+g) ^ (l32 & 15)
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    k_addr[s] = lds0 + l32 * 256 + (((2 * s + g) ^ (l32 & 15)) << 4);
    asm("" : "+v"(k_addr[s]));  // opaque: ring offsets stay immediates of the reads instead of more address registers
  }
  const int l16 = lane & 15, grp = lane >> 4;
  const int v_key = 4 * (grp >> 1) + (l16 >> 2);  // key inside a 16-key step (second read: + 8)
  unsigned v_addr[4];  // V^T fragment of d-block n: chunk 4n + 2(grp&1) + ((l16&3)>>1), half (l16&1)
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    v_addr[n] = lds0 + MF_V0 + v_key * 256 + (((4 * n + 2 * (grp & 1) + ((l16 & 3) >> 1)) ^ ((v_key & 7) << 1)) << 4) +
                (l16 & 1) * 8;
    asm("" : "+v"(v_addr[n]));
  }
  // fragment s of the 32-key K block / (ks, n) = (s >> 2, s & 3) of the 32-key V block at LDS offset `off`
  auto read_k = [&](int off, int s) { return __builtin_bit_cast(bf16x8, *(const lds_u32x4*)(k_addr[s] + off)); };
  auto read_v = [&](int off, int s) {
    const unsigned p0 = v_addr[s & 3] + (off + (s >> 2) * (16 * 256));
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p0));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p0 + 8 * 256));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  f32x16 o[4];
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[n][r] = 0.f;
  float m_run = -INFINITY;  // reference of the row's numerators: the max of the raw logits when it was last moved
  float l_run = 0.f;        // this lane's share of the row's denominator
  const float c2 = a.scale_log2;
  float nmc = 0.f;  // -m_run * c2

  // Moves the reference to the rows' max including this block, rescales what was summed so far and forms the block's
  // numerators (first block of a row, and blocks whose numerators outgrew the reference). look: the max of the tile's other
  // block is taken too, so that it does not move the reference once more (64 tokens over 46,125 entries, queries scaled by
  // 16: 69.9 -> 64.9 us).
  auto move_reference = [&](const f32x16& st, const f32x16& other, bool look, bf16x8 (&pf)[2], float& psum) {
    float mx = st[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, st[r]);
    if (look) {
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, other[r]);
    }
    // finite also where every logit so far is -inf: the numerators are 0 then, and the next finite logit moves it again
    mx = fmaxf(fmaxf(m_run, max_halves(mx)), -FLT_MAX);
    const float alpha = __builtin_amdgcn_exp2f((m_run - mx) * c2);
    m_run = mx;
    nmc = -mx * c2;
    l_run *= alpha;
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[n][r] *= alpha;
    f32x4 ps = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      pack_pair(__builtin_amdgcn_exp2f(fmaf(st[r], c2, nmc)), __builtin_amdgcn_exp2f(fmaf(st[r + 1], c2, nmc)), pf[r >> 3], r & 7);
      if (r & 2) ps = add_four(pf[r >> 3], (r >> 2) & 1, ps);
    }
    psum = ps[0];
  };

  bf16x8 kf[4], vf[4];  // fragments under way: three ahead of the products
  bf16x8 qf[8];
  // One step of the pipeline on three consecutive 32-key blocks: S^T of the next one (QK), numerators of the current one,
  // O^T += V^T P^T of the previous one. QK: the step has a next block. K_CUR / K_NEXT: LDS offsets of the K block being
  // read and of the one after it (likewise V); SECOND: the step works on a tile's second blocks (QK) and its last reads
  // belong to the next ring slot. `cut`: the next block will be masked, so a moving reference does not look at it (SECOND
  // only: in the other steps that block belongs to the next tile). `extra(s)` runs between the products.
  auto step = [&](auto qk, auto second, f32x16& s_next, const f32x16& s_cur, const bf16x8 (&p_prev)[2], bf16x8 (&p_cur)[2],
                  unsigned turn_mask, bool cut, auto extra) {
    constexpr bool QK = decltype(qk)::value, SECOND = decltype(second)::value;
    constexpr int CUR = SECOND ? 32 * 256 : 0, NEXT = SECOND ? 0 : 32 * 256;
    float e0 = 0.f, e1 = 0.f;
    f32x16 sn;
#pragma unroll
    for (int r = 0; r < 16; ++r) sn[r] = 0.f;
    float t0 = fmaf(s_cur[0], c2, nmc), t1 = fmaf(s_cur[1], c2, nmc);
    auto pack = [&](int s) { pack_pair(e0, e1, p_cur[s >> 2], 2 * (s & 3)); };
    auto do_qk = [&](int s) {
      if (QK) {
        sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s & 3], qf[s], sn, 0, 0, 0);
        if (SECOND && s >= 5) k_addr[s - 5] ^= turn_mask;
        kf[(s + 3) & 3] = s + 3 < 8 ? read_k(CUR, s + 3) : read_k(NEXT, s - 5);
      }
    };
    auto do_pv = [&](int s) {
      o[s & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s & 3], p_prev[s >> 2], o[s & 3], 0, 0, 0);
      if (SECOND && s >= 5) v_addr[s - 5] ^= turn_mask;
      vf[(s + 3) & 3] = s + 3 < 8 ? read_v(CUR, s + 3) : read_v(NEXT, s - 5);
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int s = i >> 1, f = (i >> 3) * 4 + (i & 3);  // products in fours: QK 0..3, PV 0..3, QK 4..7, PV 4..7
      if (i & 4) do_pv(f);
      else do_qk(f);
      if (i & 1) {
        e1 = __builtin_amdgcn_exp2f(t1);
        if (s < 7) t1 = fmaf(s_cur[2 * s + 3], c2, nmc);
        extra(s);
      } else {
        if (s > 0) pack(s - 1);
        e0 = __builtin_amdgcn_exp2f(t0);
        if (s < 7) t0 = fmaf(s_cur[2 * s + 2], c2, nmc);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (SECOND) {
#pragma unroll
      for (int s = 3; s < 8; ++s) k_addr[s] ^= turn_mask;
      v_addr[3] ^= turn_mask;
    }
    pack(7);
    if (QK) s_next = sn;
    // behind the step's products: as soon as four were ready, the sums cost 0.3-1 % more
    f32x4 ps0 = {0.f, 0.f, 0.f, 0.f}, ps1 = ps0;
    ps0 = add_four(p_cur[0], 0, ps0);
    ps1 = add_four(p_cur[0], 1, ps1);
    ps0 = add_four(p_cur[1], 0, ps0);
    ps1 = add_four(p_cur[1], 1, ps1);
    float psum = ps0[0] + ps1[0];
    if (__any(psum > MF_RESCALE)) move_reference(s_cur, sn, QK && SECOND && !cut, p_cur, psum);
    l_run += psum;
  };

  // Tiles of this workgroup: n of them from t_begin. Pair p = (V of tile p, K of tile p + 1), counted from t_begin, sits in
  // ring slot p & 3; the K of tile 0 in slot 3.
  const int n = t_end - t_begin;
  // Between the two steps of iteration `it`: pair it + 1 becomes visible to all wavefronts, and with it the slot of pair
  // it - 1, which every wavefront has left, is free. Each pair is 4 requests per wavefront (the last one 2).
  auto turn = [&](int it) {
    if (it + 1 >= n) return;
    if (it + 3 < n) __builtin_amdgcn_s_waitcnt(MF_VMCNT4);
    else __builtin_amdgcn_s_waitcnt(MF_VMCNT0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // Widened pieces of pair p go to its slot: the slot's last readers passed the barrier before last. They are visible two
  // barriers later; this wavefront's LDS operations complete in order, so its writes are done when fragments that it
  // requested after them have arrived.
  auto store_pending = [&](int p) {
    if (F8 && p + 1 < n) store_k(t_begin + p + 1, pend, p & 3);
    if (F8 && p < n) store_v(t_begin + p, pend, p & 3);
  };
  auto advance_both = [&]() {
    advance(sk, ck, gk, st_kc0, st_kc1);
    advance(sv, cv, gv, st_vc0, st_vc1);
  };
  // All requests of pair p, as far as its tiles exist.
  auto request = [&](int p) {
    if (p + 1 < n) request_k(p & 3);
    if (p < n) request_v(p & 3);
    advance_both();
  };

  // Masked tiles: the cache's last one if cut off, and the group's from this wavefront's diagonal on.
  const int diag_tile = n_ct + (t_w_min + 1) / MF_BN;  // first with keys beyond t_w_min
  auto masked = [&](int tile) { return tile == cache_tail || tile >= diag_tile; };
  auto mask = [&](f32x16& st, int tile, int kb) {
    const int lim = tile < n_ct ? a.c - 1 - tile * MF_BN : t_lane - (tile - n_ct) * MF_BN;
    mask_block(st, lim - 32 * kb - 4 * g);
  };
  const bool late = my_split > 1 && a.split_tiles > 2;  // the second and third pair are requested behind the first wait
  // this wavefront's last tile (relative; -1: no rows)
  const int last = wave_live ? min(n, n_ct + t_w_max / MF_BN + 1 - t_begin) - 1 : -1;

#pragma unroll
  for (int s = 0; s < 8; ++s) qf[s] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qrow + 16 * s + 8 * g));
  request_k(3);
  advance(sk, ck, gk, st_kc0, st_kc1);
  if (F8) {
    // tiles go through registers one after the other; pair 2 stays pending
    const Pieces first = pend;
    request(0);
    const Pieces p0 = pend;
    request(1);
    const Pieces p1 = pend;
    request(2);
    store_k(t_begin, first, 3);
    if (n > 1) store_k(t_begin + 1, p0, 0);
    store_v(t_begin, p0, 0);
    if (n > 2) store_k(t_begin + 2, p1, 1);
    if (n > 1) store_v(t_begin + 1, p1, 1);
  } else {
    request(0);
    if (!late) {
      request(1);
      request(2);
    }
  }
  // Everything requested so far has to be here: from now on the only vector-memory operations in flight are the tile
  // requests, which the compiler does not see.
  __builtin_amdgcn_s_waitcnt(MF_VMCNT0);
  __syncthreads();
  // The first products need no more than that. In a chunk of a split launch, which is short and starts together with all
  // others, the next pairs are requested behind the wait and awaited in the loop; a whole row block has them requested in
  // front of it, where the requests hold no products up. us requested in front / behind: chunks, 64 tokens of the 7B heads over
  // 46,125 entries 59.6 / 58.5, 10 over 100,000 40.4 / 39.7, 77 over 9,840 31.3 / 31.0, 64 of the 72B heads over 5,000 28.7 /
  // 28.3; chunks of two tiles, which need them at once, 5 over 600 11.3 / 11.7; whole row blocks, 3600 frames of 128 tokens in groups of 64 150660 / 150980, 512 of 256 in groups of 16, 72B heads,
  // 66540 / 66650.
  if (!F8 && late) {
    request(1);
    request(2);
  }

  int it = 0;
  if (last >= 0) {
    f32x16 sa, sb;  // S^T of the tile's two blocks
    bf16x8 pa[2], pb[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) sa[r] = sb[r] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k(3 * MF_TILE, s), qf[s], sa, 0, 0, 0);
      sb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k(3 * MF_TILE + 32 * 256, s), qf[s], sb, 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      kf[s] = read_k(0, s);
      vf[s] = read_v(0, s);
    }
    if (masked(t_begin)) {
      mask(sa, t_begin, 0);
      mask(sb, t_begin, 1);
    }
    {
      // The first reference is the max of the tile's both blocks: a numerator just above 1 is rounded twice as coarsely as
      // one just below, and of nearly equal logits 1 in 64 lies above this reference instead of 1 in 32 (row error over
      // 26,000 such keys 1.6e-3 with the first block's max, 1.5e-3).
      float psum;
      move_reference(sa, sb, true, pa, psum);
      l_run += psum;
    }
    // While the pairs to be stored and requested are whole (and, over an 8-bit cache, cache tiles), that work is spread
    // over a step: issued together, the requests hold the wavefront up until the address path has taken those of all
    // wavefronts.
    const int whole = min(last, (F8 ? min(n, n_ct - t_begin) : n) - 4);
    while (it < whole) {
      const unsigned turn_mask = (it & 1) ? 3 * MF_TILE : MF_TILE;  // slot it & 3 -> slot (it + 1) & 3
      step(true_type(), false_type(), sa, sb, pa, pb, 0u, false, [&](int s) {
        if (F8 && (s & 1)) {
          store_piece(s >> 1, pend.p[s >> 1], (it + 2) & 3);
          pend.p[s >> 1] = load_piece(s >> 1);
        }
      });
      turn(it);
      const unsigned dst = st_lds + ((it + 3) & 3) * MF_TILE;
      ++it;
      if (masked(t_begin + it)) mask(sa, t_begin + it, 0);
      step(true_type(), true_type(), sb, sa, pb, pa, turn_mask, masked(t_begin + it), [&](int s) {
        if (!F8 && (s & 1)) request_half(s >> 1, dst);
      });
      advance_both();
      if (masked(t_begin + it)) mask(sb, t_begin + it, 1);
    }
    while (it < last) {
      const unsigned turn_mask = (it & 1) ? 3 * MF_TILE : MF_TILE;
      step(true_type(), false_type(), sa, sb, pa, pb, 0u, false, [](int) {});
      store_pending(it + 2);
      turn(it);
      request(it + 3);
      ++it;
      if (masked(t_begin + it)) mask(sa, t_begin + it, 0);
      step(true_type(), true_type(), sb, sa, pb, pa, turn_mask, masked(t_begin + it), [](int) {});
      if (masked(t_begin + it)) mask(sb, t_begin + it, 1);
    }
    step(false_type(), false_type(), sa, sb, pa, pb, 0u, false, [](int) {});
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (s > 0 && s + 2 < 8) vf[(s + 2) & 3] = read_v(32 * 256, s + 2);
      o[s & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s & 3], pb[s >> 2], o[s & 3], 0, 0, 0);
    }
  }
  for (; it + 1 < n; ++it) {
    store_pending(it + 2);
    if (F8) __builtin_amdgcn_s_waitcnt(MF_LGKM0);
    turn(it);
    request(it + 3);
  }

  if (my_split > 1) {
    // partial result of this chunk: every chunk starts on a cache tile, whose keys all rows see, so l_tot > 0
    const bool staged = n_rows > (a.n_g > MF_BN ? MF_HB : MF_DIRECT_ROWS);
    if (staged) __syncthreads();  // the ring's last readers (its last requests have landed, see turn)
    if (!wave_live) return;
    const float l_tot = sum_halves(l_run);
    const float inv = 1.f / l_tot;
    const size_t prow0 = (size_t)chunk * ((size_t)a.h_kv * a.part_rows) + (size_t)h * a.part_rows + row0;
    float* const po = a.part_o + prow0 * MF_D;
    if (!staged) {
      if (!row_ok) return;
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *(float4*)(po + l32 * MF_D + 32 * n + 8 * q4 + 4 * g) =
              make_float4(o[n][4 * q4] * inv, o[n][4 * q4 + 1] * inv, o[n][4 * q4 + 2] * inv, o[n][4 * q4 + 3] * inv);
      if (g == 0) a.part_lse[prow0 + l32] = m_run * c2 + log2f(l_tot);
      return;
    }
    // Through LDS, 16-byte chunk c of row r at c ^ (r & 15), which keeps both sides free of bank conflicts: a store then
    // writes two whole rows. Stored from the accumulators an instruction touched 32 rows in pieces of 32 bytes, 4096 of
    // them per workgroup and all at once at the launch's end. The workgroups' rows lie powers of two apart in many calls, so
    // each wavefront starts at another pair of its rows: all at their first, they met in few memory channels. us of the call
    // from the accumulators / through LDS / and from other rows: 7B heads, 77 tokens over 9,840 entries 29.2 / 27.8 / 28.0, 200
    // over 5,000 32.2 / 31.3 / 31.3, 512 over 2,000 37.2 / 38.5 / 37.1, over 5,000 52.5 / 51.5 / 51.7; 72B heads, 64 tokens over
    // 1,500 27.1 / 30.0 / 26.8, 128 over 3,000 34.1 / 34.7 / 33.6, 300 over 3,000 47.8 / 48.1 / 47.3.
    const int rot = (blockIdx.x >> 3) * 5 + (blockIdx.x & 7) * 2 + wave;
    unsigned char* const stage = smem + wave * (32 * MF_D * 4);
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *(float4*)(stage + l32 * (MF_D * 4) + ((8 * n + 2 * q4 + g) ^ (l32 & 15)) * 16) =
            make_float4(o[n][4 * q4] * inv, o[n][4 * q4 + 1] * inv, o[n][4 * q4 + 2] * inv, o[n][4 * q4 + 3] * inv);
    if (g == 0 && row_ok) a.part_lse[prow0 + l32] = m_run * c2 + log2f(l_tot);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the wavefront's writes before its reads
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int r = 2 * ((u + rot) & 15) + g;
      if (row0 + r < n_rows) *(float4*)(po + r * MF_D + 4 * l32) = *(const float4*)(stage + r * (MF_D * 4) + (l32 ^ (r & 15)) * 16);
    }
    return;
  }
  if (!wave_live) return;
  const float l_tot = sum_halves(l_run);
  if (!row_ok) return;
  const float inv = 1.f / l_tot;
  bf16_t* orow = (bf16_t*)a.out + ((t0 + t_lane) * a.h_q + (size_t)h * r_heads + j_lane) * MF_D;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int q4 = 0; q4 < 4; q4 += 2) {
      // Registers 4 q4 .. 4 q4 + 3 hold d = 32 n + 8 q4 + 4 g + 0..3: the row's two lanes swap, so that one has 8 outputs of
      // q4 and the other of q4 + 1, and a store writes 32 bytes of each of its rows instead of 16. No barrier here: wavefronts
      // end at their rows' horizons, and the stores of those that end early cost nothing. us before / after: 99 frames over an
      // 8-bit cache 486.2 / 478.2, 256 frames of the 7B heads 2222 / 2208, 1500 tokens of the 72B heads over 600 74.8 / 71.8.
      bf16x4 pk[2];
#pragma unroll
      for (int e = 0; e < 4; ++e) pk[0][e] = (__bf16)(o[n][4 * q4 + e] * inv), pk[1][e] = (__bf16)(o[n][4 * q4 + 4 + e] * inv);
      const uint2 even = __builtin_bit_cast(uint2, pk[0]), odd = __builtin_bit_cast(uint2, pk[1]);
      const auto x = __builtin_amdgcn_permlane32_swap(even.x, odd.x, false, false);
      const auto y = __builtin_amdgcn_permlane32_swap(even.y, odd.y, false, false);
      *(uint4*)(orow + 32 * n + 8 * (q4 + g)) = make_uint4(x[0], y[0], x[1], y[1]);
    }
  if (a.lse != nullptr && g == 0)
    a.lse[(size_t)(h * r_heads + j_lane) * a.n_g + t_lane] = (m_run * c2 + log2f(l_tot)) * 0.6931471805599453f;
}

// Merge of the key split: out[row] = sum_c 2^(lse_c - lse) O_c[row], lse = log2 sum_c 2^lse_c. One workgroup of 8
// wavefronts per row: wavefront w takes chunks w, w+8, ..., eight at a time with all their loads in flight at once
// (the log-sum-exps and the partial rows alike, so a wavefront pays one memory round trip per batch), merges them
// around its own maximum, and the eight results meet in LDS. Lane l owns d = 2l, 2l+1.
constexpr int MG_WAVES = 8;
__global__ __launch_bounds__(MG_WAVES * 64) void attend_merge_kernel(AttendArgs a) {
  __shared__ float red[MG_WAVES][64][2], red_m[MG_WAVES], red_l[MG_WAVES];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r_heads = a.h_q / a.h_kv;
  const int n_rows = a.part_rows;  // rows per KV head that were split
  const long total = (long)a.h_kv * n_rows;
  const long grow = blockIdx.x;
  const int h = (int)(grow / n_rows), row = (int)(grow - (long)h * n_rows);
  const int t = row / r_heads, j = row - t * r_heads;
  float m = -INFINITY, den = 0.f, acc0 = 0.f, acc1 = 0.f;  // this wavefront's chunks, relative to m
  for (int c0 = wave; c0 < a.n_split; c0 += 8 * MG_WAVES) {
    float ls[8];
    float2 po[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = min(c0 + MG_WAVES * u, a.n_split - 1);
      ls[u] = c0 + MG_WAVES * u < a.n_split ? a.part_lse[(size_t)c * total + grow] : -INFINITY;
      po[u] = *(const float2*)(a.part_o + ((size_t)c * total + grow) * MF_D + 2 * lane);
    }
    float mb = ls[0];  // finite: chunk c0 exists
#pragma unroll
    for (int u = 1; u < 8; ++u) mb = fmaxf(mb, ls[u]);
    const float m_new = fmaxf(m, mb);
    const float keep = exp2f(m - m_new);  // 0 the first time
    den *= keep;
    acc0 *= keep;
    acc1 *= keep;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float w = exp2f(ls[u] - m_new);
      den += w;
      acc0 = fmaf(w, po[u].x, acc0);
      acc1 = fmaf(w, po[u].y, acc1);
    }
    m = m_new;
  }
  red[wave][lane][0] = acc0;
  red[wave][lane][1] = acc1;
  if (lane == 0) {
    red_m[wave] = m;  // -inf for a wavefront without chunks: weight 0 below
    red_l[wave] = den;
  }
  __syncthreads();
  if (wave != 0) return;
  float big = red_m[0];
#pragma unroll
  for (int w = 1; w < MG_WAVES; ++w) big = fmaxf(big, red_m[w]);
  float dsum = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
  for (int w = 0; w < MG_WAVES; ++w) {
    const float wgt = exp2f(red_m[w] - big);
    dsum = fmaf(wgt, red_l[w], dsum);
    o0 = fmaf(wgt, red[w][lane][0], o0);
    o1 = fmaf(wgt, red[w][lane][1], o1);
  }
  const float inv = 1.f / dsum;
  bf16x2 pk;
  pk[0] = (__bf16)(o0 * inv);
  pk[1] = (__bf16)(o1 * inv);
  bf16_t* orow = (bf16_t*)a.out + ((size_t)t * a.h_q + (size_t)h * r_heads + j) * MF_D;
  *(uint32_t*)(orow + 2 * lane) = __builtin_bit_cast(uint32_t, pk);
  if (a.lse != nullptr && lane == 0)
    a.lse[(size_t)(h * r_heads + j) * a.n_g + t] = (big + log2f(dsum)) * 0.6931471805599453f;
}

// The same merge for launches of many rows and few chunks (text chunks, small groups against a long cache): one
// wavefront per row, four rows per workgroup, no exchange through LDS. Same arithmetic order per row as a single
// wavefront of attend_merge_kernel would use: chunks in batches of BATCH around a running max.
constexpr int MR_WAVES = 4;
template <int BATCH>
__global__ __launch_bounds__(MR_WAVES * 64) void attend_merge_rows_kernel(AttendArgs a) {
  const int lane = threadIdx.x & 63;
  const int r_heads = a.h_q / a.h_kv;
  const int n_rows = a.part_rows;  // rows per KV head that were split
  const long total = (long)a.h_kv * n_rows;
  const long grow = (long)blockIdx.x * MR_WAVES + (threadIdx.x >> 6);
  if (grow >= total) return;
  const int h = (int)(grow / n_rows), row = (int)(grow - (long)h * n_rows);
  const int t = row / r_heads, j = row - t * r_heads;
  float m = -INFINITY, den = 0.f, acc0 = 0.f, acc1 = 0.f;
  for (int c0 = 0; c0 < a.n_split; c0 += BATCH) {
    float ls[BATCH];
    float2 po[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int c = min(c0 + u, a.n_split - 1);
      ls[u] = c0 + u < a.n_split ? a.part_lse[(size_t)c * total + grow] : -INFINITY;
      po[u] = *(const float2*)(a.part_o + ((size_t)c * total + grow) * MF_D + 2 * lane);
    }
    float mb = ls[0];  // finite: chunk c0 exists
#pragma unroll
    for (int u = 1; u < BATCH; ++u) mb = fmaxf(mb, ls[u]);
    const float m_new = fmaxf(m, mb);
    const float keep = exp2f(m - m_new);  // 0 the first time
    den *= keep;
    acc0 *= keep;
    acc1 *= keep;
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const float w = exp2f(ls[u] - m_new);
      den += w;
      acc0 = fmaf(w, po[u].x, acc0);
      acc1 = fmaf(w, po[u].y, acc1);
    }
    m = m_new;
  }
  const float inv = 1.f / den;
  bf16x2 pk;
  pk[0] = (__bf16)(acc0 * inv);
  pk[1] = (__bf16)(acc1 * inv);
  bf16_t* orow = (bf16_t*)a.out + ((size_t)t * a.h_q + (size_t)h * r_heads + j) * MF_D;
  *(uint32_t*)(orow + 2 * lane) = __builtin_bit_cast(uint32_t, pk);
  if (a.lse != nullptr && lane == 0)
    a.lse[(size_t)(h * r_heads + j) * a.n_g + t] = (m + log2f(den)) * 0.6931471805599453f;
}

bool attend_mfma_supported(const AttendArgs& a, int dtype) {
  // 24-bit row and 32-bit byte offsets inside one head's cache / the group's K, V
  return dtype == QP_BF16 && a.d == MF_D && a.h_kv <= 65535 && (long long)a.cap * (MF_D * 2) < (1ll << 31) &&
         (long long)a.n_g * a.h_kv * (MF_D * 2) < (1ll << 31) && a.cap < (1 << 24);
}

// Chunk length (cache tiles) for `want` chunks of a row block whose rows see at most n_gt group tiles: the last chunk
// also walks those, so chunks are made just long enough that its cache tiles plus the group tiles do not exceed the
// others' length by more than one tile (all chunks end together). Every chunk starts on a cache tile.
static int chunk_tiles(int n_ct, int want, int n_gt) {
  int st = (n_ct + want - 1) / want;
  while (st < n_ct - 1 && n_ct - ((n_ct + st - 1) / st - 1) * st + n_gt > st + 1) ++st;
  return st;
}

AttendPlan plan_attend_mfma(const AttendArgs& a, size_t split_ws_bytes) {
  AttendPlan p;
  const int r_heads = a.h_q / a.h_kv;
  const int n_rows = a.n_g * r_heads;
  const int n_rb = ((n_rows + MF_HB - 1) / MF_HB + 1) / 2;
  const int n_wg = n_rb * a.h_kv;
  const int cus = device_cu_count();
  p.mirrored = n_wg <= cus;  // all workgroups resident at once: balance them; otherwise longest first
  p.n_split = 1;
  p.split_rb = 0;
  p.split_tiles = 0;
  p.scratch_bytes = 0;
  const int n_ct = (a.c + MF_BN - 1) / MF_BN;
  const size_t per_row = (size_t)(MF_D + 1) * sizeof(float);  // a partial row and its log-sum-exp
  if (split_ws_bytes > 0 && n_wg < MF_SPLIT_BELOW && n_ct >= 4) {
    // Few rows against a long cache (text prefill, decode, small groups): split the cache of every row block over
    // chunks so that the launch still covers the chip, at most one workgroup per CU, at least two tiles per chunk.
    const size_t per_split = (size_t)a.h_kv * n_rows * per_row;
    long want = cus / n_wg;  // rounded down: all chunks' workgroups resident at once, one round
    want = std::min<long>(want, n_ct / 2);
    want = std::min<long>(want, MF_MAX_SPLIT);
    want = std::min<long>(want, (long)(std::min(split_ws_bytes, MF_SPLIT_ALL_BYTES) / per_split));
    if (want >= 2) {
      p.split_tiles = chunk_tiles(n_ct, (int)want, (a.n_g + MF_BN - 1) / MF_BN);
      p.n_split = (n_ct + p.split_tiles - 1) / p.split_tiles;
      p.split_rb = n_rb;
      p.scratch_bytes = (size_t)p.n_split * per_split;
    }
  } else if (split_ws_bytes > 0 && !p.mirrored && (8 % a.h_kv == 0 || a.h_kv % 8 == 0)) {
    // Several rounds of workgroups, one per CU at a time. The workgroups of a KV head run on the CUs of that head's
    // XCDs (`pool` CUs serve `heads` KV heads); when the last round would fill only part of them, its row blocks (the
    // shortest: earliest tokens, started last) are split into chunks so that the chunks fill the pool evenly: t row
    // blocks in s chunks each take ceil(t s / pool) / s of a round instead of a whole one.
    const int heads = 8 % a.h_kv == 0 ? 1 : a.h_kv / 8;
    const int pool = 8 % a.h_kv == 0 ? cus / a.h_kv : cus / 8;
    const int items = n_rb * heads;
    const int tail = (items % pool) / heads;  // row blocks per KV head in the partial round
    if (pool > 0 && tail > 0) {
      const int part_rows = std::min(n_rows, tail * 2 * MF_HB);
      const int n_gt = (part_rows - 1) / r_heads / MF_BN + 1;  // group tiles the split rows see at most
      double best = 0.9;  // of a round: a split must save at least a tenth of one
      for (int want = 2; want <= MF_TAIL_SPLIT_MAX; ++want) {
        const int st = chunk_tiles(n_ct, want, n_gt);
        const int ns = st > 0 ? (n_ct + st - 1) / st : 0;  // the group tiles of the last chunk can make it fewer than wanted
        if (ns < 2 || st < MF_TAIL_MIN_TILES || (size_t)ns * a.h_kv * part_rows * per_row > split_ws_bytes) continue;
        // a chunk costs its share of the row block plus a prologue (~3 % of a row block of this length and more)
        const double cost = (double)((tail * heads * ns + pool - 1) / pool) / ns + 0.03 * (ns - 1);
        if (cost < best - 1e-9) {
          best = cost;
          p.n_split = ns;
          p.split_tiles = st;
          p.split_rb = tail;
          p.scratch_bytes = (size_t)ns * a.h_kv * part_rows * per_row;
        }
      }
    }
  }
  const int n_items = (n_rb - p.split_rb) + p.split_rb * p.n_split;  // workgroups per KV head
  p.workgroups = n_items * a.h_kv;
  if (8 % a.h_kv == 0) {
    const int per = 8 / a.h_kv;
    p.workgroups = (n_items + per - 1) / per * 8;
  }
  return p;
}

static void set_lds_limit() {
  static bool attr_set[QP_MAX_DEVICES] = {};
  const int dev = current_device();
  if (dev >= 0 && attr_set[dev]) return;
  (void)hipFuncSetAttribute((const void*)attend_mfma_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            MF_LDS);
  (void)hipFuncSetAttribute((const void*)attend_mfma_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            MF_LDS);
  if (dev >= 0) attr_set[dev] = true;
}

long attend_mfma_row_blocks(int n_g, int h_q, int h_kv) {
  return (((long)n_g * (h_q / h_kv) + MF_HB - 1) / MF_HB + 1) / 2;
}

void launch_attend_mfma_run(const AttendArgs& a_in, hipStream_t s) {
  set_lds_limit();
  AttendArgs a = a_in;
  a.mirrored = 0;
  a.n_split = 1;
  a.split_rb = a.split_tiles = a.part_rows = 0;
  const long items = attend_mfma_row_blocks(a.n_last, a.h_q, a.h_kv) + (a.groups - 1) * attend_mfma_row_blocks(a.n_g, a.h_q, a.h_kv);
  long wgs = items * a.h_kv;
  if (8 % a.h_kv == 0) {
    const int per = 8 / a.h_kv;
    wgs = (items + per - 1) / per * 8;
  }
  if (a.cache_fp8)
    hipLaunchKernelGGL(attend_mfma_kernel<true>, dim3((unsigned)wgs), dim3(MF_NT), MF_LDS, s, a);
  else
    hipLaunchKernelGGL(attend_mfma_kernel<false>, dim3((unsigned)wgs), dim3(MF_NT), MF_LDS, s, a);
}

void launch_attend_mfma(const AttendArgs& a_in, void* split_ws, size_t split_ws_bytes, hipStream_t s) {
  set_lds_limit();
  AttendArgs a = a_in;
  const AttendPlan p = plan_attend_mfma(a, split_ws != nullptr ? split_ws_bytes : 0);
  a.mirrored = p.mirrored;
  a.n_split = p.n_split;
  a.split_tiles = p.split_tiles;
  a.split_rb = p.split_rb;
  a.part_rows = std::min(a.n_g * (a.h_q / a.h_kv), p.split_rb * 2 * MF_HB);
  a.part_o = nullptr;
  a.part_lse = nullptr;
  if (p.n_split > 1) {
    a.part_o = (float*)split_ws;
    a.part_lse = a.part_o + (size_t)p.n_split * a.h_kv * a.part_rows * MF_D;
  }
  if (a.cache_fp8)
    hipLaunchKernelGGL(attend_mfma_kernel<true>, dim3(p.workgroups), dim3(MF_NT), MF_LDS, s, a);
  else
    hipLaunchKernelGGL(attend_mfma_kernel<false>, dim3(p.workgroups), dim3(MF_NT), MF_LDS, s, a);
  if (p.n_split > 1) launch_attend_merge(a, s);
}

void launch_attend_merge(const AttendArgs& a, hipStream_t s) {
  const long total = (long)a.h_kv * a.part_rows;
  // few rows, many chunks (decode): a workgroup of 8 wavefronts per row; many rows and up to 32 chunks: a wavefront per
  // row. The 8-wavefront kernel loads 64 chunks' rows whatever their number: 77 tokens of the 7B heads over 9,840
  // entries (2,156 rows, 20 chunks) take 31.6 us with the other one, 33.4 with it, of which the attention is 27.
  const dim3 rows_grid((unsigned)((total + MR_WAVES - 1) / MR_WAVES));
  if (total > 1024 && a.n_split <= 8)
    hipLaunchKernelGGL(attend_merge_rows_kernel<8>, rows_grid, dim3(MR_WAVES * 64), 0, s, a);
  else if (total > 1024 && a.n_split <= 32)
    hipLaunchKernelGGL(attend_merge_rows_kernel<16>, rows_grid, dim3(MR_WAVES * 64), 0, s, a);
  else
    hipLaunchKernelGGL(attend_merge_kernel, dim3((unsigned)total), dim3(MG_WAVES * 64), 0, s, a);
}

}  // namespace qp
