// bf16 MFMA matrix product for the projections of the decoder layer around the path (gfx950):
//   Y[m][n] = sum_k X[m][k] W[n][k]      X [M][K] activations (tokens slow), W [N][K] weights ([out][in]),
// f32 accumulation, with the layer's elementwise steps fused into the store:
//   PLAIN    Y (+ bias[n]) (+ residual[m][n]) -> bf16 [M][N]          (o_proj and down_proj with the residual add)
//   QKV_ROPE Y + bias, rotary embedding on the query and key heads, scattered to Q [M][H_q][128],
//            K [M][H_kv][128], V [M][H_kv][128] (the token-major layout the attention kernels read)
//   SWIGLU   W = [gate rows ; up rows] (2 d_ff rows): SiLU(gate) * up -> bf16 [M][d_ff]
//            (Appendix D.1 of the paper: SwiGLU(x) = W_down(SiLU(W_gate x) * W_up x))
//
// Tiling. A workgroup of 8 wavefronts owns a 256 x 256 output tile and walks K in steps of 64. Both operand
// tiles (256 rows x 128 bytes each) go global -> LDS with global_load_lds_dwordx4 into rings of buffers (two for
// activations, three for weights), the next steps' tiles in flight while this step's are multiplied; one barrier per
// step, placed in the middle of the step's products so that the matrix pipe stays busy across it. Rows are
// unpadded; the
// 16-byte chunk c of row r sits at position c ^ ((r >> 1) & 7), which makes both the 1 KB stores of the loads
// and the fragment reads (16 rows x 16 bytes per quarter wavefront) conflict-free.
// Wavefront (wm, wn) of the 2 x 4 arrangement computes 128 tokens x 64 outputs as 8 x 4 blocks of
// v_mfma_f32_16x16x32_bf16 with the WEIGHT rows as the A operand and the token rows as B, so that a lane ends
// up with one token (m = lane & 15) and, per block, a run of 4 outputs: the fused steps below
// only ever combine values of the same lane:
//   * QKV_ROPE: the 256 tile columns are two heads; wavefront wn serves head wn >> 1 and, of its 128 dims, the
//     32 dims [32 (wn & 1), +32) in blocks 0 and 1 and their rotary partners (+64) in blocks 2 and 3. The weight rows are
//     fetched into LDS in that order (a permutation inside the tile, contiguous in runs of 32 rows).
//   * SWIGLU: blocks 0 and 1 hold gate columns [n0/2 + 32 wn, +32), blocks 2 and 3 the up columns of the same outputs.
// The shape of the product: at full occupancy the chip is bound by power, and a product of 16 x 16 x 32 costs less of it than
// half of one of 32 x 32 x 16, whose accumulators pass through the registers every 16 k instead of every 32. Register-only
// loops (mfma_peak_probe.hip) on random operands reach 2.14 PFLOP/s with the former and 1.85 with the latter (2.47 both on zeros). Both add
// k in runs of 8, one after the other, so the results are the same bits.
// Workgroup ids are dealt round-robin over the 8 XCDs; the workgroups an XCD runs side by side cover a block of
// token tiles x weight tiles, which bounds what its L2 has to fetch per k-step.
#include <algorithm>
#include <atomic>

#include "append.h"
#include "qp_internal.h"

namespace qp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int GM_BK = 64;   // k per ring slot
constexpr int GM_BN = 256;  // weight rows per tile of the wide tilings
// BM token rows x BN weight rows per workgroup, dealt to wavefronts of 32 MI tokens x 64 outputs. XS, WS: depth of the
// rings of LDS slots that hold activation and weight tiles, all of whose free slots are in flight: equal, or 2 and 3.
template <int BM_, int BN_, int MI_, int XS_, int WS_ = XS_>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, MI = MI_;        // MI: 32-token blocks per wavefront
  static constexpr int WN = BN / 64, WM = BM / (32 * MI);   // wavefronts across the outputs / the tokens
  static constexpr int NW = WN * WM;
  static constexpr int BK = GM_BK;
  static constexpr int ROWB = BK * 2;                       // bytes per tile row
  static constexpr int CPR = ROWB / 16;                     // 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;                      // rows one load instruction covers
  static constexpr int RPL = 256 / ROWB;                    // rows per 256 bytes of LDS (one sweep of the banks)
  static constexpr int KS = BK / 32;                        // k-steps of the MFMA per slot
  static constexpr int XT = BM * ROWB;                      // bytes of the activation tile
  static constexpr int WT = BN * ROWB;                      // ... of the weight tile
  static constexpr int XS = XS_, WS = WS_;
  static constexpr int LDS = XS * XT + WS * WT;             // activation ring, then weight ring
  static constexpr int XQ = BM / NW / RPI;                  // activation load instructions per wavefront and slot
  static constexpr int WQ = BN / NW / RPI;                  // weight load instructions per wavefront and slot
  static constexpr int PER_WAVE = XQ + WQ;
  static_assert(XQ * NW * RPI == BM && WQ * NW * RPI == BN && LDS <= 160 * 1024 && (XS == WS || (XS == 2 && WS == 3)), "tile shape");
  // chunk c of row r sits at position c ^ swizzle(r): 16 consecutive rows' reads of one chunk index, and the 1 KB
  // written by one load instruction, then touch every bank group once
  __device__ static constexpr int swizzle(int r) { return (r / RPL) & (CPR - 1); }
};
typedef Tile<256, 256, 4, 2, 3> Tile256;    // 8 wavefronts, one workgroup per CU
typedef Tile<128, 256, 2, 3> Tile128;
typedef Tile<128, 128, 1, 3> Mid;
typedef Tile<128, 64, 2, 3> Narrow128;    // 2 wavefronts, two workgroups per CU
typedef Tile<64, 64, 1, 3> Narrow64;      // ... three
typedef Tile<64, 64, 1, 5> Deep64;        // two
typedef Tile<64, 128, 1, 3> Mid64;        // 4 wavefronts, two workgroups per CU
typedef Tile<64, 256, 1, 4> Wide64;       // 8 wavefronts, all of a CU's LDS

// 64 lanes x 16 bytes global -> LDS at the wave-uniform LDS byte address lds_addr (lane L lands at lds_addr + 16 L);
// m0 is clobbered on purpose (see lds_dma16)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void gm_dma16(const unsigned char* base, unsigned byte_off, unsigned lds_addr) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(byte_off), "s"(base), "s"(lds_addr)
      : "memory", "m0");
}
#pragma clang diagnostic pop

// acc += w x, in place. The builtin leaves it to the allocator where the sum goes, and that moved accumulators around and
// spilled. What the compiler does not know of an instruction in inline assembly is how long its result takes: the accumulators
// meet no other instruction from their clearing to the end of the products, and there the wait is spelled out (the fragments
// come from LDS reads, whose counter the compiler minds as for any operand). tests/test_product_waits.py reads the assembly for it.
__device__ __forceinline__ void gm_product(f32x4& acc, const u32x4& w, const u32x4& x) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(x));
}

template <int N>
__device__ __forceinline__ void gm_wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// LDS row j of the weight tile <- which weight row (relative to the tile's first), per mode
template <int MODE>
__device__ __forceinline__ int weight_row(int j, int n0, int d_ff) {
  if (MODE == GEMM_QKV_ROPE) {  // runs of 64: half a head's rotary pairs
    const int u = (n0 + j) >> 6;
    return (u >> 1) * 128 + ((j >> 5) & 1) * 64 + (u & 1) * 32 + (j & 31);
  }
  if (MODE == GEMM_SWIGLU) return ((j >> 5) & 1) * d_ff + (n0 >> 1) + (j >> 6) * 32 + (j & 31);
  return n0 + j;
}

// Whether a split contraction on tiles of 128 or 256 outputs deals its tiles' chunks to the XCDs instead of its tiles (see launch_tile).
__device__ __forceinline__ bool deals_items(int split_k, int tiles) { return split_k > 1 && tiles % 8 != 0; }

// A grid of tiles of one kind: block `block` of `blocks` (a multiple of 8) per k chunk, over outputs n_first and up.
struct TileGrid {
  int block, blocks;
  int tiles_m, tiles_n, m_block;
  int n_first;
};
template <int MODE, typename T>
__device__ __forceinline__ void gemm_tile_product(const GemmArgs& a, const TileGrid& grid, unsigned char* smem) {
  constexpr int ROWB = T::ROWB, BM = T::BM, BN = T::BN, BK = T::BK;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int wm = wave / T::WN, wn = wave % T::WN;

  // workgroup id -> (weight tile, token tile). Ids go round-robin over the 8 XCDs; each XCD takes an equal run of the
  // tiles in an order of blocks of up to 8 token tiles x 4 weight tiles: of the 32 workgroups that an XCD runs side by
  // side, its L2 then fetches 8 + 4 operand tiles per k-step for 32 products. (Weight tiles dealt to the XCDs in turn
  // left them unequal: 18 weight tiles x 12 token tiles put 36 workgroups on two XCDs of 32 CUs, 166 us for QKV of 3000
  // tokens at 7B sizes, 99 now.)
  // A split contraction has a grid row per k chunk, and its tiles are dealt row by row, or (deals_items) the chunks of its
  // tiles, tile by tile, over the whole grid.
  const int tiles = grid.tiles_m * grid.tiles_n;
  const bool by_item = T::BN >= 128 && deals_items(a.split_k, tiles);
  const int block = by_item ? blockIdx.y * grid.blocks + grid.block : grid.block;
  const int items = by_item ? tiles * a.split_k : tiles, per_xcd = (items + 7) >> 3;
  int id = (block & 7) * per_xcd + (block >> 3), chunk = blockIdx.y;
  if ((block >> 3) >= per_xcd || id >= items) return;  // padding of the mapping (whole workgroup, before any barrier)
  if (by_item) {
    const int tile = id / a.split_k;
    chunk = id - tile * a.split_k;
    id = tile;
  }
  // block `quad` of n_quads has the weight tiles quad, quad + n_quads, ...: nw of them, one more in the first n_more blocks
  const int n_quads = (grid.tiles_n + 3) / 4, fewer = grid.tiles_n / n_quads, n_more = grid.tiles_n - fewer * n_quads;
  const int in_more = n_more * (fewer + 1) * grid.tiles_m;
  const int nw = id < in_more ? fewer + 1 : fewer, rel = id < in_more ? id : id - in_more;
  const int q0 = rel / (nw * grid.tiles_m), in_quad = rel - q0 * nw * grid.tiles_m;
  const int quad = id < in_more ? q0 : n_more + q0;
  const int mc = in_quad / (nw * grid.m_block), in_blk = in_quad - mc * nw * grid.m_block;
  const int mh = min(grid.m_block, grid.tiles_m - mc * grid.m_block);         // token tiles of this block of m_block
  const int tm = mc * grid.m_block + in_blk % mh, tn = quad + n_quads * (in_blk / mh);
  const int m0 = tm * BM, n0 = grid.n_first + tn * BN;
  const int d_ff = a.n >> 1;

  // staging: activation load q of this wavefront covers tile rows (BM/NW) wave + RPI q + lane / CPR, weight load q
  // rows (BN/NW) wave + RPI q + lane / CPR; LDS position lane % CPR of the row holds chunk position ^ swizzle(row)
  const unsigned char* xg = (const unsigned char*)a.x;
  const unsigned char* wg = (const unsigned char*)a.w;
  const size_t row_b = (size_t)a.k * 2;
  unsigned x_off[T::XQ], w_off[T::WQ];
  const int wb = MODE == GEMM_SWIGLU ? (n0 >> 1) : MODE == GEMM_QKV_ROPE ? n0 & ~127 : n0;  // first weight row this tile may touch
  // offsets relative to the tile's first row (the launcher checks that they fit 32 bits)
#pragma unroll
  for (int q = 0; q < T::XQ; ++q) {
    const int r = (BM / T::NW) * wave + T::RPI * q + lane / T::CPR;
    const int xr = min(m0 + r, a.m - 1);  // rows past the end: computed, not stored
    x_off[q] = (unsigned)((size_t)(xr - m0) * row_b) + (unsigned)((lane % T::CPR) ^ T::swizzle(r)) * 16;
  }
#pragma unroll
  for (int q = 0; q < T::WQ; ++q) {
    const int r = (BN / T::NW) * wave + T::RPI * q + lane / T::CPR;
    const int wr = min(weight_row<MODE>(r, n0, d_ff), a.n - 1);
    w_off[q] = (unsigned)((size_t)(wr - wb) * row_b) + (unsigned)((lane % T::CPR) ^ T::swizzle(r)) * 16;
  }
  // contraction split (launches of few tiles): the k-steps are dealt to chunks, each leaving an f32 partial tile
  const int step_begin = chunk * a.steps_per_split;
  const unsigned char* x_base = xg + (size_t)m0 * row_b + (size_t)step_begin * ROWB;
  const unsigned char* w_base = wg + (size_t)wb * row_b + (size_t)step_begin * ROWB;
  const unsigned smem_lds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const unsigned x_lds = smem_lds + wave * (BM / T::NW) * ROWB, w_lds = smem_lds + T::XS * T::XT + wave * (BN / T::NW) * ROWB;

  // activation / weight load instruction p_ of a step into slot slot_ of its ring
#define GM_ISSUE_X(p_, step_, slot_) gm_dma16(x_base, x_off[p_] + (unsigned)(step_) * ROWB, x_lds + (slot_)*T::XT + 1024 * (p_));
#define GM_ISSUE_W(p_, step_, slot_) gm_dma16(w_base, w_off[p_] + (unsigned)(step_) * ROWB, w_lds + (slot_)*T::WT + 1024 * (p_));

  // fragment addresses inside a slot: row (l16 + 16 block), chunk 4 s + g of k-step s
  int f_off[T::KS];
#pragma unroll
  for (int s = 0; s < T::KS; ++s) f_off[s] = l16 * ROWB + (((4 * s + g) ^ T::swizzle(l16)) << 4);
  const int x_frag = wm * (32 * T::MI) * ROWB;
  const int w_frag = T::XS * T::XT + wn * 64 * ROWB;

  constexpr int NJ = 4, NI = 2 * T::MI;  // 16 x 16 blocks per wavefront across the outputs / the tokens
  f32x4 acc[NJ][NI];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
      asm volatile("" : "+v"(acc[j][i]));
    }

  // Ring schedule. All slots are free at the start, so the first steps are requested at once. Inside the
  // loop the barrier sits between the two k-steps of a step: by then every wavefront has read all its
  // fragments of the step (its slots can be refilled), the next step's tiles have landed, and the wait at the
  // barrier and the latency of the next step's first fragment reads run under the second k-step's products.
  // With equal rings of the smaller tilings all refill requests are issued there too. At 256 x 256 that is 64 of them, and
  // the address path takes 16 cycles for each, falls behind, and holds up the
  // products behind the requests. So that tiling (rings of 2 and 3) spreads them: a step t issues W(t + 2) in its first half,
  // into the slot that step t - 1 left, and behind the barrier X(t + 2), which is awaited there a step later: half of it
  // in the first half of step t + 1 left it half a step and cost 5-8 %. The 128 x 256 tiling (equal rings of 3)
  // puts its requests behind every other product behind the barrier, two steps ahead of their wait. us, weights from HBM, in the
  // first half of the next step / there: 2048 x 3584 x 18944 255.6 / 251.8, 2048 x 4096 x 14336 204.1 / 200.4, 1024 x 6144 x 5120
  // 76.9 / 75.9, 768 x 8192 x 29568 421 / 416; in chunks 520 x 3584 x 18944 92.4 / 89.9, 400 x 8192 x 29568 236 / 230. Behind
  // every product they are all under way a little sooner, but ragged or short launches lose: every other / every product 1024 x
  // 6144 x 5120 76.7 / 74.9, 1920 x 3584 x 18944 256 / 250, but 1024 x 8192 x 8192 121.5 / 125.4, 2048 x 4096 x 4096 62.1 / 63.9, 300
  // x 59136 x 8192 342 / 357, 520 x 3584 x 18944 91.5 / 95.4, 900 tokens of it 132 / 139.
  // PFLOP/s of products of 32 x 32 x 16 with the barrier behind three quarters of a step / of this loop, random inputs, one weight:
  // 4096 x 59136 x 8192 1.38 / 1.46, 4096 x 8192 x 29568 1.36 / 1.48, 2048 x 37888 x 3584 1.24 / 1.33, 8192 x 8192 x 8192 1.35 /
  // 1.47, 1024 x 8192 x 8192 1.19 / 1.29. Launches of 128 x 256 tiles with weights from HBM gained little by the shape: 2048 x 3584 x
  // 18944 259 us / 257, x 3584 55.3 / 54.8, 1024 x 8192 x 29568 434 / 433. On zeros, which leave the clock alone, 8192 x 8192 x
  // 8192 runs at 1.80, and at 1.98 with the lines of later steps touched ahead of the requests, so that these find them in the
  // L2; on random inputs that cost 1 %.
  // Requests complete in order: when step t + 1 is awaited at the end of step t, what may stay in flight is, with equal
  // rings, the XS - 2 steps after it, and with rings of 2 and 3 the weights of step t + 2.
  const int n_steps = min(a.steps_per_split, a.k / BK - step_begin);
  constexpr int XS = T::XS, WS = T::WS, PW = T::PER_WAVE;
#pragma unroll
  for (int p = 0; p < XS; ++p)
    if (p < n_steps) {
#pragma unroll
      for (int q = 0; q < T::XQ; ++q) GM_ISSUE_X(q, p, p)
#pragma unroll
      for (int q = 0; q < T::WQ; ++q) GM_ISSUE_W(q, p, p)
    }
  // the first step's tiles have landed: all but the later requests are complete
  if (XS > 3 && n_steps >= XS) gm_wait_vmcnt<(XS - 1) * PW>();
  else if (XS >= 3 && n_steps >= 3) gm_wait_vmcnt<2 * PW>();
  else if (n_steps >= 2) gm_wait_vmcnt<PW>();
  else gm_wait_vmcnt<0>();
  __syncthreads();
  // Fragments: two sets of the weights', and of the activations' in the small tilings; the 128 x 256 and 256 x 256 ones have one
  // of these, each refilled for the next k-step behind its last product. 256 x 256 has no registers for two (two for the last of
  // the eight, so that no read is issued right in front of the barrier, changed nothing). 128 x 256, us with two sets / one, weights
  // from HBM: 2048 x 3584 x 18944 249.9 / 244.6, 2048 x 4096 x 14336 198.6 / 194.1, 1024 x 6144 x 5120 75.6 / 74.6, 768 x 8192 x 29568
  // 414 / 409, 300 x 59136 x 8192 323 / 322 (one weight, from the caches: 2048 x 3584 x 18944 222 / 227); 128 x 64: 256 x 1024 x
  // 4096 13.6 / 13.8, 100 x 4608 x 3584 21.7 / 21.7.
  constexpr int XSETS = T::BN == 256 && T::MI >= 2 ? 1 : 2;
  u32x4 wf[2][NJ], xf[XSETS][NI];
#define GM_READ_W(wst_, s_, j_) wf[s_][j_] = *(const u32x4*)((wst_) + w_frag + (j_) * 16 * ROWB + f_off[s_]);
#define GM_READ_X(xst_, s_, i_) xf[(s_) % XSETS][i_] = *(const u32x4*)((xst_) + x_frag + (i_) * 16 * ROWB + f_off[s_]);
  // behind product mf of a k-step: the fragments of the next one, k-step s_
#define GM_READ_AHEAD(xst_, wst_, s_, mf_)                                                                     \
  {                                                                                                            \
    if ((mf_) < NJ) GM_READ_W(wst_, s_, (mf_) < NJ ? (mf_) : 0)                                                \
    if (XSETS == 1 ? (mf_) % NJ == NJ - 1 : (mf_) < NI) GM_READ_X(xst_, s_, XSETS == 1 ? (mf_) / NJ : (mf_) < NI ? (mf_) : 0)  \
  }
  // One product of k-step s by index: NJ in a row share the activations' fragment, and the last of them and the next one the
  // weights', back and forth: every operand that stays saves power. us forth only / back and forth, weights from HBM: 8192 x 8192 x
  // 8192 756 / 746, 4096 x 8192 x 29568 1326 / 1311, 4096 x 59136 x 8192 2760 / 2747; launches of 128 x 256 tiles do not change.
#define GM_J(mf_) ((((mf_) / NJ) & 1) ? NJ - 1 - (mf_) % NJ : (mf_) % NJ)
#define GM_MFMA_ONE(s_, mf_)                                                                                   \
  gm_product(acc[GM_J(mf_)][(mf_) / NJ], wf[s_][GM_J(mf_)], xf[(s_) % XSETS][(mf_) / NJ]);
  constexpr int NM = NJ * NI;              // products per k-step
  constexpr int PER = (PW + NM - 1) / NM;  // refill requests behind each of them
#pragma unroll
  for (int j = 0; j < NJ; ++j) GM_READ_W(smem, 0, j)
#pragma unroll
  for (int i = 0; i < NI; ++i) GM_READ_X(smem, 0, i)
  int xslot = 0, wslot = 0;
  constexpr int EVERY = T::MI == 2 && T::BN == 256 ? 2 : 1;  // ... or one behind every other product
  static_assert(XS <= 5 && (XS - 1) * PW <= 63, "the waits spelled out, and what vmcnt counts");
  static_assert(T::KS == 2, "two k-steps of the products per slot");
  static_assert(XS != WS || EVERY == 1 || (PER == 1 && PW <= NM / EVERY), "all requests within a k-step");
  static_assert(XS == WS || (T::XQ == 4 && T::WQ == 4 && T::MI == 4), "where rings of 2 and 3 put their requests");
  // One step that has a successor; refill: there is a step left to request into the freed slots.
  auto step_and_next = [&](int step, bool refill, auto wait) {
    const unsigned char *xst = smem + xslot * T::XT, *wst = smem + wslot * T::WT;
    const int wfree = wslot == 0 ? WS - 1 : wslot - 1;  // the slot that the step before left
#pragma unroll
    for (int mf = 0; mf < NM; ++mf) {
      GM_MFMA_ONE(0, mf)
      GM_READ_AHEAD(xst, wst, 1, mf)
      __builtin_amdgcn_sched_barrier(0);
      if (XS != WS && mf % 8 == 4 && refill) GM_ISSUE_W(mf / 8, step + 2, wfree)
      __builtin_amdgcn_sched_barrier(0);
    }
    const int xnext = xslot == XS - 1 ? 0 : xslot + 1, wnext = wslot == WS - 1 ? 0 : wslot + 1;
    wait();           // this wavefront's part of the next step's tiles has landed (later ones may still be in flight) ...
    __syncthreads();  // ... everyone's has, and everyone has read its last fragments of this step's slots
    const unsigned char *xst_next = smem + xnext * T::XT, *wst_next = smem + wnext * T::WT;
#pragma unroll
    for (int mf = 0; mf < NM; ++mf) {
      GM_MFMA_ONE(1, mf)
      GM_READ_AHEAD(xst_next, wst_next, 0, mf)
      __builtin_amdgcn_sched_barrier(0);
      if (XS != WS) {
        if (mf % 4 == 2 && mf / 4 < T::XQ && refill) GM_ISSUE_X(mf / 4, step + XS, xslot)
      } else if (refill && mf % EVERY == EVERY - 1) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const int p = mf / EVERY * PER + u;
          if (p < T::XQ) GM_ISSUE_X(p, step + XS, xslot)
          else if (p < PW) GM_ISSUE_W(p - T::XQ, step + WS, wslot)
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    xslot = xnext, wslot = wnext;
  };
  // A wavefront whose tokens all lie past the end multiplies nothing: it requests its part of the tiles and keeps the barriers.
  // Its products cost power, and with the other wavefronts of its SIMD the matrix pipe. us with them / without: 900 x 3584 x 18944
  // 135 / 129, 260 and 300 x 59136 x 8192 338 / 322 and 345 / 335, 258 x 3584 x 18944 60.7 / 57.9, 16 x 8192 x 8192 36.2 / 32.6, QKV
  // of 3 tokens 1536 -> 2048 10.0 / 9.3 and 2048 -> 2560 10.8 / 10.3; full tiles do not change.
  auto idle_and_next = [&](int step, bool refill, auto wait) {
    if (XS != WS && refill) {
      const int wfree = wslot == 0 ? WS - 1 : wslot - 1;
#pragma unroll
      for (int q = 0; q < T::WQ; ++q) GM_ISSUE_W(q, step + 2, wfree)
    }
    wait();
    __syncthreads();
    if (refill) {
#pragma unroll
      for (int q = 0; q < T::XQ; ++q) GM_ISSUE_X(q, step + XS, xslot)
      if (XS == WS)
#pragma unroll
        for (int q = 0; q < T::WQ; ++q) GM_ISSUE_W(q, step + WS, wslot)
    }
    xslot = xslot == XS - 1 ? 0 : xslot + 1, wslot = wslot == WS - 1 ? 0 : wslot + 1;
  };
  auto walk = [&](auto and_next) {  // every step but the last
    int step = 0;
    for (; step + XS < n_steps; ++step) and_next(step, true, [] { gm_wait_vmcnt<XS != WS ? T::WQ : (XS - 2) * PW>(); });
    for (; step + 1 < n_steps; ++step)
      and_next(step, false, [&] {
        if (XS == WS && XS >= 5 && step + 4 < n_steps) gm_wait_vmcnt<3 * PW>();
        else if (XS == WS && XS >= 4 && step + 3 < n_steps) gm_wait_vmcnt<2 * PW>();
        else if (XS == WS && XS >= 3 && step + 2 < n_steps) gm_wait_vmcnt<PW>();
        else gm_wait_vmcnt<0>();
      });
  };
  const int mw = m0 + wm * (32 * T::MI);  // this wavefront's first token
  if (mw >= a.m) {
    walk(idle_and_next);
    if (MODE != GEMM_SWIGLU && a.split_k == 1) __syncthreads();  // the one in front of the staging
    return;
  }
  walk(step_and_next);
  {  // last step: nothing left to request or to wait for
    const unsigned char *xst = smem + xslot * T::XT, *wst = smem + wslot * T::WT;
#pragma unroll
    for (int mf = 0; mf < NM; ++mf) {
      GM_MFMA_ONE(0, mf)
      GM_READ_AHEAD(xst, wst, 1, mf)
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int mf = 0; mf < NM; ++mf) GM_MFMA_ONE(1, mf)
  }
#undef GM_MFMA_ONE
#undef GM_J
#undef GM_READ_AHEAD
#undef GM_READ_W
#undef GM_READ_X
#undef GM_ISSUE_X
#undef GM_ISSUE_W

  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15\n\ts_nop 7");  // the last products' results, which nothing may take from in front of here
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i) asm volatile("" : "+v"(acc[j][i]));
  __builtin_amdgcn_sched_barrier(0);
  // ---- store: lane owns token m = m0 + (32 MI) wm + 16 i + l16 and, in block j, outputs 4 g + 0..3
  const int u64 = (n0 >> 6) + wn;  // QKV_ROPE: which run of 64 outputs (half a head's rotary pairs) this wavefront has
  if (a.split_k > 1) {
    // partial sums of this k chunk, f32 [chunk][m][n] with n the output's logical column (for QKV: head * 128 + dim);
    // gemm_reduce_kernel adds the chunks in order and applies the mode's store
    float* part = a.partial + (size_t)chunk * a.m * a.n;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      int n;
      if (MODE == GEMM_QKV_ROPE) n = (u64 >> 1) * 128 + (u64 & 1) * 32 + (j >> 1) * 64 + 16 * (j & 1) + 4 * g;
      else n = n0 + wn * 64 + j * 16 + 4 * g;
      if (n >= a.n) continue;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int m = mw + i * 16 + l16;
        if (m >= a.m) continue;
        *(float4*)(part + (size_t)m * a.n + n) = make_float4(acc[j][i][0], acc[j][i][1], acc[j][i][2], acc[j][i][3]);
      }
    }
    return;
  }
  if (MODE == GEMM_SWIGLU) {  // half as many outputs: 64-byte runs of rows staged as below gained nothing (7.5 us per tile)
    bf16_t* out = (bf16_t*)a.out;
#pragma unroll
    for (int j = 0; j < NJ / 2; ++j) {
      const int n = (n0 >> 1) + wn * 32 + 16 * j + 4 * g;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int m = mw + i * 16 + l16;
        if (m >= a.m) continue;
        bf16x4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gate = acc[j][i][e], up = acc[j + 2][i][e];
          pk[e] = (__bf16)(gate / (1.f + __expf(-gate)) * up);
        }
        *(uint2*)(out + (size_t)m * d_ff + n) = __builtin_bit_cast(uint2, pk);
      }
    }
    return;
  }
  // Results go through LDS, bf16, so that a store instruction writes whole runs of rows: 8 rows x 128 bytes (PLAIN) or 16
  // rows x 64 (QKV_ROPE: half of a half head), 16 bytes per lane; a residual is read the same way. Stored from the
  // accumulator layout an instruction touched 32 rows in pieces of 16 bytes, and a short contraction was bound by that:
  // 8192 x 8192 x 512, four tiles per CU, 154 us (with a residual 169), now 102 (109; the library's plain product 81);
  // x 3584 437 (457), now 376 (400); 4096 x 4096 x 512 31 (47), now 26 (30).
  // Each wavefront stages its own tokens x outputs, so one barrier (the ring's last readers) is all it takes. Row r's
  // 16-byte chunk c sits at c ^ (r & 7) (128-byte rows) or c ^ ((r >> 2) & 3) (64-byte rows), which keeps the 16-byte accesses
  // free of bank conflicts. The 8-byte ones of the accumulator layout have them in 128-byte rows, where rows r and r + 8 of a
  // half wavefront's 16 meet: counted at 8192 x 8192, 4 cycles per write, 12 % of the LDS cycles at k = 512 and 2 % at k = 3584, and
  // 2 per read of a residual, 14 and 3 % in all.
  __syncthreads();
  constexpr int SROW = MODE == GEMM_PLAIN ? 128 : 64;  // bytes of a staged row
  constexpr int SC = SROW / 16;                         // its chunks
  constexpr int SBLK = 32 * SROW;                       // bytes of 32 staged tokens
  constexpr int SREG = (MODE == GEMM_QKV_ROPE ? 2 : 1) * T::MI * SBLK;  // this wavefront's region
  static_assert(T::NW * SREG <= T::LDS, "staging fits the rings");
  unsigned char* const stage = smem + wave * SREG;
  auto swizzled = [](int r, int c) { return c ^ (SC == 8 ? r & 7 : (r >> 2) & 3); };
  // this lane's run of 4 outputs in block j16 of 16 (chunk 2 j16 + g / 2, half g & 1) of its token of block i in region `blk`
  auto staged = [&](int blk, int i, int j16) {
    const int r = 16 * (i & 1) + l16;
    return (uint2*)(stage + blk * SBLK + r * SROW + swizzled(r, 2 * j16 + (g >> 1)) * 16 + (g & 1) * 8);
  };
  auto settle = [] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };  // the wavefront's writes before its reads
  const int s_row = lane / SC, s_chunk = lane % SC;  // where this lane reads and stores
  auto chunk_of = [&](int blk, int r) { return *(const u32x4*)(stage + blk * SBLK + r * SROW + swizzled(r, s_chunk) * 16); };
  if (MODE == GEMM_PLAIN) {
    const bf16_t* bias = (const bf16_t*)a.bias;
    bf16_t* out = (bf16_t*)a.out;
    const int nw0 = n0 + wn * 64, n_lane = nw0 + 8 * s_chunk;
    const bool has_res = a.residual != nullptr;
    if (has_res) {  // into the staging region, to be replaced by the results in place (it may be the output itself)
      u32x4 rv[T::MI][32 * SC / 64];
#pragma unroll
      for (int i = 0; i < T::MI; ++i)
#pragma unroll
        for (int u = 0; u < 32 * SC / 64; ++u)  // past the end: not used
          rv[i][u] = *(const u32x4*)((const bf16_t*)a.residual + (size_t)min(mw + 32 * i + u * (64 / SC) + s_row, a.m - 1) * a.n + min(n_lane, a.n - 8));
#pragma unroll
      for (int i = 0; i < T::MI; ++i)
#pragma unroll
        for (int u = 0; u < 32 * SC / 64; ++u) {
          const int r = u * (64 / SC) + s_row;
          *(u32x4*)(stage + i * SBLK + r * SROW + swizzled(r, s_chunk) * 16) = rv[i][u];
        }
      settle();
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float b[4] = {0.f, 0.f, 0.f, 0.f}, r[4] = {0.f, 0.f, 0.f, 0.f};
        if (bias != nullptr) {
          const uint2 raw = *(const uint2*)(bias + min(nw0 + j * 16 + 4 * g, a.n - 4));
          b[0] = bf16lo_to_f32(raw.x), b[1] = bf16hi_to_f32(raw.x), b[2] = bf16lo_to_f32(raw.y), b[3] = bf16hi_to_f32(raw.y);
        }
        uint2* const at = staged(i >> 1, i, j);
        if (has_res) {
          const uint2 raw = *at;
          r[0] = bf16lo_to_f32(raw.x), r[1] = bf16hi_to_f32(raw.x), r[2] = bf16lo_to_f32(raw.y), r[3] = bf16hi_to_f32(raw.y);
        }
        bf16x4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = (__bf16)((acc[j][i][e] + b[e]) + r[e]);
        *at = __builtin_bit_cast(uint2, pk);
      }
    settle();
#pragma unroll
    for (int i = 0; i < T::MI; ++i)
#pragma unroll
      for (int u = 0; u < 32 * SC / 64; ++u) {
        const int r = u * (64 / SC) + s_row, m = mw + 32 * i + r;
        if (m < a.m && n_lane < a.n) *(u32x4*)(out + (size_t)m * a.n + n_lane) = chunk_of(i, r);
      }
  } else {  // GEMM_QKV_ROPE
    // head of this wavefront and where its rows go
    const int head = u64 >> 1;
    const int dim0 = (u64 & 1) * 32;  // block 0: dims dim0 + ..., block 1: dim0 + 64 + ...
    const bf16_t* bias = (const bf16_t*)a.bias + (size_t)head * 128;
    bf16_t* dst;
    int heads_dst, head_dst;
    bool rotate = true;
    if (head < a.h_q) dst = (bf16_t*)a.q, heads_dst = a.h_q, head_dst = head;
    else if (head < a.h_q + a.h_kv) dst = (bf16_t*)a.k_out, heads_dst = a.h_kv, head_dst = head - a.h_q;
    else dst = (bf16_t*)a.v_out, heads_dst = a.h_kv, head_dst = head - a.h_q - a.h_kv, rotate = false;
#pragma unroll
    for (int j = 0; j < NJ / 2; ++j) {
      const int f = dim0 + 16 * j + 4 * g;  // rotary frequency index of the run's first element
      float4 cs0[NI], cs1[NI];
      if (rotate) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const float* cs = a.cos_sin + ((size_t)min(mw + i * 16 + l16, a.m - 1) * 64 + f) * 2;
          cs0[i] = *(const float4*)cs, cs1[i] = *(const float4*)(cs + 4);
        }
      }
      float b0[4], b1[4];
      {
        const uint2 r0 = *(const uint2*)(bias + f), r1 = *(const uint2*)(bias + 64 + f);
        b0[0] = bf16lo_to_f32(r0.x), b0[1] = bf16hi_to_f32(r0.x), b0[2] = bf16lo_to_f32(r0.y), b0[3] = bf16hi_to_f32(r0.y);
        b1[0] = bf16lo_to_f32(r1.x), b1[1] = bf16hi_to_f32(r1.x), b1[2] = bf16lo_to_f32(r1.y), b1[3] = bf16hi_to_f32(r1.y);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        float lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) lo[e] = acc[j][i][e] + b0[e], hi[e] = acc[j + 2][i][e] + b1[e];
        if (rotate) {
          const float c[4] = {cs0[i].x, cs0[i].z, cs1[i].x, cs1[i].z}, s[4] = {cs0[i].y, cs0[i].w, cs1[i].y, cs1[i].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) rotate_pair(lo[e], hi[e], c[e], s[e]);
        }
        bf16x4 p0, p1;
#pragma unroll
        for (int e = 0; e < 4; ++e) p0[e] = (__bf16)lo[e], p1[e] = (__bf16)hi[e];
        *staged(2 * (i >> 1), i, j) = __builtin_bit_cast(uint2, p0);
        *staged(2 * (i >> 1) + 1, i, j) = __builtin_bit_cast(uint2, p1);
      }
    }
    settle();
    bf16_t* const col = dst + (size_t)head_dst * 128 + dim0 + 8 * s_chunk;
#pragma unroll
    for (int i = 0; i < T::MI; ++i)
#pragma unroll
      for (int u = 0; u < 32 * SC / 64; ++u) {
        const int r = u * (64 / SC) + s_row, m = mw + 32 * i + r;
        if (m < a.m) {
          bf16_t* const at = col + (size_t)m * heads_dst * 128;
          *(u32x4*)at = chunk_of(2 * i, r);
          *(u32x4*)(at + 64) = chunk_of(2 * i + 1, r);
        }
      }
    if (a.append.k == nullptr || head < a.h_q) return;
    // the same rows into the cache; in the loop above the question cost the launches that append nothing 0.5 %
    const int dim = dim0 + 8 * s_chunk;
#pragma unroll
    for (int i = 0; i < T::MI; ++i)
#pragma unroll
      for (int u = 0; u < 32 * SC / 64; ++u) {
        const int r = u * (64 / SC) + s_row, m = mw + 32 * i + r;
        if (m < a.m) {
          append_chunk(a.append, !rotate, head_dst, m, dim, chunk_of(2 * i, r));
          append_chunk(a.append, !rotate, head_dst, m, dim + 64, chunk_of(2 * i + 1, r));
          if (rotate && dim == 0) append_index(a.append, head_dst, m, a.m);
        }
      }
  }
}

template <int MODE, typename T>
__global__ __launch_bounds__(T::NW * 64) void gemm_bf16_kernel(GemmArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  gemm_tile_product<MODE, T>(a, TileGrid{(int)blockIdx.x, (int)gridDim.x, a.tiles_m, a.tiles_n, a.m_block, 0}, smem);
}

// Two tilings in one launch: whole rounds of T over the first outputs, U over the rest. Blocks start in order, so the smaller
// tiles of the last round follow the larger ones onto the CUs as they become free.
template <int MODE, typename T, typename U>
__global__ __launch_bounds__(T::NW * 64) void gemm_mixed_kernel(GemmArgs a, TileGrid rest) {
  static_assert(T::NW == U::NW, "one workgroup size");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int first = (int)gridDim.x - rest.blocks;  // blocks of T
  if ((int)blockIdx.x < first) {
    gemm_tile_product<MODE, T>(a, TileGrid{(int)blockIdx.x, first, a.tiles_m, a.tiles_n, a.m_block, 0}, smem);
  } else {
    rest.block = (int)blockIdx.x - first;
    gemm_tile_product<MODE, U>(a, rest, smem);
  }
}

// Second launch of a split contraction: sums the chunks' partial tiles in chunk order and applies the mode's store.
// One thread per token and run of 4 outputs (QKV_ROPE: per run of 4 dims of a head's first half and their rotary
// partners).
constexpr int RD_BATCH = 4;  // chunks whose loads are in flight together
template <int MODE, bool APPEND>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmArgs a) {
  const long id = (long)blockIdx.x * 256 + threadIdx.x;
  const int runs = MODE == GEMM_QKV_ROPE ? a.n / 8 : a.n / 4;  // per token
  if (id >= (long)a.m * runs) return;
  const int m = (int)(id / runs), r = (int)(id - (long)m * runs);
  const size_t stride = (size_t)a.m * a.n;
  if (MODE == GEMM_PLAIN) {
    const int n = 4 * r;
    const float* p = a.partial + (size_t)m * a.n + n;
    float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int c0 = 0; c0 < a.split_k; c0 += RD_BATCH) {
      float4 t[RD_BATCH];
#pragma unroll
      for (int u = 0; u < RD_BATCH; ++u) t[u] = *(const float4*)(p + min(c0 + u, a.split_k - 1) * stride);
#pragma unroll
      for (int u = 0; u < RD_BATCH; ++u)
        if (c0 + u < a.split_k) y.x += t[u].x, y.y += t[u].y, y.z += t[u].z, y.w += t[u].w;
    }
    if (a.bias != nullptr) {
      const uint2 raw = *(const uint2*)((const bf16_t*)a.bias + n);
      y.x += bf16lo_to_f32(raw.x), y.y += bf16hi_to_f32(raw.x), y.z += bf16lo_to_f32(raw.y), y.w += bf16hi_to_f32(raw.y);
    }
    if (a.residual != nullptr) {
      const uint2 raw = *(const uint2*)((const bf16_t*)a.residual + (size_t)m * a.n + n);
      y.x += bf16lo_to_f32(raw.x), y.y += bf16hi_to_f32(raw.x), y.z += bf16lo_to_f32(raw.y), y.w += bf16hi_to_f32(raw.y);
    }
    bf16x4 pk;
    pk[0] = (__bf16)y.x, pk[1] = (__bf16)y.y, pk[2] = (__bf16)y.z, pk[3] = (__bf16)y.w;
    *(uint2*)((bf16_t*)a.out + (size_t)m * a.n + n) = __builtin_bit_cast(uint2, pk);
  } else if (MODE == GEMM_QKV_ROPE) {
    const int head = r / 16, f = 4 * (r % 16);  // f: first of 4 rotary frequencies
    const float* p = a.partial + (size_t)m * a.n + head * 128 + f;
    float4 lo4 = make_float4(0.f, 0.f, 0.f, 0.f), hi4 = lo4;
    for (int c0 = 0; c0 < a.split_k; c0 += RD_BATCH) {
      float4 t[RD_BATCH], v[RD_BATCH];
#pragma unroll
      for (int u = 0; u < RD_BATCH; ++u) {
        const float* pc = p + min(c0 + u, a.split_k - 1) * stride;
        t[u] = *(const float4*)pc, v[u] = *(const float4*)(pc + 64);
      }
#pragma unroll
      for (int u = 0; u < RD_BATCH; ++u)
        if (c0 + u < a.split_k) {
          lo4.x += t[u].x, lo4.y += t[u].y, lo4.z += t[u].z, lo4.w += t[u].w;
          hi4.x += v[u].x, hi4.y += v[u].y, hi4.z += v[u].z, hi4.w += v[u].w;
        }
    }
    float lo[4] = {lo4.x, lo4.y, lo4.z, lo4.w}, hi[4] = {hi4.x, hi4.y, hi4.z, hi4.w};
    const bf16_t* bias = (const bf16_t*)a.bias + (size_t)head * 128;
    const uint2 r0 = *(const uint2*)(bias + f), r1 = *(const uint2*)(bias + 64 + f);
    lo[0] += bf16lo_to_f32(r0.x), lo[1] += bf16hi_to_f32(r0.x), lo[2] += bf16lo_to_f32(r0.y), lo[3] += bf16hi_to_f32(r0.y);
    hi[0] += bf16lo_to_f32(r1.x), hi[1] += bf16hi_to_f32(r1.x), hi[2] += bf16lo_to_f32(r1.y), hi[3] += bf16hi_to_f32(r1.y);
    bf16_t* dst;
    int heads_dst, head_dst;
    if (head < a.h_q) dst = (bf16_t*)a.q, heads_dst = a.h_q, head_dst = head;
    else if (head < a.h_q + a.h_kv) dst = (bf16_t*)a.k_out, heads_dst = a.h_kv, head_dst = head - a.h_q;
    else dst = (bf16_t*)a.v_out, heads_dst = a.h_kv, head_dst = head - a.h_q - a.h_kv;
    if (head < a.h_q + a.h_kv) {
      const float4 cs0 = *(const float4*)(a.cos_sin + ((size_t)m * 64 + f) * 2);
      const float4 cs1 = *(const float4*)(a.cos_sin + ((size_t)m * 64 + f + 2) * 2);
      const float c[4] = {cs0.x, cs0.z, cs1.x, cs1.z}, sn[4] = {cs0.y, cs0.w, cs1.y, cs1.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) rotate_pair(lo[e], hi[e], c[e], sn[e]);
    }
    bf16x4 p0, p1;
#pragma unroll
    for (int e = 0; e < 4; ++e) p0[e] = (__bf16)lo[e], p1[e] = (__bf16)hi[e];
    bf16_t* row = dst + ((size_t)m * heads_dst + head_dst) * 128;
    *(uint2*)(row + f) = __builtin_bit_cast(uint2, p0);
    *(uint2*)(row + 64 + f) = __builtin_bit_cast(uint2, p1);
    if (APPEND && head >= a.h_q) {
      const bool is_v = head >= a.h_q + a.h_kv;
      append_run(a.append, is_v, head_dst, m, f, __builtin_bit_cast(uint2, p0));
      append_run(a.append, is_v, head_dst, m, f + 64, __builtin_bit_cast(uint2, p1));
      if (!is_v && f == 0) append_index(a.append, head_dst, m, a.m);
    }
  }
}

// The PLAIN reduction with the RMSNorm of its result behind it (the layer's o_proj before the second norm): a workgroup
// per token holds the row, rounded as stored, between the sums and the scaling. As two launches the norm of 64 tokens
// cost 5.9 us, nearly all of it the start of one more dependent launch: 7B layer, 64 tokens 223.8 -> 218.4 us.
constexpr int RNK_THREADS = 512;
constexpr int RNK_RUNS = 4;  // runs of 4 outputs per thread: rows of up to 8192
__global__ __launch_bounds__(RNK_THREADS) void gemm_reduce_norm_kernel(GemmArgs a, const bf16_t* __restrict__ norm_w,
                                                                       bf16_t* __restrict__ norm_out, float eps) {
  __shared__ float wave_ss[RNK_THREADS / 64];
  const int m = blockIdx.x, tid = threadIdx.x, runs = a.n / 4;
  const size_t stride = (size_t)a.m * a.n;
  uint2 row[RNK_RUNS], wv[RNK_RUNS];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < RNK_RUNS; ++i) {
    const int r = tid + i * RNK_THREADS;
    if (r >= runs) continue;
    const float* p = a.partial + (size_t)m * a.n + 4 * r;
    wv[i] = *(const uint2*)(norm_w + 4 * r);
    const uint2 raw = a.residual != nullptr ? *(const uint2*)((const bf16_t*)a.residual + (size_t)m * a.n + 4 * r) : make_uint2(0u, 0u);
    float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int c0 = 0; c0 < a.split_k; c0 += 2 * RD_BATCH) {
      float4 t[2 * RD_BATCH];
#pragma unroll
      for (int u = 0; u < 2 * RD_BATCH; ++u) t[u] = *(const float4*)(p + min(c0 + u, a.split_k - 1) * stride);
#pragma unroll
      for (int u = 0; u < 2 * RD_BATCH; ++u)
        if (c0 + u < a.split_k) y.x += t[u].x, y.y += t[u].y, y.z += t[u].z, y.w += t[u].w;
    }
    y.x += bf16lo_to_f32(raw.x), y.y += bf16hi_to_f32(raw.x), y.z += bf16lo_to_f32(raw.y), y.w += bf16hi_to_f32(raw.y);
    bf16x4 pk;
    pk[0] = (__bf16)y.x, pk[1] = (__bf16)y.y, pk[2] = (__bf16)y.z, pk[3] = (__bf16)y.w;
    row[i] = __builtin_bit_cast(uint2, pk);
    *(uint2*)((bf16_t*)a.out + (size_t)m * a.n + 4 * r) = row[i];
    const float f[4] = {bf16lo_to_f32(row[i].x), bf16hi_to_f32(row[i].x), bf16lo_to_f32(row[i].y), bf16hi_to_f32(row[i].y)};
#pragma unroll
    for (int e = 0; e < 4; ++e) ss = fmaf(f[e], f[e], ss);
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) wave_ss[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < RNK_THREADS / 64; ++w) tot += wave_ss[w];
  const float inv = 1.f / sqrtf(tot / (float)a.n + eps);
#pragma unroll
  for (int i = 0; i < RNK_RUNS; ++i) {
    const int r = tid + i * RNK_THREADS;
    if (r >= runs) continue;
    uint2 o;
    o.x = (uint32_t)f32_to_bf16_rne(bf16lo_to_f32(row[i].x) * inv * bf16lo_to_f32(wv[i].x)) |
          ((uint32_t)f32_to_bf16_rne(bf16hi_to_f32(row[i].x) * inv * bf16hi_to_f32(wv[i].x)) << 16);
    o.y = (uint32_t)f32_to_bf16_rne(bf16lo_to_f32(row[i].y) * inv * bf16lo_to_f32(wv[i].y)) |
          ((uint32_t)f32_to_bf16_rne(bf16hi_to_f32(row[i].y) * inv * bf16hi_to_f32(wv[i].y)) << 16);
    *(uint2*)(norm_out + (size_t)m * a.n + 4 * r) = o;
  }
}

bool gemm_supported(const GemmArgs& a, int mode) {
  if (a.m <= 0 || a.n <= 0 || a.k <= 0 || a.k % 64 != 0) return false;
  // byte offsets inside a tile's row range are 32-bit (plus the k offset of the step)
  const size_t span = (size_t)(mode == GEMM_SWIGLU ? a.n / 2 + GM_BN : GM_BN) * a.k * 2 + (size_t)a.k * 2;  // GM_BN >= BM
  if (span >= ((size_t)1 << 32)) return false;
  if (mode == GEMM_PLAIN) return a.n % 8 == 0;
  if (mode == GEMM_QKV_ROPE) return a.h_q > 0 && a.h_kv > 0 && a.n == (a.h_q + 2 * a.h_kv) * 128 && a.n % GM_BN == 0;
  if (mode == GEMM_SWIGLU) return a.n % (2 * 128) == 0 && a.n % GM_BN == 0;
  return false;
}

static std::atomic<int> g_forced_tile_rows{0};  // 0: choose per launch; 128 / 256: tests cover both tilings
void gemm_force_tile_rows(int rows) { g_forced_tile_rows.store(rows, std::memory_order_relaxed); }

// The tiling that finishes soonest: a launch lasts ceil(tiles / CUs) rounds of one tile each. A tile's time by its size,
// measured per 64-wide k-step with one workgroup per CU and weights from HBM: 256 x 256 1.36 us, 128 x 256 0.82, 128 x 128 0.54
// (one weight: 1.39, 0.76, 0.44; the costs below are of a loop of 32 x 32 x 16 products, 1.55, 0.96 and 0.60 us, and still fit). Fewer
// products per fragment read and per request, so small tiles pay only where they fill CUs that the larger leave idle:
// 7B o_proj at 700 tokens, 84 / 168 tiles, 47 -> 31 us; 72B down at 512, 128 / 256 tiles, 413 -> 281 us.
//
// Whole rounds of the large tile may be followed by a round of a smaller one instead of one that is mostly empty: the first
// `wide` weight tiles of 256 outputs then make the whole rounds and the others take the smaller tile, in the same launch.
// A tile's products walk k in the same order in every tiling, so the results are the same bits. us one tiling (the better of 256
// and 128 token rows) / mixed, weights from HBM: SwiGLU 512 x 37888 x 3584 (1 round and 160 tiles of 128 x 128) 162 / 126, 1500 324 /
// 310, 4096 824 / 778; 4096 x 59136 x 8192 (14 and 224 of 128 x 256) 2738 / 2644; plain 2048 / 4096 x 10240 x 8192 302 / 256 and
// 511 / 473; 5000 x 3584 x 18944 697 / 545; 4096 x 4608 x 3584 137 / 116. An estimate within 1.5 % keeps one tiling.
struct TileChoice {
  int rows, cols;
  double cost;  // of the launch, in 256 x 256 tiles one after the other
  int wide;     // 0, or weight tiles of 256 x 256 before the tiles of rest_cols
  int rest_cols;
};
static TileChoice gemm_tile(const GemmArgs& a) {
  const int forced = g_forced_tile_rows.load(std::memory_order_relaxed);
  if (forced != 0) return {forced, GM_BN, 0, 0, 0};
  static const struct {
    int rows, cols;
    double cost;
  } kinds[] = {{256, 256, 1.0}, {128, 256, 0.62}, {128, 128, 0.39}};
  const int cus = device_cu_count();
  TileChoice best{256, 256, 0, 0, 0};
  double best_cost = 1e30;
  for (const auto& t : kinds) {
    const long tiles = (long)((a.m + t.rows - 1) / t.rows) * ((a.n + t.cols - 1) / t.cols);
    const double cost = t.cost * (double)((tiles + cus - 1) / cus);
    if (cost < best_cost) best_cost = cost, best = {t.rows, t.cols, cost, 0, 0};
  }
  const long tiles_m = (a.m + 255) / 256, tiles_n = (a.n + 255) / 256;
  const long rounds = tiles_m * tiles_n / cus;
  const long wide = rounds * cus / tiles_m;
  if (rounds > 0 && wide > 0 && wide < tiles_n)
    for (int k = 1; k < 3; ++k) {
      const auto& t = kinds[k];
      const long tiles = (long)((a.m + t.rows - 1) / t.rows) * ((a.n - 256 * wide + t.cols - 1) / t.cols);
      const double cost = (double)rounds + t.cost * (double)((tiles + cus - 1) / cus);
      if (cost < 0.985 * best_cost) best_cost = cost, best = {256, 256, cost, (int)wide, t.cols};
    }
  return best;
}
int gemm_tile_rows(const GemmArgs& a) { return gemm_tile(a).rows; }
int gemm_tile_cols(const GemmArgs& a) { return gemm_tile(a).cols; }
int gemm_tile_blocks(const GemmArgs& a) {
  const TileChoice t = gemm_tile(a);
  auto blocks = [&](long m, long n) { return (int)(((a.m + m - 1) / m * n + 7) / 8 * 8); };
  if (t.wide == 0) return blocks(t.rows, (a.n + t.cols - 1) / t.cols);
  return blocks(256, t.wide) + blocks(128, (a.n - 256 * t.wide + t.rest_cols - 1) / t.rest_cols);
}

// Contraction split: launches whose tiles would occupy at most a quarter of the CUs (few tokens against a long k:
// text chunks and decode steps through the layer, where the weights are streamed once and HBM is the bound) deal the
// k-steps to chunks, at most one workgroup per CU in all, at least 4 steps per chunk, as many chunks as the scratch holds.
// One chunk more, rounded up, starts its last workgroups only when others end: 72B QKV at 64 tokens, 40 tiles, 7 chunks
// (280 workgroups) 54.0 us, 6 chunks 41.4; 100 x 14336 x 4096 5 chunks of 56 tiles 49.5, 4 chunks 34.7.
//
// With 256-wide tiles a matrix of few outputs needs many chunks for that, and every chunk writes and re-reads an f32
// copy of the output: the 7B down projection at 64 tokens moved 34 MB of partials beside 136 MB of weights, and each
// workgroup had 16 steps to hide its start behind. Where more than NARROW_ABOVE chunks would be wanted (fewer than 32
// wide tiles: 7B o_proj and down up to 256 tokens, 7B QKV up to 128), tiles of 64 outputs are taken instead, in the
// largest power of two of chunks that keeps tiles x chunks at 2.25 per CU (3, 6, 7 and 9 chunks measured up to a third
// slower on the down projection than 4 and 8), at most NARROW_ABOVE. us at 7B sizes, wide tiles / 64 outputs, 64 tokens:
// QKV 25.7 / 18.1, o_proj 22.4 / 13.7, down 63.3 / 36.8; 128 tokens 33.2 / 24.7, 29.9 / 17.8, 78.3 / 47.5; 200 tokens
// o_proj 31.5 / 20.6, down 73.8 / 63.1; 3 tokens 19.8 / 13.2, 17.0 / 11.6, 53.9 / 29.0. At 72B sizes (8 chunks or fewer)
// the wide tiles are as fast or faster and stay: o_proj at 64 tokens 34.7 against 35.3-39.3, down 97.9 against 101-120.
// So does SwiGLU, which is not split. The 2.25: with 72 tiles (576 workgroups in 8 chunks) 8 chunks against 4 take 23.8 /
// 26.5 us at 40 tokens and k = 8192, 31.8 / 35.3 at 100 tokens, but 13.4 / 13.3 and 19.9 / 17.8 at k = 3584; with 80
// tiles, which take 4, 24.5 / 27.2 and 34.0 / 36.1, but 14.1 / 13.4 and 20.1 / 18.0: the line lies where long and short
// contractions lose about as much.
//
// Above a quarter of the CUs a product without fused steps is still split where two or three chunks of its 128 x 256 tiles
// fill the chip (at least 4/5 of it, one round) and the estimate, with the tile times above and the partial sums at 4.5 TB/s,
// is a tenth below the unsplit one: long contractions whose tiles leave CUs idle or are small ones. (The estimate's 1.55 and 0.95
// us per step are those of the loop of 32 x 32 x 16 products, both about 1.15 times the present ones.) us unsplit / split, weights from HBM:
// 3584 x 18944 at 520 tokens 136 / 89, 640 160 / 104, 768 157 / 105, 900 137 / 122, 1024 158 / 142, 1100 155 / 143; 8192 x
// 29568 at 400 268 / 211, 512 276 / 243. At k = 3584 (o_proj) there is nothing to gain.
//
// Of these products of few outputs, long contractions take tiles of 128 outputs instead (64 or 128 token rows), one workgroup
// per CU, dealt to the XCDs by items as the 256-wide ones are: an activation fragment read meets twice the outputs and a
// request brings twice the weights, and a chunk of a long contraction still has the steps to hide its start. us 64 outputs /
// 128, weights from HBM: 3584 x 18944 at 16 tokens 28.8 / 28.1, 64 35.7 / 31.1, 100 42.5 / 35.1, 128 46.3 / 37.8, 200 61.0 /
// 50.2, 250 70.8 / 55.7; 5120 x 13824 at 64 and 128 44.0 / 32.7 and 58.7 / 38.6; 3584 x 5120 at 64 and 128 16.0 / 15.1 and 21.6 /
// 19.5. They need at least 5/8 of the CUs: 2560 outputs at 64 tokens, 160 workgroups, 16.9 / 15.8; 2048, 128 of them, 14.2 / 15.7.
// Up to 32 tokens, where fewer requests are for activations, they need more than 160 of 256: 2560 x 9728 at 3, 16, 32 and 48 tokens
// 17.9 / 18.4, 18.6 / 19.1, 19.7 / 19.7, 21.0 / 20.6; 2816 x 18944, 176 workgroups, at 3 and 16 28.8 / 28.4, 29.7 / 29.3.
// With shorter contractions 64 outputs stay: at k = 3584 8 chunks of 28 tiles of 128 take 13.5 and of 56 tiles of 64 13.5-13.8.
// There, up to 64 tokens, half as many chunks fill the chip if 4 of them make 7/8 to all of a workgroup per CU, with a ring of
// 5 slots in the room of the second one, and leave half the partial sums: 3584 x 3584 at 64 and 16 tokens 13.8 / 12.2 and 11.5 /
// 10.1 (with 3 slots no gain). 4 chunks of fewer tiles lose (2048 x 8192, 128 workgroups, 14.2 / 16.9).
// Both rules are for PLAIN: other chunks add in another order, and QKV's sums decide which near-tied keys are kept.
constexpr int NARROW_ABOVE = 8;
constexpr int MID_STEPS = 80;  // k-steps from which a contraction is long
GemmSplit gemm_plan_split(const GemmArgs& a, int mode, size_t scratch_bytes) {
  GemmSplit p{1, a.k / GM_BK, 0, 0, 0};
  if (mode == GEMM_SWIGLU || scratch_bytes == 0 || gemm_uses_gemv(a)) return p;
  const int rows = gemm_tile_rows(a), cus = device_cu_count();
  const long tiles_m = (a.m + rows - 1) / rows, tiles = tiles_m * ((a.n + GM_BN - 1) / GM_BN);
  const int steps = a.k / GM_BK;
  if (tiles * 4 > cus && mode == GEMM_PLAIN && g_forced_tile_rows.load(std::memory_order_relaxed) == 0) {
    const long halves = (long)((a.m + 127) / 128) * ((a.n + GM_BN - 1) / GM_BN);  // tiles of 128 x 256
    const double us = 1.55 * gemm_tile(a).cost * steps;  // unsplit
    const size_t per_chunk = (size_t)a.m * a.n * sizeof(float);
    for (int want = 2; want <= 3; ++want) {
      const long wgs = halves * want;
      if (wgs > cus || wgs * 5 < (long)cus * 4 || want * per_chunk > scratch_bytes || steps < 4 * want) continue;
      const int per = (steps + want - 1) / want;
      if (0.95 * per + 4 + 2.0 * want * per_chunk / 4.5e6 > 0.9 * us) continue;
      p.steps_per_split = per;
      p.split_k = (steps + per - 1) / per;
      p.scratch_bytes = (size_t)p.split_k * per_chunk;
      p.halves = 1;
      return p;
    }
  }
  if (tiles * 4 > cus || steps < 8) return p;
  long want = (cus + tiles - 1) / tiles;
  if (want > steps / 4) want = steps / 4;
  const bool few_outputs = want > NARROW_ABOVE;
  if (want > cus / tiles) want = cus / tiles;
  const size_t per_chunk = (size_t)a.m * a.n * sizeof(float);
  if (few_outputs && rows == 128 && g_forced_tile_rows.load(std::memory_order_relaxed) == 0) {
    const long mid = tiles_m * ((a.n + Mid::BN - 1) / Mid::BN);
    long mid_want = std::min<long>(NARROW_ABOVE, cus / mid);
    if ((size_t)mid_want * per_chunk > scratch_bytes) mid_want = (long)(scratch_bytes / per_chunk);
    if (mode == GEMM_PLAIN && steps >= MID_STEPS && mid_want >= 2 && mid * mid_want * 8 >= (long)cus * 5 + (a.m <= 32 ? 1 : 0)) {
      want = mid_want;
      p.narrow = Mid::BN;
    } else {
      const long narrow = tiles_m * ((a.n + Narrow64::BN - 1) / Narrow64::BN);
      want = NARROW_ABOVE;
      while (want > 1 && narrow * want > 2 * cus + cus / 4) want /= 2;  // a quarter of a chip above: 72 tiles x 8 measured better than x 4
      if (mode == GEMM_PLAIN && want == 8 && a.m <= 64 && narrow * 4 <= cus && narrow * 4 * 8 >= (long)cus * 7) want = 4;
      p.narrow = Narrow64::BN;
    }
  }
  if ((size_t)want * per_chunk > scratch_bytes) want = (long)(scratch_bytes / per_chunk);
  if (want < 2) return GemmSplit{1, steps, 0, 0, 0};
  p.steps_per_split = (int)((steps + want - 1) / want);
  p.split_k = (steps + p.steps_per_split - 1) / p.steps_per_split;  // every chunk non-empty
  p.scratch_bytes = (size_t)p.split_k * per_chunk;
  return p;
}

template <int MODE, typename T>
static hipError_t launch_tile(GemmArgs a, hipStream_t s) {
  static bool attr_done[QP_MAX_DEVICES] = {};
  const int dev = current_device();
  if (dev < 0) return hipErrorInvalidDevice;
  const int lds = T::LDS;
  if (!attr_done[dev]) {
    hipError_t e = hipFuncSetAttribute((const void*)gemm_bf16_kernel<MODE, T>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_done[dev] = true;
  }
  a.tiles_m = (a.m + T::BM - 1) / T::BM;
  a.tiles_n = (a.n + T::BN - 1) / T::BN;
  a.m_block = a.tiles_m < 8 ? a.tiles_m : 8;
  const long tiles = (long)a.tiles_m * a.tiles_n;
  // Tiles of one workgroup per CU that are few and no multiple of 8 leave XCDs short if only they are dealt: 42 tiles x 6
  // chunks were 36 workgroups on seven XCDs of 32 CUs and none on the last. us dealt by tiles / by items: 3584 x 18944 at
  // 257 / 300 / 384 tokens 90 / 96 / 107 -> 59 / 62 / 69; 4608 x 3584 at 160 / 256 32 / 38 -> 23 / 26. Narrow tiles, two and
  // three to a CU, have the room: 4608 x 3584 at 128 tokens 24.0, by items 25.1. Chunk by chunk an XCD would read one range
  // of k of all rows, and rows 16 KB apart then meet in few memory channels: 8192 x 8192 at 3 tokens 29.5 -> 32.7.
  // So deals_items deals the items; the grid is the same either way, and what it has too much ends at once.
  const dim3 grid((unsigned)((tiles + 7) / 8 * 8), a.split_k);
  hipLaunchKernelGGL((gemm_bf16_kernel<MODE, T>), grid, dim3(T::NW * 64), lds, s, a);
  return hipSuccess;
}

template <int MODE, typename U>
static hipError_t launch_mixed(GemmArgs a, int wide, hipStream_t s) {
  typedef Tile256 T;
  static bool attr_done[QP_MAX_DEVICES] = {};
  const int dev = current_device();
  if (dev < 0) return hipErrorInvalidDevice;
  constexpr int lds = T::LDS > U::LDS ? T::LDS : U::LDS;
  if (!attr_done[dev]) {
    hipError_t e = hipFuncSetAttribute((const void*)gemm_mixed_kernel<MODE, T, U>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_done[dev] = true;
  }
  auto blocks = [](long tiles) { return (int)((tiles + 7) / 8 * 8); };
  a.tiles_m = (a.m + T::BM - 1) / T::BM;
  a.tiles_n = wide;
  a.m_block = a.tiles_m < 8 ? a.tiles_m : 8;
  TileGrid rest{};
  rest.n_first = wide * T::BN;
  rest.tiles_m = (a.m + U::BM - 1) / U::BM;
  rest.tiles_n = (a.n - rest.n_first + U::BN - 1) / U::BN;
  rest.m_block = rest.tiles_m < 8 ? rest.tiles_m : 8;
  rest.blocks = blocks((long)rest.tiles_m * rest.tiles_n);
  hipLaunchKernelGGL((gemm_mixed_kernel<MODE, T, U>), dim3((unsigned)(blocks((long)a.tiles_m * wide) + rest.blocks)), dim3(T::NW * 64),
                     lds, s, a, rest);
  return hipSuccess;
}

// reduce = false leaves a split product's partial sums to the caller (a.split_k says whether there are any)
template <int MODE>
static hipError_t launch_mode(GemmArgs& a, void* scratch, size_t scratch_bytes, hipStream_t s, bool reduce = true) {
  const GemmSplit sp = gemm_plan_split(a, MODE, scratch != nullptr ? scratch_bytes : 0);
  a.split_k = sp.split_k, a.steps_per_split = sp.steps_per_split, a.partial = (float*)scratch;
  hipError_t e;
  if (sp.narrow == Mid::BN) {  // PLAIN only
    if constexpr (MODE == GEMM_PLAIN) e = a.m <= 64 ? launch_tile<MODE, Mid64>(a, s) : launch_tile<MODE, Mid>(a, s);
    else e = hipErrorInvalidValue;
  } else if (sp.narrow) {  // never for SWIGLU, which is not split
    if constexpr (MODE != GEMM_SWIGLU) {
      if (a.m > 64) e = launch_tile<MODE, Narrow128>(a, s);
      // up to one workgroup per CU there is room for a deeper ring
      else if ((a.n + Deep64::BN - 1) / Deep64::BN * a.split_k <= device_cu_count()) e = launch_tile<MODE, Deep64>(a, s);
      else e = launch_tile<MODE, Narrow64>(a, s);
    } else {
      e = hipErrorInvalidValue;
    }
  } else if (a.split_k == 1 && gemm_tile(a).wide > 0) {
    const TileChoice t = gemm_tile(a);
    e = t.rest_cols == 128 ? launch_mixed<MODE, Mid>(a, t.wide, s) : launch_mixed<MODE, Tile128>(a, t.wide, s);
  } else if (a.split_k == 1 && gemm_tile_cols(a) == 128) {
    e = launch_tile<MODE, Mid>(a, s);
  } else if (MODE == GEMM_SWIGLU && a.m <= 64 && gemm_tile_rows(a) == 128 && g_forced_tile_rows.load(std::memory_order_relaxed) == 0) {
    // 64 token rows instead of 128 that are half padding, a slot more in the ring. us 128 / 64 rows, weights from HBM: 37888 x
    // 3584 at 5, 16, 40 and 64 tokens 53.4 / 50.7, 53.7 / 51.5, 55.9 / 54.1, 57.7 / 56.5 (tiles of 128 outputs 58-66, of 64 52-62:
    // more requests for the same activations); 59136 x 8192 at 30 and 64 171.4 / 169.9, 173.6 / 172.2.
    if constexpr (MODE == GEMM_SWIGLU) e = launch_tile<MODE, Wide64>(a, s);
    else e = hipErrorInvalidValue;
  } else {
    e = sp.halves || gemm_tile_rows(a) == 128 ? launch_tile<MODE, Tile128>(a, s) : launch_tile<MODE, Tile256>(a, s);
  }
  if (e != hipSuccess || a.split_k == 1 || !reduce) return e;
  const long threads = (long)a.m * (MODE == GEMM_QKV_ROPE ? a.n / 8 : a.n / 4);
  const dim3 grid((unsigned)((threads + 255) / 256));
  if (MODE == GEMM_QKV_ROPE && a.append.k != nullptr) hipLaunchKernelGGL((gemm_reduce_kernel<MODE, MODE == GEMM_QKV_ROPE>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((gemm_reduce_kernel<MODE, false>), grid, dim3(256), 0, s, a);
  return hipSuccess;
}

// A handful of tokens take the weight-streaming kernel (gemv_bf16.hip) unless a tiling is forced (tests then reach
// the split contraction of this kernel at those sizes too).
bool gemm_uses_gemv(const GemmArgs& a) {
  return gemv_applies(a) && g_forced_tile_rows.load(std::memory_order_relaxed) == 0;
}

hipError_t launch_gemm_norm(const GemmArgs& a_in, const void* norm_w, void* norm_out, float eps, void* scratch,
                            size_t scratch_bytes, hipStream_t s) {
  GemmArgs a = a_in;
  a.split_k = 1;
  const bool fits = a.n <= 4 * RNK_RUNS * RNK_THREADS && a.bias == nullptr;
  const hipError_t e = gemm_uses_gemv(a) ? launch_gemv_bf16(a, GEMM_PLAIN, s)
                                         : launch_mode<GEMM_PLAIN>(a, scratch, scratch_bytes, s, !fits);
  if (e != hipSuccess) return e;
  if (fits && a.split_k > 1)
    hipLaunchKernelGGL(gemm_reduce_norm_kernel, dim3((unsigned)a.m), dim3(RNK_THREADS), 0, s, a, (const bf16_t*)norm_w,
                       (bf16_t*)norm_out, eps);
  else
    launch_rms_norm(a.out, norm_w, norm_out, a.m, a.n, eps, s);
  return hipSuccess;
}

hipError_t launch_gemm_bf16(const GemmArgs& a_in, int mode, void* scratch, size_t scratch_bytes, hipStream_t s) {
  GemmArgs a = a_in;
  if (gemm_uses_gemv(a)) return launch_gemv_bf16(a, mode, s);
  switch (mode) {
    case GEMM_PLAIN: return launch_mode<GEMM_PLAIN>(a, scratch, scratch_bytes, s);
    case GEMM_QKV_ROPE: return launch_mode<GEMM_QKV_ROPE>(a, scratch, scratch_bytes, s);
    case GEMM_SWIGLU: return launch_mode<GEMM_SWIGLU>(a, nullptr, 0, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace qp
