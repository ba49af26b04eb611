// Tile attention on the matrix cores (paper Section 2.1 "full attention" over one tile's
// T x tile_h x tile_w tokens; Section 3: tiles exchange no Q/K/V).
//
// Flash-style: a workgroup of 8 wavefronts owns 256 query rows of one head (32 per wavefront) and
// streams the tile's keys and values through a 4-stage LDS ring, 64 keys per stage, filled by
// direct global->LDS transfers; the N x N score matrix is never stored.  All products are bf16
// MFMA (32x32x16) with fp32 accumulation, softmax statistics are fp32.
//
// Transposed products keep every value in its lane between the two GEMMs:  S^T = K Q^T  puts one
// query per lane column (lane l holds query l%32, 16 keys of a 32-key block in its accumulator
// registers), so the exponentials, packed to bf16, already sit in the B-operand layout of
// O^T = V^T P^T.  V^T fragments come out of LDS through the transposing read (ds_read_b64_tr_b16);
// K and V rows are stored with XOR-swizzled 16-byte chunks so both fragment reads are free of bank
// conflicts.
//
// Vector work beside the MFMAs costs issue slots and, on a power-limited part, clock, so the softmax is
// cut to one exponential, one add and half a convert per score:  Q is pre-multiplied by log2(e)*scale (one bf16 rounding)
// and the score accumulators start at -M, the softmax reference, so the MFMA result is the
// exponent itself.  M is an online-softmax running maximum refreshed lazily (see Softmax below).
// A SIMD overlaps MFMA and vector work only across wavefronts, never inside one, so the two
// wavefronts of each SIMD run half an iteration apart (see "Schedule" in the kernel).
//
// A NaN in Q, K or V reaches every output that depends on it: maxima pass it by, exponentials and sums carry it.
#include <type_traits>
#include <atomic>
#include "attention_common.h"

namespace sg {
namespace {

#define SG_INLINE __attribute__((always_inline))   // on the kernel's lambdas: a lambda left as a call pins every captured array in memory

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kBR = kWaves * 32;   // query rows per workgroup
constexpr int kBC = 64;            // keys per stage
constexpr int kStages = 4;
constexpr int kXcd = 8;
constexpr int kRowBytes = 256;
constexpr int kTileBytes = kBC * kRowBytes;          // one K (or V) stage: 16 KiB
constexpr int kVRegion = kStages * kTileBytes;       // V stages start at 64 KiB
constexpr int kLdsBytes = 2 * kStages * kTileBytes;  // 128 KiB

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N == 0 || N == 4 || N == 8 || N == 12, "");
  if (N == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (N == 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  if (N == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  if (N == 12) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
}
__device__ __forceinline__ void meet() {  // workgroup barrier that nothing is scheduled across
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Softmax state of one query (replicated in lanes l and l^32).  Scores leave the MFMA already in the
// exponent domain: t = log2(e) * scale * <q, k> - M, because Q is pre-multiplied by log2(e) * scale and
// the accumulator of the first MFMA of each chain starts at -M (M = the reference the exponentials are
// taken against).  M is an online-softmax running maximum that is refreshed lazily: as long as no
// exponential of a stage exceeds 2^16 the reference stays, so the common path needs no row maximum, no
// subtraction and no rescaling of the output accumulators; the result is the same softmax, since any
// common reference cancels in sum(p v) / sum(p).  (Sums of p v stay finite for |v| below 2^111: p < 2^16.)
// LATE kernels keep Q as stored, scale behind the product and take M as the true running maximum (see late_half).
// Score and probability arrays have this fixed extent for either head_dim (NB <= kMaxSB blocks are used):
// their types then do not depend on a template parameter, which the register-pinning asm statements need.
constexpr int kMaxSB = 4;

struct Softmax {
  float M;   // reference, log2 domain
  float l;   // this lane's share of sum(p)
};

// Scores of keys at or beyond n_keys become -inf.  Branch- and compare-free (sign mask + bit select), so the
// 16 NB decisions do not each occupy a pair of scalar registers.
// Register (kb, r) holds row R = 8 (r >> 2) + 4 half + (r & 3) of its block: key 32 kb + R of the stage (head_dim 128), or key
// 2 (32 (kb >> 1) + R) + (kb & 1) (head_dim 64, two keys per slot).
template <int NB>
__device__ __forceinline__ void mask_tail(f32x16 (&t)[kMaxSB], const int key0, const int n_keys) {
  const int half = (threadIdx.x & 63) >> 5;
  const int limit = n_keys - key0 - (NB == 2 ? 4 : 8) * half;
#pragma unroll
  for (int kb = 0; kb < NB; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = 8 * (r >> 2) + (r & 3);
      const int c = (NB == 2) ? 32 * kb + row : 2 * (32 * (kb >> 1) + row) + (kb & 1);
      const uint32_t beyond = (uint32_t)((limit - 1 - c) >> 31);   // all ones if c >= limit
      t[kb][r] = __uint_as_float((__float_as_uint(t[kb][r]) & ~beyond) | (0xff800000u & beyond));
    }
}

// p[2 kb + h] = bf16(exp2(t[kb][8h..8h+7])) in B-operand order for blocks B0 .. B0 + NB - 1; returns this lane's sum of the exponentials
template <int NB, int B0 = 0>
__device__ __forceinline__ float exp_block(const f32x16 (&t)[kMaxSB], bf16x8 (&p)[2 * kMaxSB]) {
  float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
  for (int kb = B0; kb < B0 + NB; ++kb)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float e[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) e[r] = __builtin_amdgcn_exp2f(t[kb][8 * h + r]);
#pragma unroll
      for (int r = 0; r < 8; ++r) p[2 * kb + h][r] = (__bf16)e[r];
#pragma unroll
      for (int r = 0; r < 8; r += 2) { sum0 += e[r]; sum1 += e[r + 1]; }
    }
  return sum0 + sum1;
}
// row maximum of blocks B0 .. B0 + NB - 1 of the stage for this lane's query, combined over both halves of the wavefront
template <int NB, int B0 = 0>
__device__ __forceinline__ float block_max(const f32x16 (&t)[kMaxSB]) {
  float mx0 = t[B0][0], mx1 = t[B0 + 1][0];
#pragma unroll
  for (int r = 1; r < 15; r += 2) {
    mx0 = fmaxf(fmaxf(mx0, t[B0][r]), t[B0][r + 1]);
    mx1 = fmaxf(fmaxf(mx1, t[B0 + 1][r]), t[B0 + 1][r + 1]);
  }
  mx0 = fmaxf(mx0, t[B0][15]);
  mx1 = fmaxf(mx1, t[B0 + 1][15]);
#pragma unroll
  for (int kb = B0 + 2; kb < B0 + NB; ++kb) {
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      if (kb & 1) mx1 = fmaxf(fmaxf(mx1, t[kb][r]), t[kb][r + 1]);
      else mx0 = fmaxf(fmaxf(mx0, t[kb][r]), t[kb][r + 1]);
    }
  }
  const float mx = fmaxf(mx0, mx1);
  const uint32_t mu = __float_as_uint(mx);
  const auto sw = __builtin_amdgcn_permlane32_swap(mu, mu, false, false);
  return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}
__device__ __forceinline__ f32x16 zero16() {
  return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}
constexpr float kOverflowGuard = 65536.0f;   // a stage's exponentials may grow to 2^16 before the reference moves

// Packed tile; window of a canvas; window that does not cross a canvas edge and whose width is a multiple of 8 (see the DMA loader).
enum { kLinear = 0, kWindow = 1, kWalk = 2 };

// LATE: Q is multiplied as stored and the scores by log2(e) * scale in fp32, against the true running maximum; the other forms scale
// Q first and keep a lazy reference.
// REFRESH: the launch also refreshes the cache of the tiles it attends (packed tiles: refresh <- the tile's Q, K, V,
// has_cache <- 1).
// SHORT: tiles of few stages.  Beside its stages a workgroup of 1,000 tokens spent two fifths of its 70,000 cycles on code that is
// fetched for an iteration or two - 3,600 cycles an iteration before the steady loop, 4,900 on the first behind it, 2,700 inside - and this
// form has one copy of an iteration for all of them.  Where both are warm it is up to 5 % slower an iteration (scalar branches, scalar registers
// spilled).
template <int D, int MODE, bool LATE, bool REFRESH, bool SHORT>
__global__ __launch_bounds__(kThreads) void attention_bf16_kernel(const View16 vw, const float c_log2, const int heads,
                                                                  const int n_qblocks, const int n_tiles, const int cu_per_xcd,
                                                                  const AttnTable tab, const uint8_t* __restrict__ run_flags,
                                                                  uint8_t* __restrict__ has_cache) {
  static_assert(D == 128 || D == 64, "head_dim 64 or 128");
  static_assert(!REFRESH || MODE == kLinear, "a packed tile's input is refreshed");
  static_assert(MODE != kWalk || (D == 128 && !LATE), "head_dim 64 and late scaling: packed tiles and planned windows");
  // LDS rows ("slots") are always 256 bytes.  With head_dim 128 a slot is one key and a stage 64 keys; with
  // head_dim 64 a stage is 128 keys and slot s holds the keys 2 s and 2 s + 1, neighbours in a tile row, so the
  // transfers, the fragment reads and the MFMA count per stage are the same and only the pairing of
  // fragments with accumulators differs (see qk and pv).
  constexpr int kSB = (D == 128) ? 2 : 4;   // 32-key score blocks per stage
  constexpr int kKeys = 32 * kSB;           // keys per stage
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  SG_LDS uint8_t* const lds = (SG_LDS uint8_t*)smem;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

  // Work = (active tile, head, query block) triples, query block fastest.  Workgroups are dealt round-robin
  // to the 8 XCDs; renumber so that each XCD walks a contiguous range of the work and its CUs stream the same
  // head's K/V through one L2.  Only the tiles whose run flag is set are numbered, so the work is spread
  // evenly over the XCDs whichever tiles the gate reuses; the rest of the grid exits here.
  const uint32_t active = attn_active_mask(run_flags, n_tiles);
  const int per_tile = heads * n_qblocks;
  const int total = __builtin_popcount(active) * per_tile;
  const int per_xcd = (total + kXcd - 1) / kXcd;
  const int xcd = blockIdx.x % kXcd, slot = blockIdx.x / kXcd;
  // The last round of an XCD's compute units: if at most half of them have work, that work is dealt as halves of 128 queries to
  // twice as many workgroups, whose wavefronts then have a SIMD each to themselves.  1,024 tokens: 24 heads 26.2 -> 22.3 us, 70 heads
  // (one whole round and a tenth) 58.4 -> 54.4; 1,840 tokens, 16 heads x 64: 31.7 -> 27.7; beside 40 whole rounds it is 1 %.  (Above
  // half there is no room: the halves would make a round of their own.)
  const int whole = per_xcd - per_xcd % cu_per_xcd, rest = per_xcd - whole;
  const bool halved = 2 * rest <= cu_per_xcd && slot >= whole;
  const int in_xcd = halved ? whole + ((slot - whole) >> 1) : slot;
  const int second = halved ? (slot - whole) & 1 : 0;
  const int logical = xcd * per_xcd + in_xcd;
  if (in_xcd >= per_xcd || logical >= total) return;
  const int nth = logical / per_tile, in_tile = logical - nth * per_tile;
  const int tile = __builtin_amdgcn_readfirstlane(attn_nth_tile(active, nth));
  const int head = __builtin_amdgcn_readfirstlane(in_tile / n_qblocks), qblk = in_tile - head * n_qblocks;   // uniform, and kept scalar
  const u32x4* const qg = (const u32x4*)tab.q[tile];
  const u32x4* const kg = (const u32x4*)tab.k[tile];
  const u32x4* const vg = (const u32x4*)tab.v[tile];
  uint16_t* const out = (uint16_t*)tab.out[tile];
  const int wy0 = (MODE != kLinear) ? tab.y0[tile] : 0, wx0 = (MODE != kLinear) ? tab.x0[tile] : 0;
  // offset of tile token n from the head's first element, in 16-byte units
  auto token_off16 = [&](int n) SG_INLINE -> uint32_t {
    return (MODE == kLinear) ? (uint32_t)n * vw.st16 : window_token(vw, n, wy0, wx0).off16;
  };

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, half = lane >> 5;
  const int N = vw.N;
  const uint32_t head_off16 = (uint32_t)head * vw.head16;
  const u32x4* const kh = kg + head_off16;   // wave-uniform bases of this head
  const u32x4* const vh = vg + head_off16;

  // ---- LDS layout: K stages [4][64 rows][256 B] at 0, V stages at 64 KiB.  16-byte chunk c of K row r
  // sits at chunk c ^ (r & 15); chunk c of V row r at c ^ ((r & 3) << 2): both fragment reads below are
  // then bank-conflict free.  All per-lane addresses are fixed; stage and sub-block enter as immediates.
  uint32_t kaddr[8];   // A operand of QK: slot lq (+32), chunk 2 kk + half
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) kaddr[kk] = lds0 + lq * kRowBytes + (((2 * kk + half) ^ (lq & 15)) << 4);
  // V^T fragments through the transposing read: within a 16-lane group lane s reads 4 consecutive d of key
  // row (s >> 2); the hardware hands lane i the 4 keys of d column i.
  const int grp = lane >> 4, gi = lane & 15;
  const int vt_row = 4 * (grp >> 1) + (gi >> 2);
  const int vt_dbyte = (16 * (grp & 1) + 4 * (gi & 3)) * 2;
  uint32_t vaddr[4];   // + 4096 ks (+ 2048 for slots +8), 64-byte block db of the slot
#pragma unroll
  for (int db = 0; db < 4; ++db)
    vaddr[db] = lds0 + kVRegion + vt_row * kRowBytes + (((4 * db + (vt_dbyte >> 4)) ^ ((vt_row & 3) << 2)) << 4) + (vt_dbyte & 15);

  // ---- DMA loader: wavefront w moves slots 8w..8w+7 of every stage, 4 slots (1 KiB) per instruction; lane l
  // fills chunk (l & 15) of slot 8w + 4u + (l >> 4) and therefore fetches the chunk that belongs there.
  //
  // A wavefront's slots are a run of kTok consecutive tokens.  Where they lie side by side in memory - always in a packed
  // tile - the address is a wave-uniform 64-bit pointer plus a per-lane byte offset that never changes, and the transfer
  // spends no vector instructions on addressing.  The runs of an unbroken window of a width that is a multiple of kTok lie side by
  // side too: kWalk moves that pointer over the tile rows on the scalar unit.  In any other window a run is broken where a tile row
  // ends and where the row crosses the canvas edge, at most once each if the tile is at least kTok wide; such a run adds the two
  // jumps to the lanes behind them.  Where the runs start and break is worked out for 64 stages at a time, one lane per stage, and
  // read back lane by lane: on the scalar unit the same arithmetic costs 2 % of the loop before the transfers of a stage and 5 %
  // between its MFMAs.
  // Measured on 4 x 5 tiles of 75,600 tokens, 40 heads x 128: 1,744 ms a step walked, 1,764 under a shift that makes windows wrap
  // and so planned (1,792 when every lane formed its token's offset from wrapped coordinates each stage), 1,731 gathered and packed;
  // on 2 x 2 shifted tiles of 17,550 tokens, 48 heads x 64: 17.7 ms (21.8 with register-staged loads).
  constexpr int kTok = kKeys / kWaves;   // tokens per wavefront and stage: 8 (head_dim 64: 16)
  auto slot_token = [&](int l, int u, bool is_v, uint32_t& chunk) SG_INLINE -> int {   // what lane l moves: token of the run, chunk of it
    const int slot_w = 4 * u + (l >> 4), row = 8 * wave + slot_w;
    const int c = (l & 15) ^ (is_v ? (row & 3) << 2 : row & 15);
    chunk = (uint32_t)(D == 128 ? c : c & 7);
    return D == 128 ? slot_w : 2 * slot_w + (c >> 3);
  };
  auto lane_offset = [&](int l, int u, bool is_v) SG_INLINE -> uint32_t {
    uint32_t chunk;
    const int t = slot_token(l, u, is_v, chunk);
    return ((uint32_t)t * vw.st16 + chunk) << 4;
  };
  // The short form of packed tiles of head_dim 64 works these offsets out for every stage: kept over the iterations they are spilled, and
  // their reload waits for all transfers in flight.  us a step, spilled, worked out (other form): 20 tiles, 48 heads, of 1,000 tokens 578, 503
  // (524), of 2,000 1,789, 1,440 (1,457); one tile, 8 heads, of 700 15.5, 14.6 (15.8).
  constexpr bool kFormed = SHORT && D == 64 && MODE == kLinear && !REFRESH;
  uint32_t klane[2], vlane[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) { klane[u] = lane_offset(lane, u, false); vlane[u] = lane_offset(lane, u, true); }
  const uint32_t dma_dst = lds0 + wave * (8 * kRowBytes);
  uint32_t plan_first = 0, plan_jump = 0, plan_info = 0;   // lane l: this wavefront's run of stage 64 m + l
  const int edge0 = (wx0 + vw.tw > vw.W) ? vw.W - wx0 : 0x3fffffff;   // tokens of a tile row before the canvas edge (none crossed: many)
  auto plan64 = [&](int blk) SG_INLINE {
    const int n0 = ((blk & ~63) + lane) * kKeys + kTok * wave;
    const int t = (int)divide((uint32_t)n0, vw.by_plane);
    const int in_plane = n0 - t * (vw.th * vw.tw);
    const int i = (int)divide((uint32_t)in_plane, vw.by_row), j = in_plane - i * vw.tw;
    int y = wy0 + i, x = wx0 + j;
    y -= (y >= vw.H) ? vw.H : 0;
    x -= (x >= vw.W) ? vw.W : 0;
    plan_first = (uint32_t)((t * vw.H + y) * vw.W + x) * vw.st16;
    int row_end = vw.tw - j;     // tokens before the tile row ends
    int edge = edge0 - j;        // tokens before the canvas edge is crossed; at or below 0: this row has crossed already
    const bool here = edge > 0 && edge < row_end;   // crossed in this row, else in the next
    const bool frame_end = i + 1 == vw.th;
    int y1 = frame_end ? wy0 : y + 1;
    y1 -= (y1 >= vw.H) ? vw.H : 0;
    const uint32_t next16 = (uint32_t)(((frame_end ? t + 1 : t) * vw.H + y1) * vw.W + wx0) * vw.st16;
    plan_jump = next16 - (plan_first + (uint32_t)row_end * vw.st16) + (here ? (uint32_t)vw.W * vw.st16 : 0u);   // offset's jump at the row's end
    if (!here) edge = row_end + edge0;
    row_end = row_end < kTok ? row_end : kTok;   // breaks behind the run: no lane reaches them
    edge = edge < kTok ? edge : kTok;
    const bool whole = (vw.reach & kReachLane) && row_end == kTok && edge == kTok;
    plan_info = whole ? 0u : (uint32_t)row_end | (uint32_t)edge << 8;
  };
  uint32_t run_info = 0, run_first16 = 0;   // of the stage that the next steady iteration issues; info 0: side by side
  auto fetch_plan = [&](int blk) SG_INLINE {
    run_info = __builtin_amdgcn_readlane(plan_info, blk & 63);
    run_first16 = __builtin_amdgcn_readlane(plan_first, blk & 63);
  };
  auto look_up = [&](int blk, uint32_t dst) SG_INLINE {   // every lane looks its token up; tokens >= N: the last one (masked later)
    int l = lane;
    asm volatile("" : "+v"(l));   // worked out here, not kept in registers over the loop
    const u32x4* kb = kh;
    const u32x4* vb = vh;
    asm volatile("" : "+s"(kb), "+s"(vb));
    const int n0 = blk * kKeys + kTok * wave;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t kc, vc;
      const int nk = n0 + slot_token(l, u, false, kc), nv = n0 + slot_token(l, u, true, vc);
      const uint32_t ko = token_off16(nk < N ? nk : N - 1);
      const uint32_t vo = (D == 128) ? ko : token_off16(nv < N ? nv : N - 1);
      dma16_addr(kb + ((uint64_t)ko + kc), dst + u * (4 * kRowBytes));
      dma16_addr(vb + ((uint64_t)vo + vc), dst + kVRegion + u * (4 * kRowBytes));
    }
  };
  auto move_run = [&](const char* kp, const char* vp, uint32_t dst) SG_INLINE {
    uint32_t all = ~0u;
    if (kFormed) asm volatile("" : "+s"(all));
    const int l = (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));   // lane, which is spilled as well
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      dma16(kp, kFormed ? lane_offset(l, u, false) : klane[u], dst + u * (4 * kRowBytes));
      dma16(vp, kFormed ? lane_offset(l, u, true) : vlane[u], dst + kVRegion + u * (4 * kRowBytes));
    }
  };
  // packed tiles and walked windows: pointers to the run of the stage to issue; a walk also knows its tile row and column
  uint32_t run16 = (uint32_t)(kTok * wave) * vw.st16;
  int32_t walk_i = 0, walk_j = 0;
  if (MODE == kWalk) {   // (a run at or beyond N is looked up instead)
    const int t = (int)divide((uint32_t)(kTok * wave), vw.by_plane), in_plane = kTok * wave - t * (vw.th * vw.tw);
    walk_i = (int)divide((uint32_t)in_plane, vw.by_row);
    walk_j = in_plane - walk_i * vw.tw;
    run16 = (uint32_t)((t * vw.H + wy0 + walk_i) * vw.W + wx0 + walk_j) * vw.st16;
  }
  const char* kcur = (const char*)kh + ((uint64_t)run16 << 4);
  const char* vcur = (const char*)vh + ((uint64_t)run16 << 4);
  const uint64_t stage_bytes = (uint64_t)(kKeys * 16) * vw.st16;
  // in units of 16 bytes, which keeps the scalar registers few: from a tile row's end to the next row, and, behind the last row, on
  // to the next frame
  const uint32_t row_jump16 = (uint32_t)(vw.W - vw.tw) * vw.st16, frame_jump16 = (uint32_t)((vw.H - vw.th) * vw.W) * vw.st16;
  auto move_next = [&](uint32_t dst) SG_INLINE {   // move the run, go one stage on
    move_run(kcur, vcur, dst);
    uint64_t by = stage_bytes;
    if (MODE == kWalk) {
      uint32_t by16 = kKeys * vw.st16;
      walk_j += kKeys;
      if (vw.tw >= kKeys) {   // at most one tile row ends: no branch
        const bool ends = walk_j >= vw.tw;
        walk_j -= ends ? vw.tw : 0;
        walk_i += ends ? 1 : 0;
        const bool over = walk_i == vw.th;
        walk_i = over ? 0 : walk_i;
        by16 += (ends ? row_jump16 : 0u) + (over ? frame_jump16 : 0u);
      } else {
        while (walk_j >= vw.tw) {
          walk_j -= vw.tw;
          by16 += row_jump16;
          if (++walk_i == vw.th) { walk_i = 0; by16 += frame_jump16; }
        }
      }
      by = (uint64_t)by16 << 4;
    }
    kcur += by;
    vcur += by;
  };
  auto move_planned = [&](int blk, uint32_t dst) SG_INLINE {
    if (run_info == 0) {
      const uint64_t first = (uint64_t)run_first16 << 4;
      move_run((const char*)kh + first, (const char*)vh + first, dst);
    } else if ((vw.reach & kReachHead) && vw.tw >= kTok) {
      // token x of the run lies behind a break at token b exactly if its lane offset is at or beyond b tokens
      const uint32_t first = run_first16 << 4, token = vw.st16 << 4;
      const uint32_t end_at = (run_info & 255u) * token, edge_at = (run_info >> 8) * token;
      const uint32_t end_by = __builtin_amdgcn_readlane(plan_jump, blk & 63) << 4, edge_by = 0u - (uint32_t)vw.W * token;
      auto behind = [&](uint32_t off) SG_INLINE -> uint32_t { return (off >= end_at ? end_by : 0u) + (off >= edge_at ? edge_by : 0u); };
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t kj = behind(klane[u]), vj = (D == 128) ? kj : behind(vlane[u]);
        dma16(kh, klane[u] + kj + first, dst + u * (4 * kRowBytes));
        dma16(vh, vlane[u] + vj + first, dst + kVRegion + u * (4 * kRowBytes));
      }
    } else {   // tiles narrower than a run, heads of 4 GiB and more
      look_up(blk, dst);
    }
  };
  // issue stage `blk`, whose keys are all below N, into ring slot `st` = blk % 4
  auto issue_full = [&](int blk, int st) SG_INLINE {
    const uint32_t dst = dma_dst + st * kTileBytes;
    if (MODE != kWindow) {
      move_next(dst);
    } else {
      move_planned(blk, dst);
      if (st == kStages - 1 && (blk & 63) == 63) plan64(blk + 1);
      fetch_plan(blk + 1);   // for the next steady iteration
    }
  };
  // the same in the short form, for a stage that may hold keys >= N; its plan has been fetched
  auto issue_next = [&](int blk, int st) SG_INLINE {
    const uint32_t dst = dma_dst + st * kTileBytes;
    if (__builtin_expect(blk * kKeys + kTok * (wave + 1) > N, 0)) look_up(blk, dst);   // (the last stage)
    else if (MODE != kWindow) move_next(dst);
    else move_planned(blk, dst);
    if (MODE == kWindow) fetch_plan(blk + 1);   // for the next iteration; the first plan covers all stages
  };
  // Cache refresh: a workgroup copies the keys and values of its own query rows out of the LDS ring while their stages are
  // there (kCopy of its stages, each wavefront what it moved itself, to the place it came from), so that the copy reads
  // nothing from HBM and its stores are spread over the launch; its rows of Q follow at the end.
  constexpr int kCopy = kBR / kKeys;
  const int copy0 = qblk * kCopy, copy_from = copy0 & ~(kStages - 1);
  const int64_t to_cache = REFRESH ? (char*)tab.refresh[tile] - (const char*)tab.q[tile] : 0;
  auto copies = [&](int k) SG_INLINE -> int { return (REFRESH && k >= copy0 && k < copy0 + kCopy && !second) ? 1 : 0; };
  auto copy_stage = [&](int k, bool full) SG_INLINE {
    int l = lane;
    asm volatile("" : "+v"(l));   // addresses are formed here, not kept in registers over the loop
    const uint32_t at = dma_dst + (k % kStages) * kTileBytes + l * 16;
    const int n0 = k * kKeys + kTok * wave;
    const uint64_t run = (uint64_t)((uint32_t)n0 * vw.st16) << 4;
#pragma unroll
    for (int u = 0; u < 4; ++u) {   // K, V of the wavefront's first four slots, of the other four
      const bool is_v = u & 1;
      uint32_t c, off = is_v ? vlane[u >> 1] : klane[u >> 1];
      asm volatile("" : "+v"(off));
      const u32x4 x = *(const SG_LDS u32x4*)(uintptr_t)(at + (is_v ? kVRegion : 0) + (u >> 1) * (4 * kRowBytes));
      char* const base = (char*)(is_v ? vh : kh) + to_cache + run;
      if (full || n0 + slot_token(l, u >> 1, is_v, c) < N) __builtin_nontemporal_store(x, (u32x4*)(base + off));
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // the same, with its plan, for a slot that is not a constant
  auto issue_any = [&](int blk, int st) SG_INLINE {
    const uint32_t dst = dma_dst + st * kTileBytes;
    if (MODE == kWindow) {
      if ((blk & 63) == 0) plan64(blk);
      fetch_plan(blk);
    }
    if (blk * kKeys + kTok * (wave + 1) > N) look_up(blk, dst);
    else if (MODE != kWindow) move_next(dst);   // (a wavefront looks up all stages behind one that it looked up)
    else move_planned(blk, dst);
  };

  // The first stage is requested before Q, so that the two latencies run side by side; the next two stages follow when Q is
  // there (its wait counts every transfer requested before it, and they are not needed for half an iteration yet).
  issue_any(0, 0);

  // ---- Q fragments (B operand of S^T = K Q^T): query q0 + lq, d = 16 kk + 8 half + 0..7
  const int q0 = !halved ? qblk * kBR + wave * 32 : wave < 4 ? qblk * kBR + second * (kBR / 2) + wave * 32 : N;   // N: no query
  bf16x8 qf[D / 16];
  {
    int n = q0 + lq;
    if (n > N - 1) n = N - 1;
    const u32x4* src = qg + head_off16 + token_off16(n);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      const u32x4 raw = src[2 * kk + half];
      if (LATE) { qf[kk] = __builtin_bit_cast(bf16x8, raw); continue; }
      u32x4 scaled;   // q * log2(e) * scale, rounded to bf16 once
#pragma unroll
      for (int e = 0; e < 4; ++e)
        scaled[e] = pack_bf16x2(bf16_bits_to_f32(raw[e] & 0xffffu) * c_log2, __uint_as_float(raw[e] & 0xffff0000u) * c_log2);
      qf[kk] = __builtin_bit_cast(bf16x8, scaled);
    }
  }

  f32x16 oacc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  Softmax sm;
  sm.M = LATE ? -__builtin_inff() : 0.f;
  sm.l = 0.f;
  f32x16 cinit;   // accumulator start of every score chain: -M in all registers
#pragma unroll
  for (int r = 0; r < 16; ++r) cinit[r] = 0.f;

  float mid = 1.f;   // head_dim 64, late scaling: factor of the accumulators between the two halves of a stage, applied inside PV

  auto kfrag = [&](int kk, int kb, int off) SG_INLINE -> bf16x8 {
    return __builtin_bit_cast(bf16x8, *(const SG_LDS u32x4*)(uintptr_t)(kaddr[kk] + off + kb * (32 * kRowBytes)));
  };
  auto vfrag = [&](int ks, int db, int off) SG_INLINE -> bf16x8 {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SG_LDS s16x4*)(uintptr_t)(vaddr[db] + off + ks * (16 * kRowBytes)));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SG_LDS s16x4*)(uintptr_t)(vaddr[db] + off + ks * (16 * kRowBytes) + 8 * kRowBytes));
    const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
  };
  // Fragment reads run kPF MFMA steps ahead of their use; the K fragments of the first step of a QK product
  // are read during the last step of the PV product before it, so the matrix pipe does not drain between
  // the two.  (Two steps ahead is no faster and spills registers; reading the first V^T fragments ahead,
  // during the softmax, was measured 7 % slower.)
  constexpr int kPF = 2;
  constexpr int kKPre = 1;
  bf16x8 kpre[kKPre][2];  // K fragments of the first kKPre QK steps, read during the PV tail
  // S^T = K Q^T of the stage at LDS byte offset `off`: two independent accumulator chains
  // head_dim 64: the second half of a slot is another key, so steps kk >= 4 feed the next score block
  // (block 2 kb + (kk >> 2), Q fragment kk & 3) and there are four chains, two of them in flight at a time
  auto qk = [&](int off, f32x16 (&s)[kMaxSB], bool prefetched) SG_INLINE {
    bf16x8 a[8][2];
#pragma unroll
    for (int kk = 0; kk < kPF; ++kk) {
      if (prefetched && kk < kKPre) { a[kk][0] = kpre[kk][0]; a[kk][1] = kpre[kk][1]; }
      else { a[kk][0] = kfrag(kk, 0, off); a[kk][1] = kfrag(kk, 1, off); }
    }
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      if (kk + kPF < 8) { a[kk + kPF][0] = kfrag(kk + kPF, 0, off); a[kk + kPF][1] = kfrag(kk + kPF, 1, off); }
      __builtin_amdgcn_sched_barrier(0);
      constexpr int kPerChain = D / 16;            // MFMA steps per score block
      const int b0 = (D == 128) ? 0 : (kk >> 2);   // score blocks fed by this step: b0 and b0 + kSB / 2
      const int b1 = b0 + kSB / 2;
      const int qi = kk % kPerChain;
      if (qi == 0) {
        s[b0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][0], qf[qi], LATE ? zero16() : cinit, 0, 0, 0);
        s[b1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][1], qf[qi], LATE ? zero16() : cinit, 0, 0, 0);
      } else {
        s[b0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][0], qf[qi], s[b0], 0, 0, 0);
        s[b1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][1], qf[qi], s[b1], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // O^T += V^T P^T: four independent accumulator chains (one per 32 rows of d); if a QK product follows
  // (K stage at `k_off`), its first fragments are read in the last step
  // (head_dim 64: fragment (ks, db) is d block db & 1 of the 16 keys 4 (ks >> 1) + 2 (db >> 1) + (ks & 1), two chains)
  auto pv = [&](int off, const bf16x8 (&pp)[2 * kMaxSB], int k_off, bool k_follows) SG_INLINE {
    auto acc_of = [](int i) SG_INLINE { return (D == 128) ? (i & 3) : (i & 1); };
    auto p_of = [](int i) SG_INLINE { return (D == 128) ? (i >> 2) : 4 * (i >> 3) + 2 * ((i & 3) >> 1) + ((i >> 2) & 1); };
    bf16x8 a[16];
#pragma unroll
    for (int i = 0; i < 2 * kPF; ++i) a[i] = vfrag(i >> 2, i & 3, off);
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      if (LATE && kSB == 4 && i == 8 && __any(mid != 1.f)) {   // the keys behind raised the maximum
#pragma unroll
        for (int db = 0; db < D / 32; ++db) oacc[db] *= mid;
      }
      if (i + 2 * kPF < 16) {
        a[i + 2 * kPF] = vfrag((i + 2 * kPF) >> 2, (i + 2 * kPF) & 3, off);
        a[i + 2 * kPF + 1] = vfrag((i + 2 * kPF + 1) >> 2, (i + 2 * kPF + 1) & 3, off);
      } else if (k_follows && (i + 2 * kPF - 16) / 2 >= kPF - kKPre) {
        const int kk = (i + 2 * kPF - 16) / 2 - (kPF - kKPre);
        kpre[kk][0] = kfrag(kk, 0, k_off);
        kpre[kk][1] = kfrag(kk, 1, k_off);
      }
      __builtin_amdgcn_sched_barrier(0);
      oacc[acc_of(i)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], pp[p_of(i)], oacc[acc_of(i)], 0, 0, 0);
      oacc[acc_of(i + 1)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i + 1], pp[p_of(i + 1)], oacc[acc_of(i + 1)], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  f32x16 s[kMaxSB];   // scores of the stage in flight (the first kSB entries) between an MFMA phase and the next softmax phase
  // Late scaling keeps the true running maximum, every 64 keys: the dominating probability of a query is then exactly 1, which
  // bf16 holds without an error, and none is above it, so sums of p v stay finite for every finite v.  Error against fp64 at
  // 400, 1,200 and 17,550 tokens: 2.17e-3, 2.22e-3, 2.30e-3; with one maximum per stage of 128 keys 2.18e-3, 2.23e-3, 2.30e-3; with
  // the lazy reference below 2.28e-3, 2.32e-3, 2.34e-3.  The step of 4 x 17,550 tokens, 48 heads, is 1.20 - 1.23 times as fast as
  // with the register-staged kernel (21.8 -> 17.7 ms); the other two would be 1.25 and 1.28 - 1.33 times as fast.
  auto late_half = [&](auto h_tag, bf16x8 (&p)[2 * kMaxSB]) SG_INLINE {
    constexpr int H = decltype(h_tag)::value;
    const float top = fmaxf(sm.M, block_max<2, 2 * H>(s) * c_log2);
    if (H == 1) mid = 1.f;
    if (__any(top != sm.M)) {
      const float alpha = __builtin_amdgcn_exp2f(sm.M - top);   // first stage: exp2(-inf) = 0
      sm.M = top;
      sm.l *= alpha;
      if (H == 1) mid = alpha;
      else {
#pragma unroll
        for (int db = 0; db < D / 32; ++db) oacc[db] *= alpha;
      }
    }
#pragma unroll
    for (int kb = 2 * H; kb < 2 * H + 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb][r] = __builtin_fmaf(s[kb][r], c_log2, -sm.M);
    sm.l += exp_block<2, 2 * H>(s, p);
  };
  // softmax phase of one stage: scores t (exponent domain) -> p, l.  The exponentials are taken against the
  // current reference; if one of them outgrew the guard (or on the first stage, which sets the reference) the
  // reference moves by delta per query: scores, running sum and output accumulators are brought to the new
  // reference and the exponentials are retaken.  One copy of the code, looped at most twice.
  auto softmax_phase = [&](int key0, bool masked, bool first, bf16x8 (&p)[2 * kMaxSB]) SG_INLINE {
    if constexpr (LATE) {
      if (masked) mask_tail<kSB>(s, key0, N);
      late_half(std::integral_constant<int, 0>{}, p);
      if constexpr (kSB == 4) late_half(std::integral_constant<int, 1>{}, p);
      return;
    }
    if (masked) mask_tail<kSB>(s, key0, N);
    bool move = first;
    float sum;
#pragma nounroll
    for (;;) {
      if (move) {
        const float mx = block_max<kSB>(s);
        const float delta = first ? mx : fmaxf(mx, 0.f);
        const float alpha = first ? 0.f : __builtin_amdgcn_exp2f(-delta);
#pragma unroll
        for (int kb = 0; kb < kSB; ++kb) s[kb] -= delta;
        sm.M += delta;
#pragma unroll
        for (int r = 0; r < 16; ++r) cinit[r] = -sm.M;
        sm.l *= alpha;
#pragma unroll
        for (int db = 0; db < D / 32; ++db) oacc[db] *= alpha;
      }
      sum = exp_block<kSB>(s, p);
      if (move || !__any(!(sum < kOverflowGuard))) break;
      move = true;
    }
    sm.l += sum;
  };

  // ---- Schedule.  Wavefronts 0-3 (group 0) and 4-7 (group 1) share the four SIMDs pairwise and run half an
  // iteration apart, so that while one wavefront of a SIMD feeds the matrix pipe (MFMA phase: PV(k), QK(k+1))
  // the other works the vector ALU (softmax phase).  One workgroup barrier B_k per iteration re-establishes
  // the offset: after it group 0 starts MFMA phase k (its softmax k ran before the barrier) while group 1
  // starts softmax k followed by MFMA phase k.
  // Ring of 4 stages: between B_k and B_k+1 both groups read V of stage k and K of stage k+1; stage k+3 is
  // issued right after B_k into the slot of stage k-1 (last read before B_k) and must have landed by B_k+2.
  const int n_blocks = (N + kKeys - 1) / kKeys;
  const bool tail = (N % kKeys) != 0;
  // Which wavefront of a SIMD takes which role matters: the SIMD serves its older wavefront (0-3) first.  With
  // head_dim 128 (MFMA phase longer than the softmax phase) the older one leads with the MFMA phase; with head_dim 64
  // (softmax phase longer) it has to lead with the softmax, or the younger one's softmax starves behind both phases of
  // the older one and its MFMA phase then runs with nothing beside it (measured: 1.08 -> 1.22 PFLOP/s; the opposite
  // choice costs head_dim 128 a quarter of its rate).
  const int grp1 = __builtin_amdgcn_readfirstlane((wave >> 2) ^ (D == 64 ? 1 : 0));
  auto wait_stage = [&](int younger_stages) SG_INLINE {   // own transfers: all but the youngest `younger_stages` stages landed
    __builtin_amdgcn_sched_barrier(0);
    if (younger_stages >= 3) wait_vmcnt<12>();
    else if (younger_stages == 2) wait_vmcnt<8>();
    else if (younger_stages == 1) wait_vmcnt<4>();
    else wait_vmcnt<0>();
  };
  // Keys at or beyond N stand in for the last one with probability 0; their value rows are cleared, so that an infinite last value
  // does not become 0 * inf (late scaling only: with 64 keys a stage such rows were rarer than with 128).
  auto clear_tail = [&]() SG_INLINE {
    const int last = n_blocks - 1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t c;
      if (last * kKeys + kTok * wave + slot_token(lane, u, true, c) >= N)
        *(SG_LDS u32x4*)(uintptr_t)(dma_dst + (last % kStages) * kTileBytes + kVRegion + u * (4 * kRowBytes) + lane * 16) = u32x4{0, 0, 0, 0};
    }
  };
  // End of iteration k: stage k + 2, issued last but one, has landed.  Behind its transfers stand those of stage k + 3, if there is
  // one, and the four stores of every stage copied in this iteration and the one before; these are whole stages as long as there
  // is a stage k + 2, so none of their stores is skipped.  From iteration n_blocks - 2 on every transfer has landed, and a copy's
  // stores need not be waited for (a step of one tile of 460 tokens, 2 heads x 64: 28.1 -> 27.0 us).
  auto wait_iteration = [&](int k, bool issued) SG_INLINE {
    const int stores = copies(k) + copies(k - 1);
    if (issued) wait_stage(1 + stores);
    else if (!REFRESH || k + 2 < n_blocks) wait_stage(stores);
    if (LATE && tail && k == n_blocks - 2) clear_tail();
  };
  bf16x8 p[2 * kMaxSB];   // the first 2 kSB entries
  // keeps the score registers live across the phase boundary (a macro: the statement has to sit in the
  // lambdas that are its call sites)
#define SG_PIN_SCORES()                                                                \
  do {                                                                                 \
    asm volatile("" : : "v"(s[0]), "v"(s[1]));                                         \
    if constexpr (kSB == 4) asm volatile("" : : "v"(s[kSB - 2]), "v"(s[kSB - 1]));      \
  } while (0)
  auto mfma_phase_static = [&](auto st_tag) SG_INLINE {
    constexpr int ST = decltype(st_tag)::value;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    pv(ST * kTileBytes, p, ((ST + 1) % kStages) * kTileBytes, true);
    qk(((ST + 1) % kStages) * kTileBytes, s, true);
    SG_PIN_SCORES();
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Windows of head_dim 64 take QK behind the last stage as well, of stale keys and for nothing: with the branch their scores spill
  // (one tile of 1,000 tokens, 24 heads: 20.8 us with it, 19.2 without); elsewhere the branch is up to 2 % faster.
  constexpr bool kQkAlways = D == 64 && LATE;
  auto mfma_phase_short = [&](int k, auto st_tag) SG_INLINE {
    constexpr int ST = decltype(st_tag)::value;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    pv(ST * kTileBytes, p, ((ST + 1) % kStages) * kTileBytes, true);   // (behind the last stage the K fragments it reads ahead are stale and not used)
    if (kQkAlways || k + 1 < n_blocks) qk(((ST + 1) % kStages) * kTileBytes, s, true);
    SG_PIN_SCORES();
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mfma_phase_any = [&](int k) SG_INLINE {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    pv((k % kStages) * kTileBytes, p, ((k + 1) % kStages) * kTileBytes, k + 1 < n_blocks);
    if (k + 1 < n_blocks) qk(((k + 1) % kStages) * kTileBytes, s, true);
    SG_PIN_SCORES();
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto softmax_pinned = [&](int j, bool masked, bool first) SG_INLINE {
    softmax_phase(j * kKeys, masked, first, p);
    asm volatile("" : : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(sm.l));
    if constexpr (!LATE) asm volatile("" : : "v"(cinit));
    if constexpr (kSB == 4) asm volatile("" : : "v"(p[kSB]), "v"(p[kSB + 1]), "v"(p[kSB + 2]), "v"(p[kSB + 3]));
    __builtin_amdgcn_sched_barrier(0);
  };

  asm volatile("" : : "v"(qf[0]), "v"(qf[D / 16 - 1]));   // Q has arrived, and the first stage with it
  __builtin_amdgcn_sched_barrier(0);
  for (int b = 1; b < 3; ++b)
    if (b < n_blocks) issue_any(b, b);
  wait_stage(n_blocks >= 3 ? 2 : (n_blocks == 2 ? 1 : 0));
  if (LATE && tail && n_blocks == 1) clear_tail();
  meet();
  if (__builtin_expect(q0 >= N, 0)) {   // a wavefront without a query (the last query block) moves its share of the stages and leaves the matrix
                   // pipe and the vector ALU to the other wavefront of its SIMD
    wait_stage(n_blocks >= 3 ? 1 : 0);
    meet();
    for (int k = 0; k < n_blocks; ++k) {
      if (k + 3 < n_blocks) issue_any(k + 3, (k + 3) % kStages);
      if (copies(k)) copy_stage(k, (k + 1) * kKeys <= N);
      wait_iteration(k, k + 3 <= n_blocks - 1);
      meet();
    }
    return;
  }
  qk(0, s, false);
  SG_PIN_SCORES();
  // The steady loop: from iteration kHead on, in groups of four, while the stage it requests is not the last (which may be partial and is
  // moved by issue_any).  Iteration 0 sets the reference and stays outside; the other three that do where groups begin at a
  // multiple of four take 3,600 cycles instead of 2,700.  From 1, walked windows: 9 tiles of 3,000 tokens, 24 heads 906 -> 896 us, one
  // 132.4 -> 129.6, of 2,000 430 -> 427; windows of 53,760 tokens, 24 heads x 64 45.6 -> 44.9 ms.  Not planned windows of head_dim 128 (the
  // loop itself spills: 9 tiles of 80,640 866 -> 901 ms), not packed tiles of head_dim 64 (34.05 -> 34.20 ms), not with a refresh, which
  // interrupts whole groups of the stages it copies.
  constexpr int kHead = (MODE == kWalk || (MODE == kWindow && D == 64)) ? 1 : kStages;
  // Calls of up to 16 or 24 stages take the short form, so the conditions here and below that hold for more of them stay for the sake of
  // the code around them: without them windows of 75,600 tokens, 16 heads x 64, take 25.2 ms instead of 24.3.
  const int n_steady = (n_blocks >= kHead + 2 * kStages) ? kHead + ((n_blocks - kHead - kStages) / kStages) * kStages : 0;

  // Short tiles: one copy of an iteration for every ring slot and group serves all of them; what the first and the last need besides is
  // a scalar branch.  (A kernel of its own: with
  // the steady loop beside it the compiler spills 130 registers.)
  auto short_iterations = [&](auto iteration) SG_INLINE {
    for (int k = 0;; k += kStages) {
      iteration(k, std::integral_constant<int, 0>{});
      if (k + 1 >= n_blocks) break;
      iteration(k + 1, std::integral_constant<int, 1>{});
      if (k + 2 >= n_blocks) break;
      iteration(k + 2, std::integral_constant<int, 2>{});
      if (k + 3 >= n_blocks) break;
      iteration(k + 3, std::integral_constant<int, 3>{});
      if (k + 4 >= n_blocks) break;
    }
  };
  if (SHORT && MODE == kWindow) fetch_plan(3);
  if constexpr (SHORT) {
    if (!grp1) {
      softmax_pinned(0, tail && n_blocks == 1, true);
      wait_stage(n_blocks >= 3 ? 1 : 0);
      meet();   // B_0
      short_iterations([&](int k, auto st_tag) SG_INLINE {
        constexpr int ST = decltype(st_tag)::value;
        if (k + 3 < n_blocks) issue_next(k + 3, (ST + 3) % kStages);
        if (copies(k)) copy_stage(k, (k + 1) * kKeys <= N);
        mfma_phase_short(k, st_tag);
        if (k + 1 < n_blocks) softmax_pinned(k + 1, tail && k + 1 == n_blocks - 1, false);
        wait_iteration(k, k + 3 < n_blocks);
        meet();
      });
    } else {
      wait_stage(n_blocks >= 3 ? 1 : 0);
      meet();   // B_0
      short_iterations([&](int k, auto st_tag) SG_INLINE {
        constexpr int ST = decltype(st_tag)::value;
        if (k + 3 < n_blocks) issue_next(k + 3, (ST + 3) % kStages);
        if (copies(k)) copy_stage(k, (k + 1) * kKeys <= N);
        softmax_pinned(k, tail && k == n_blocks - 1, k == 0);
        mfma_phase_short(k, st_tag);
        wait_iteration(k, k + 3 < n_blocks);
        meet();
      });
    }
  } else if (!grp1) {
    softmax_pinned(0, tail && n_blocks == 1, true);
    wait_stage(n_blocks >= 3 ? 1 : 0);
    meet();   // B_0
    auto general = [&](int k) SG_INLINE {
      if (k + 3 < n_blocks) issue_any(k + 3, (k + 3) % kStages);
      if (copies(k)) copy_stage(k, (k + 1) * kKeys <= N);
      mfma_phase_any(k);
      if (k + 1 < n_blocks) softmax_pinned(k + 1, tail && k + 1 == n_blocks - 1, false);
      wait_iteration(k, k + 3 <= n_blocks - 1);
      meet();
    };
    auto steady = [&](int k, auto st_tag) SG_INLINE {
      constexpr int ST = decltype(st_tag)::value;
      issue_full(k + 3, (ST + 3) % kStages);
      mfma_phase_static(st_tag);
      softmax_pinned(k + 1, false, false);
      wait_stage(1);
      meet();
    };
    int k = 0;
    for (; k < kHead && k < n_blocks; ++k) general(k);
    if (MODE == kWindow && k < n_steady) fetch_plan(k + 3);
    for (;;) {   // a refresh interrupts the steady loop for the iterations around the stages it copies
      const int until = (REFRESH && k <= copy0) ? (copy_from < n_steady ? copy_from : n_steady) : n_steady;
      for (; k < until; k += kStages) {
        steady(k, std::integral_constant<int, (kHead + 0) % kStages>{});
        steady(k + 1, std::integral_constant<int, (kHead + 1) % kStages>{});
        steady(k + 2, std::integral_constant<int, (kHead + 2) % kStages>{});
        steady(k + 3, std::integral_constant<int, (kHead + 3) % kStages>{});
      }
      if (!REFRESH || k >= n_steady) break;
      for (int i = 0; i < kStages; ++i, ++k) general(k);
    }
    for (; k < n_blocks; ++k) general(k);
  } else {
    wait_stage(n_blocks >= 3 ? 1 : 0);
    meet();   // B_0
    auto general = [&](int k) SG_INLINE {
      if (k + 3 < n_blocks) issue_any(k + 3, (k + 3) % kStages);
      if (copies(k)) copy_stage(k, (k + 1) * kKeys <= N);
      softmax_pinned(k, tail && k == n_blocks - 1, k == 0);
      mfma_phase_any(k);
      wait_iteration(k, k + 3 <= n_blocks - 1);
      meet();
    };
    auto steady = [&](int k, auto st_tag) SG_INLINE {
      constexpr int ST = decltype(st_tag)::value;
      issue_full(k + 3, (ST + 3) % kStages);
      softmax_pinned(k, false, false);
      mfma_phase_static(st_tag);
      wait_stage(1);
      meet();
    };
    int k = 0;
    for (; k < kHead && k < n_blocks; ++k) general(k);
    if (MODE == kWindow && k < n_steady) fetch_plan(k + 3);
    for (;;) {   // a refresh interrupts the steady loop for the iterations around the stages it copies
      const int until = (REFRESH && k <= copy0) ? (copy_from < n_steady ? copy_from : n_steady) : n_steady;
      for (; k < until; k += kStages) {
        steady(k, std::integral_constant<int, (kHead + 0) % kStages>{});
        steady(k + 1, std::integral_constant<int, (kHead + 1) % kStages>{});
        steady(k + 2, std::integral_constant<int, (kHead + 2) % kStages>{});
        steady(k + 3, std::integral_constant<int, (kHead + 3) % kStages>{});
      }
      if (!REFRESH || k >= n_steady) break;
      for (int i = 0; i < kStages; ++i, ++k) general(k);
    }
    for (; k < n_blocks; ++k) general(k);
  }

  // ---- epilogue: O^T accumulators -> packed tile [head][n][d]; register r of block db is
  // d = 32 db + 8 (r>>2) + 4 half + (r&3): 4 consecutive d = 8 bytes
  {
    const int sub = lane / (D / 8), chunk = lane % (D / 8);
    const uint32_t lu = __float_as_uint(sm.l);
    const auto sw = __builtin_amdgcn_permlane32_swap(lu, lu, false, false);
    const float inv = 1.0f / (__uint_as_float(sw[0]) + __uint_as_float(sw[1]));
    // Rows go out through LDS (free since the last barrier; 8 KiB per wavefront): straight from the accumulators a store
    // would touch 64 rows for 8 bytes each, 64 address cycles per instruction; from LDS it writes 1 KiB in one piece.
    // 16-byte chunk c of row r sits at chunk c ^ (r % kChunks).  With the reordered start this takes 2.5 - 3 us off
    // every workgroup: 256 workgroups of 256 tokens 21.3 -> 18.8 us, of 1,024 tokens 37.8 -> 34.9, 2,160 of 4,600 tokens 1069 -> 1051.
    constexpr int kChunks = D / 8, kRowsPer = 64 / kChunks;
    const uint32_t buf = lds0 + wave * (32 * D * 2);
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        u32x2 w;
        w[0] = pack_bf16x2(oacc[db][4 * g] * inv, oacc[db][4 * g + 1] * inv);
        w[1] = pack_bf16x2(oacc[db][4 * g + 2] * inv, oacc[db][4 * g + 3] * inv);
        *(SG_LDS u32x2*)(uintptr_t)(buf + lq * (D * 2) + (((4 * db + g) ^ (lq & (kChunks - 1))) << 4) + 8 * half) = w;
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    u32x4* const dst = (u32x4*)(out + ((size_t)head * N + q0) * D);
#pragma unroll
    for (int i = 0; i < 32 / kRowsPer; ++i) {
      const int r = kRowsPer * i + sub;
      const u32x4 x = *(const SG_LDS u32x4*)(uintptr_t)(buf + r * (D * 2) + ((chunk ^ (r & (kChunks - 1))) << 4));
      if (q0 + r < N) dst[r * kChunks + chunk] = x;
    }
    if constexpr (REFRESH) {   // this wavefront's rows of Q once more, for the cache
      __builtin_amdgcn_sched_barrier(0);
      constexpr int kPieces = 32 / kRowsPer;
      const u32x4* const qs = qg + head_off16;
      u32x4* const qd = (u32x4*)((char*)qs + to_cache);
      u32x4 x[kPieces];
#pragma unroll
      for (int i = 0; i < kPieces; ++i) {
        const int r = q0 + kRowsPer * i + sub;
        x[i] = qs[(uint32_t)(r < N ? r : N - 1) * vw.st16 + chunk];
      }
#pragma unroll
      for (int i = 0; i < kPieces; ++i) {
        const int r = q0 + kRowsPer * i + sub;
        if (r < N) __builtin_nontemporal_store(x[i], qd + (uint32_t)r * vw.st16 + chunk);
      }
      if (in_tile == 0 && tid == 0) has_cache[tile] = 1;
    }
  }
}

}  // namespace

int launch_attention_bf16(const TileView& tv, int heads, int head_dim, float scale, const AttnBatch& b, hipStream_t s) {
  if (head_dim != 128 && head_dim != 64) return SG_ERR_UNSUPPORTED;
  if (b.n_tiles <= 0) return SG_OK;
  int dev = 0, n_cu = 0;
  SG_HIP_TRY(hipGetDevice(&dev));
  SG_HIP_TRY(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
  // Windows of head_dim 64 that do not fill the pipeline of the streaming kernel take the register-staged one: up to 448 tokens, and up to
  // 960 where there are workgroups for more than half of the compute units.  (Fewer are dealt as halves here, which the other does
  // not do.)  Register-staged and streaming, us a step: 9 tiles, 24 heads, of 300 tokens 29.6 and 33.9, of 500 38.5 and 40.9, of 700 64.1
  // and 69.6, of 832 91.3 and 89.4, of 960 103.7 and 100.8, of 1,000 108 and 101, of 1,100 146 and 127, of 1,200 155 and 147; 20 tiles, 16
  // heads, of 770 115 and 120, of 960 133.8 and 133.5, of 1,100 201 and 180; 4 tiles, 12 heads, of 960 31.7 and 32.3, of 1,100 36.4 and
  // 35.2; 8 heads, of 400 17.5 and 18.6, of 512 18.7 and 17.7.
  if (head_dim == 64 && tv.window) {
    const int64_t workgroups = (int64_t)b.n_tiles * heads * ((tv.N + kBR - 1) / kBR);
    if (tv.N <= 448 || (tv.N <= 960 && 2 * workgroups > n_cu)) return launch_attention_bf16_short(tv, heads, scale, b, s);
  }
  const View16 vw = make_view16(tv);
  // Windows of head_dim 128 whose runs of 8 tokens all lie side by side (width a multiple of 8, none of the launch crosses a canvas
  // edge) are walked.  A step of 20 tiles of 75,600 tokens, 40 heads: 1,744 ms walked, 1,793 - 1,817 planned, 1,731 gathered and
  // packed; 9 tiles of 3,840 tokens 2.245 and 2.263 ms.  (A launch in which some windows wrap is planned as a whole: walking the
  // others in a launch of their own costs small steps a partial last round, 4 % at 9 tiles of 3,840 tokens.)
  bool wraps = false;
  for (int i = 0; i < b.n_tiles && tv.window; ++i) wraps = wraps || b.y0[i] + tv.th > tv.H || b.x0[i] + tv.tw > tv.W;
  const bool walk = head_dim == 128 && tv.window && !wraps && tv.tw % 8 == 0 && (vw.reach & kReachLane);
  // Windows of head_dim 64 and others whose offsets inside a head leave 32 bits are scaled late: these calls have always had the
  // smaller error (2.2e-3 against fp64, scaled first 2.9e-3).
  const bool late = head_dim == 64 || (!walk && !(vw.reach & kReachHead));
  // a packed tile whose tokens are so far apart that 16 of them span 4 GiB is read like a window (of itself)
  const bool window = tv.window || !(vw.reach & kReachLane);
  const int n_qblocks = (tv.N + kBR - 1) / kBR;
  const float c_log2 = scale * 1.4426950408889634f;
  // the kernels need more dynamic LDS than the default limit; the attribute is set once per device and kernel
  constexpr int kMaxDevices = 64;
  static std::atomic<bool> attr_set[kMaxDevices][16];   // zero-initialised; set twice by racing threads is harmless
  const int cu_per_xcd = n_cu / kXcd > 0 ? n_cu / kXcd : 1;
  // the cache refresh rides on this launch for packed tiles (their inputs are one contiguous run each)
  const bool fuse_refresh = b.refresh_dst && b.has_cache && !window;
  for (int t0 = 0; t0 < b.n_tiles; t0 += kAttnTilesPerLaunch) {
    const int n = (b.n_tiles - t0 < kAttnTilesPerLaunch) ? b.n_tiles - t0 : kAttnTilesPerLaunch;
    AttnTable tab;
    for (int i = 0; i < kAttnTilesPerLaunch; ++i) {
      const bool in = i < n;
      tab.q[i] = in ? b.q[t0 + i] : nullptr;
      tab.k[i] = in ? b.k[t0 + i] : nullptr;
      tab.v[i] = in ? b.v[t0 + i] : nullptr;
      tab.out[i] = in ? b.out[t0 + i] : nullptr;
      tab.y0[i] = (in && b.y0) ? b.y0[t0 + i] : 0;
      tab.x0[i] = (in && b.x0) ? b.x0[t0 + i] : 0;
    }
    const int64_t total = (int64_t)n * heads * n_qblocks;   // the grid covers every tile; skipped tiles' share exits at once
    const int64_t attn_blocks = ((total + kXcd - 1) / kXcd + cu_per_xcd / 2) * kXcd;   // with room for a halved last round
    if (attn_blocks > (1ll << 31) - 1) return SG_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)attn_blocks);
    const uint8_t* flags = b.run_flags ? b.run_flags + t0 : nullptr;
    for (int i = 0; i < kAttnTilesPerLaunch; ++i) tab.refresh[i] = (fuse_refresh && i < n) ? b.refresh_dst[t0 + i] : nullptr;
    auto launch = [&](auto kern, int slot) -> int {
      if (dev < 0 || dev >= kMaxDevices || !attr_set[dev][slot].load(std::memory_order_acquire)) {
        SG_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
        if (dev >= 0 && dev < kMaxDevices) attr_set[dev][slot].store(true, std::memory_order_release);
      }
      kern<<<grid, kThreads, kLdsBytes, s>>>(vw, c_log2, heads, n_qblocks, n, cu_per_xcd, tab, flags,
                                             fuse_refresh ? b.has_cache + t0 : nullptr);
      return SG_OK;
    };
    // Short form, us a step with the other form and with it, 9 tiles, 24 heads.  head_dim 128: 300 tokens 42.6 and 39.7, 700 87.7 and 82.7,
    // 1,365 256 and 250, 1,500 276 and 273, 2,000 417 and 418, 4,600 1,933 and 1,974; one tile of 700 20.0 and 18.2.  head_dim 64: refreshed, of
    // which six run, 300 52.9 and 50.9, 1,500 185 and 177, 3,000 481 and 477, 4,600 941 and 951; windows of 1,500 217 and 202, 3,000 674 and
    // 671, 4,600 1,419 and 1,440; packed without a refresh, 48 heads, 9 tiles of 400 101 and 97, 1,000 243 and 235, 2,000 657 and 649, 3,000
    // 1,270 and 1,275, one of 3,000 135 and 138 (8 heads 36.4 and 38.0).  Of many rounds, 20 tiles, 48 heads: head_dim 128, 1,000 626 and 606,
    // 1,536 1,190 and 1,180; head_dim 64, refreshed, 1,500 1,016 and 985, 3,000 2,895 and 2,878, windows of 1,500 887 and 834, 3,000 2,936 and 2,921.
    const bool plain64 = head_dim == 64 && !window && !fuse_refresh;
    const bool is_short = tv.N <= (plain64 ? 2048 : head_dim == 64 ? 3072 : 1536);   // 24 stages, 16
    int st = SG_OK;
#define SG_BF16(D, MODE, LATE, REFRESH, SLOT) \
  (is_short ? launch(attention_bf16_kernel<D, MODE, LATE, REFRESH, true>, SLOT) : launch(attention_bf16_kernel<D, MODE, LATE, REFRESH, false>, SLOT + 8))
    if (head_dim == 64)
      st = window ? SG_BF16(64, kWindow, true, false, 0) : fuse_refresh ? SG_BF16(64, kLinear, false, true, 1) : SG_BF16(64, kLinear, false, false, 2);
    else if (walk)
      st = SG_BF16(128, kWalk, false, false, 7);
    else if (window)
      st = late ? SG_BF16(128, kWindow, true, false, 3) : SG_BF16(128, kWindow, false, false, 4);
    else
      st = fuse_refresh ? SG_BF16(128, kLinear, false, true, 5) : SG_BF16(128, kLinear, false, false, 6);
#undef SG_BF16
    if (st != SG_OK) return st;
    SG_HIP_TRY(hipGetLastError());
  }
  if (b.refreshed) *b.refreshed = fuse_refresh;
  return SG_OK;
}

}  // namespace sg
