// Tile attention, fp32, on the bf16 matrix instruction (paper Section 2.1 "full attention" over one tile's T x tile_h x tile_w
// tokens; Section 3: tiles exchange no Q/K/V), for calls with enough queries to fill the device with workgroups of 128.
//
// Every fp32 number is the sum of three bf16 numbers, 24 bits in three times 8.  Of the nine products of two numbers' parts six count:
// 1 x 1, 1 x 2, 2 x 1, 2 x 2, 1 x 3, 3 x 1.  Every part is rounded, so the second is at most 2^-8 and the third 2^-17 of a number, and what
// is left out of a product 2^-24 of it (2 x 3 and 3 x 2; of N(0, 1) numbers 2^-27.4 in the mean square, where rounding the product to
// fp32 is 2^-25.2).  With a first part that is cut off, one instruction less, it would be 2^-22.  A bf16 product of 16 channels or
// keys takes 32 cycles, where the fp32 instruction takes 512: six of them 192.  The products of first parts are summed apart from
// the others, so that the full-size sums are rounded once per 16 channels or keys and the others' roundings are 2^-8 smaller.
// Error against fp64, fp32 instruction (channels in four chains, keys in four or eight shares) -> here: 2,880 tokens x 128 5.2e-7 ->
// 3.9e-7, 9,000 8.6e-7 -> 6.5e-7; 4,000 x 64 5.9e-7 -> 4.4e-7; 65 - 1,500 tokens a quarter smaller.
//
// A workgroup owns 128 queries of one head, 32 per wavefront, one wavefront per SIMD with the whole register file (Q's parts and two
// output sums take 224 of its 512 registers).  K and V of a stage (32 keys, head_dim 64: 64) are read as fp32, split in registers and
// stored to LDS once for the four wavefronts, double-buffered, one workgroup barrier per stage.  A wavefront's stream is laid out by
// hand, in steps of up to six vector instructions behind every matrix product: the softmax of stage j, whose probabilities are split
// as well, beside QK of stage j + 1, and the splitting of the next stages beside PV of stage j.  Products are transposed, S^T = K Q^T and
// O^T = V^T P^T, so that the probabilities stay in their lanes; V is stored transposed, 8 keys of a channel side by side, as one
// lane of PV contracts them.
//
// Numbers whose parts bf16's range does not hold (tell_range says which) are looked for on the way; a workgroup whose tile has one does its
// queries once more on the fp32 instruction, with the result and the range of the kernel for few queries, at 0.8 of its speed.  With such
// values against the fp32 instruction alone: the step of 2,880 tokens 1,547 us and 1,220, with one in the last stage 2,219; 120 heads of 129 tokens x
// 64 42 and 23.  (A second launch for them would need flags in memory, which the call does not have.)
//
// Bound: the vector instructions beside the products (matrix pipe busy 48 % of the cycles) and the clock, 2.06 GHz under this mix.  Measured,
// fp32 instruction -> here, us a step, on one box (others are up to 5 % faster): 4 tiles of 2,880 tokens, 8 heads x 128 1,225 -> 812 (167 TFLOP/s;
// a large fp32 matrix product 154), 16 heads x 64 1,286 -> 842; 9,000 tokens, 12 heads x 128 4,276 -> 3,119; 4 tiles of 700, 8 heads x 64 62 -> 50;
// 200 heads of 65 tokens x 128 23.3 -> 19.5.  Of the first, 0.8 % are the test of the values for 0.  Taken back:
// 8 wavefronts of 16 queries with 16x16x32 products, two per SIMD (821: twice the fragment reads, and a wavefront whose neighbour is at
// the barrier waits for every dependent product), V in rows with transposing reads (862).
#include <atomic>
#include <type_traits>
#include <utility>
#include "attention_f32_block.h"

namespace sg {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kBR = kWaves * 32;   // query rows per workgroup
constexpr int kXcd = 8;
constexpr int kRowBytes = 256;
constexpr int kPlane = 32 * kRowBytes;     // one part (first, second, third 8 bits) of a stage of K or V
constexpr int kStageBytes = 3 * kPlane;
constexpr int kVRegion = 2 * kStageBytes;
constexpr int kFlags = 4 * kStageBytes;    // [2][wavefront]
static_assert(kVRegion + 2 * kStageBytes == kFlags, "");
constexpr int kLdsBytes = kFlags + 2 * kWaves * 4;
static_assert(kBlockLds<1, 4> <= kLdsBytes, "the fp32 form of a workgroup's queries");
// What the parts hold (see tell_range)
constexpr float kMaxFactor = 1.152921504606846976e18f;   // 2^60: |q scale log2(e)|, |k|, |v|
constexpr uint32_t kMinValue2 = (127 - 100) << 24;       // bits of 2^-100, shifted left by one: |v| unless 0
constexpr float kLowest = -100.f;                        // log2 of a probability against the reference; below it values have to be in
constexpr float kWideMax = 16777216.f;                   // 2^24 ..
constexpr uint32_t kWideMin2 = (127 - 50) << 24;         // 2^-50
constexpr float kSlack = 24.f;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t cvt2(float a, float b) {
  const bf16x2 two = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, two);
}

// f(A), f(A + 1), .. f(B - 1) with constants
template <int A, class F, int... I>
__device__ __forceinline__ void for_each(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, A + I>{}), ...);
}
template <int A, int B, class F>
__device__ __forceinline__ void for_range(F&& f) {
  for_each<A>(f, std::make_integer_sequence<int, (B > A ? B - A : 0)>{});
}

template <int D, int MODE>
__global__ __launch_bounds__(kThreads, 1) void attention_f32_split_kernel(const View16 vw, const float scale, const double c_log2, const int heads,
                                                                          const int n_qblocks, const int n_tiles, const AttnTable tab,
                                                                          const uint32_t head_bytes, const uint8_t* __restrict__ run_flags) {
  constexpr int kPar = 128 / D;             // keys in a slot, an LDS row of 256 bytes
  constexpr int kKeys = 32 * kPar;          // keys per stage
  constexpr int kDB = D / 32;               // output blocks of 32 channels
  constexpr int kKK = D / 16;               // products per score chain
  constexpr int kNP = 8 * kPar;             // pairs of scores a lane holds of a stage: of score block b, key b of the slots
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  SG_LDS uint8_t* const lds = (SG_LDS uint8_t*)smem;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

  const uint32_t active = attn_active_mask(run_flags, n_tiles);
  const int per_tile = heads * n_qblocks;
  const int total = __builtin_popcount(active) * per_tile;
  const int per_xcd = (total + kXcd - 1) / kXcd;
  const int slot_x = blockIdx.x / kXcd;
  const int logical = (blockIdx.x % kXcd) * per_xcd + slot_x;
  if (slot_x >= per_xcd || logical >= total) return;
  const int nth = logical / per_tile, in_tile = logical - nth * per_tile;
  const int tile = __builtin_amdgcn_readfirstlane(attn_nth_tile(active, nth));
  const int head = __builtin_amdgcn_readfirstlane(in_tile / n_qblocks), qblk = in_tile - head * n_qblocks;
  const int wy0 = (MODE == kWindow) ? tab.y0[tile] : 0, wx0 = (MODE == kWindow) ? tab.x0[tile] : 0;
  // offset of tile token n from the tile's pointers, in units of 8 elements (32 bytes)
  auto token_off8 = [&](int n) SG_INLINE -> uint32_t {
    return (MODE == kLinear) ? (uint32_t)n * vw.st16 : window_token(vw, n, wy0, wx0).off16;
  };
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, half = lane >> 5;
  const int N = vw.N;
  const int n_blocks = (N + kKeys - 1) / kKeys;
  const bool tail = (N % kKeys) != 0;
  const size_t head_off = (size_t)head * vw.head16 * 32;
  const char* const qh = (const char*)tab.q[tile] + head_off;
  const char* const kh = (const char*)tab.k[tile] + head_off;
  const char* const vh = (const char*)tab.v[tile] + head_off;
  const int q0 = qblk * kBR + wave * 32;
  const char* const q_row = qh + (size_t)token_off8(q0 + lq < N ? q0 + lq : N - 1) * 32;

  // ---- three bf16 parts of four fp32 numbers, each the nearest to what is left, so that they add up to the number; the second is at most
  // 2^-8 of the number's power of two, the third 2^-17.  In five steps, of which the first and the third are a conversion and what
  // takes its result (a dependent instruction waits 9 cycles); no more than six instructions fit between two matrix products.
  struct Split {
    float x[4];            // the numbers, what is left of them
    float y[4];
    uint32_t h[2], m[2], l[2];
    __device__ __forceinline__ void step(int i) {
      if (i == 0 || i == 2) {
        uint32_t (&part)[2] = (i == 0) ? h : m;
#pragma unroll
        for (int e = 0; e < 2; ++e) part[e] = cvt2(x[2 * e], x[2 * e + 1]);
        asm volatile("" : "+v"(part[0]), "+v"(part[1]));   // both halves from this one
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          y[2 * e] = __uint_as_float(part[e] << 16);
          y[2 * e + 1] = __uint_as_float(part[e] & 0xffff0000u);
        }
        asm volatile("" : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3]));
      } else if (i == 1 || i == 3) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] -= y[e];
        asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
      } else {
#pragma unroll
        for (int e = 0; e < 2; ++e) l[e] = cvt2(x[2 * e], x[2 * e + 1]);
        asm volatile("" : "+v"(l[0]), "+v"(l[1]));
      }
    }
  };
  constexpr int kSplitSteps = 5;

  // ---- Q (B operand of S^T): query q0 + lq, step kk: channels 16 kk + 8 half + 0..7
  bf16x8 qf[3][kKK];
  float factor_most = 0.f;   // largest |q scale| and |k| that this lane has seen, largest and smallest |v|
#pragma unroll
  for (int kk = 0; kk < kKK; ++kk) {
    const f32x4 x0 = *(const f32x4*)(q_row + (16 * kk + 8 * half) * 4), x1 = *(const f32x4*)(q_row + (16 * kk + 8 * half) * 4 + 16);
    u32x4 part[3];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      Split s;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        s.x[c] = (float)((e == 0 ? x0[c] : x1[c]) * c_log2);
        factor_most = fmaxf(factor_most, fabsf(s.x[c]));
      }
#pragma unroll
      for (int i = 0; i < kSplitSteps; ++i) s.step(i);
#pragma unroll
      for (int c = 0; c < 2; ++c) { part[0][2 * e + c] = s.h[c]; part[1][2 * e + c] = s.m[c]; part[2][2 * e + c] = s.l[c]; }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      qf[i][kk] = __builtin_bit_cast(bf16x8, part[i]);
      asm volatile("" : "+a"(qf[i][kk]));   // AccVGPRs are their home
    }
  }

  // ---- staging.  K: thread t moves 4 channels (of key t / 16 % 2 of the slot, head_dim 64) of slots t / 32 + 8 u of every stage;
  // 16-byte chunk c of slot r sits at chunk c ^ (r % 16).  V: thread t moves 8 slots of channels 2 (t % 64) and + 1, those slots that one
  // lane of PV contracts, so that V lies transposed: row = key of the slot * 64 + channel, 4 chunks of 8 slots, chunk g at
  // g ^ (row / 4 % 4) of row row ^ (row / 16 % 2).  Fragment reads and stores are laid out over all banks (14 % of the LDS cycles are conflicts even so).
  const int k_slot = tid >> 5, k_par = (D == 128) ? 0 : ((tid >> 4) & 1);
  const uint32_t k_ch4 = (tid & (D / 4 - 1)) * 16;
  uint32_t kdst[2];   // u even, odd (+ 16 slots for u >= 2)
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int r = k_slot + 8 * u;
    kdst[u] = lds0 + r * kRowBytes + ((((tid & 31) >> 1) ^ (r & 15)) << 4) + 8 * (tid & 1);
  }
  const int v_row = 2 * lane, v_par = (D == 128) ? 0 : (v_row >> 6);
  const uint32_t v_ch4 = ((D == 128) ? v_row : (v_row & 63)) * 4;
  const uint32_t vdst0 = lds0 + kVRegion + (v_row ^ ((v_row >> 4) & 1)) * 64 + ((wave ^ ((v_row >> 2) & 3)) << 4);
  const uint32_t vdst1 = vdst0 ^ 64;   // of the second channel
  // slot e of this wavefront's chunk, g = 2 ks + half
  auto v_slot = [&](int e) SG_INLINE -> int { return 16 * (wave >> 1) + 4 * (wave & 1) + 8 * (e >> 2) + (e & 3); };
  f32x4 kx[4];
  f32x2 vx[8];
  uint32_t k_from[4];              // of this thread's K
  uint32_t off_k = 0, off_v = 0;   // lane l: byte offset of key l % kKeys of the stage whose K was requested last, whose V comes next
  auto next_offsets = [&](int stage) SG_INLINE {
    const int n = stage * kKeys + (lane & (kKeys - 1));
    off_v = off_k;
    off_k = token_off8(n < N ? n : N - 1) * 32;
#pragma unroll
    for (int u = 0; u < 4; ++u) k_from[u] = (uint32_t)__shfl((int)off_k, kPar * (k_slot + 8 * u) + k_par, 64) + k_ch4;
  };
  auto load_k = [&](int u) SG_INLINE { kx[u] = *(const f32x4*)(kh + k_from[u]); };
  auto load_v = [&](int e) SG_INLINE {
    if constexpr (D == 128) {
      const uint32_t off = __builtin_amdgcn_readlane(off_v, v_slot(e));
      vx[e] = *(const f32x2*)(vh + (off + v_ch4));
    } else {   // the lanes' channels are those of two keys
      const uint32_t off0 = __builtin_amdgcn_readlane(off_v, 2 * v_slot(e)), off1 = __builtin_amdgcn_readlane(off_v, 2 * v_slot(e) + 1);
      vx[e] = *(const f32x2*)(vh + ((v_par ? off1 : off0) + v_ch4));
    }
  };
  float v_most = 0.f;
  Split sp;
  u32x4 vpart[3];
  // steps of moving a stage of K: range, 4 x (four elements, store), requests; of V: range, 2 channels x (2 x four elements, store), requests
  constexpr int kKQuad = kSplitSteps + 1, kKSteps = 2 + 4 * kKQuad + 4, kVChannel = 2 * kSplitSteps + 1, kVRange = 8, kVSteps = kVRange + 2 * kVChannel + 8;
  auto range_step = [&](float a, float b, float& most) SG_INLINE { most = fmaxf(fmaxf(most, fabsf(a)), fabsf(b)); };
  float most2[2] = {0.f, 0.f};   // in two chains
  uint32_t least2[2] = {0xffffffffu, 0xffffffffu};
  uint32_t zeros2[2] = {0, 0};   // all bits set: a value of 0 has been seen
  auto k_step = [&](auto m_tag, int j) SG_INLINE {
    constexpr int m = decltype(m_tag)::value;
    if constexpr (m < 2) {
#pragma unroll
      for (int e = 0; e < 8; e += 2) range_step(kx[2 * m + (e >> 2)][e & 3], kx[2 * m + (e >> 2)][(e & 3) + 1], (e & 2) ? most2[1] : most2[0]);
      asm volatile("" : "+v"(most2[0]), "+v"(most2[1]));
    } else if constexpr (m < 2 + 4 * kKQuad) {
      constexpr int u = (m - 2) / kKQuad, i = (m - 2) % kKQuad;
      if constexpr (i < kSplitSteps) {
        if constexpr (i == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) sp.x[e] = kx[u][e];
        }
        sp.step(i);
      } else {
        const uint32_t dst = kdst[u & 1] + (j & 1) * kStageBytes + (u >> 1) * (16 * kRowBytes);
        *(SG_LDS u32x2*)(uintptr_t)dst = u32x2{sp.h[0], sp.h[1]};
        *(SG_LDS u32x2*)(uintptr_t)(dst + kPlane) = u32x2{sp.m[0], sp.m[1]};
        *(SG_LDS u32x2*)(uintptr_t)(dst + 2 * kPlane) = u32x2{sp.l[0], sp.l[1]};
      }
    } else {
      load_k(m - 2 - 4 * kKQuad);
    }
  };
  auto v_step = [&](auto m_tag, int j) SG_INLINE {
    constexpr int m = decltype(m_tag)::value;
    if constexpr (m < kVRange) {
      constexpr int e = 2 * (m & 3);
      const float a = vx[e][m >> 2], b = vx[e + 1][m >> 2];
      range_step(a, b, v_most);
      const uint32_t ta = (__float_as_uint(a) << 1) - 1u, tb = (__float_as_uint(b) << 1) - 1u;   // a zero becomes the largest
      const uint32_t lo = ta < tb ? ta : tb, hi = ta < tb ? tb : ta;
      least2[m & 1] = lo < least2[m & 1] ? lo : least2[m & 1];
      zeros2[m & 1] = hi > zeros2[m & 1] ? hi : zeros2[m & 1];
      asm volatile("" : "+v"(v_most), "+v"(least2[m & 1]), "+v"(zeros2[m & 1]));
    } else if constexpr (m < kVRange + 2 * kVChannel) {
      constexpr int c = (m - kVRange) / kVChannel, at = (m - kVRange) % kVChannel, q = at / kSplitSteps, i = at % kSplitSteps;
      if constexpr (at < 2 * kSplitSteps) {
        if constexpr (i == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) sp.x[e] = vx[4 * q + e][c];
        }
        sp.step(i);
        if constexpr (i == kSplitSteps - 1) {
#pragma unroll
          for (int e = 0; e < 2; ++e) { vpart[0][2 * q + e] = sp.h[e]; vpart[1][2 * q + e] = sp.m[e]; vpart[2][2 * q + e] = sp.l[e]; }
        }
      } else {
        const uint32_t dst = (c ? vdst1 : vdst0) + ((j + 1) & 1) * kStageBytes;
#pragma unroll
        for (int x = 0; x < 3; ++x) *(SG_LDS u32x4*)(uintptr_t)(dst + x * kPlane) = vpart[x];
      }
    } else {
      load_v(m - kVRange - 2 * kVChannel);
    }
  };
  auto fill_tail_values = [&](int stage) SG_INLINE {   // values of keys >= N, whose probability is 0: neither an infinite last one nor 0
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (stage * kKeys + kPar * v_slot(e) + v_par >= N) vx[e] = f32x2{1.f, 1.f};
  };
  // K of stage j + 2 and V of stage j + 1 are in registers: their parts go to LDS, K of stage j + 3 and V of stage j + 2 are requested
  constexpr int kStageSteps = kKSteps + kVSteps;
  auto stage_step = [&](auto m_tag, int j) SG_INLINE {
    constexpr int m = decltype(m_tag)::value;
    if constexpr (m < kKSteps) k_step(m_tag, j);
    else v_step(std::integral_constant<int, m - kKSteps>{}, j);
  };
  auto stage_begin = [&](int j) SG_INLINE {
    next_offsets(j + 3);
    if (tail && j + 1 == n_blocks - 1) fill_tail_values(j + 1);
  };
  // What a wavefront has seen goes into one of two sets of flags, in turn: a wavefront that still reads one is not overtaken, as a barrier
  // lies between two calls.  The three parts of a factor or value hold all its 24 bits, and no sum overflows, if it lies between
  // 2^-100 and 2^60; below that factors are of no weight, values are if they are 0.  Probabilities below 2^-100 lose bits and below
  // 2^-126 are 0.  That is of no weight beside the key that the reference comes from, with its probability of 1 or more, if all values lie
  // between 2^-50 and 2^24; if that key's value is 0, such probabilities may be all that a channel holds.
  float gap = 0.f;   // the lowest log2 of a probability
  int told = 0;
  auto tell_range = [&]() SG_INLINE {
    const float factor = fmaxf(factor_most, fmaxf(most2[0], most2[1]));
    const uint32_t least = least2[0] < least2[1] ? least2[0] : least2[1];
    const bool zero = (zeros2[0] > zeros2[1] ? zeros2[0] : zeros2[1]) == 0xffffffffu;
    const uint32_t seen = (__any(!(factor < kMaxFactor) || !(v_most < kMaxFactor) || least < kMinValue2) ? 1u : 0u) |
                          (__any(gap < kLowest) ? 2u : 0u) | (__any(!(v_most < kWideMax) || least < kWideMin2 || zero) ? 4u : 0u);
    if (lane == 0) *(SG_LDS uint32_t*)(uintptr_t)(lds0 + kFlags + (told & 1) * (kWaves * 4) + wave * 4) = seen;
  };
  auto meet = [&]() SG_INLINE {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto out_of_range = [&]() SG_INLINE -> bool {   // behind the barrier: the same in all wavefronts
    const uint32_t at = lds0 + kFlags + (told & 1) * (kWaves * 4);
    const u32x4 f = *(const SG_LDS u32x4*)(uintptr_t)at;
    ++told;
    const uint32_t seen = __builtin_amdgcn_readfirstlane(f[0] | f[1] | f[2] | f[3]);
    return (seen & 1u) || (seen & 6u) == 6u;
  };

  // ---- fragments
  uint32_t kaddr[8];   // A operand of QK: slot lq, chunk 2 c2 + half
#pragma unroll
  for (int c2 = 0; c2 < 8; ++c2) kaddr[c2] = lds0 + lq * kRowBytes + (((2 * c2 + half) ^ (lq & 15)) << 4);
  uint32_t vaddr[2];   // A operand of PV: row 32 rb + lq of V^T, chunk 2 ks + half
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) vaddr[ks] = lds0 + kVRegion + (lq ^ (lq >> 4)) * 64 + (((2 * ks + half) ^ ((lq >> 2) & 3)) << 4);
  // with the address of the ring slot's chunk; parts and rows enter as immediates
  auto kfrag = [&](uint32_t at, int part) SG_INLINE -> bf16x8 {
    return __builtin_bit_cast(bf16x8, *(const SG_LDS u32x4*)(uintptr_t)(at + part * kPlane));
  };
  auto vfrag = [&](uint32_t at, int rb, int part) SG_INLINE -> bf16x8 {
    return __builtin_bit_cast(bf16x8, *(const SG_LDS u32x4*)(uintptr_t)(at + part * kPlane + rb * 2048));
  };
  f32x16 ohi[kDB], olo[kDB];    // output: products of the first parts; the others
  f32x16 shi[kPar], slo[kPar];  // scores of the next stage, alike: register r of block b is slot 8 (r >> 2) + 4 half + (r & 3), key b of it
#pragma unroll
  for (int db = 0; db < kDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) ohi[db][r] = olo[db][r] = 0.f;
  float ref = -__builtin_inff(), l = 0.f;   // softmax reference, this lane's share of the sum

  // products (part of A, part of B) of a group of six, the smallest first, and the order in which A's parts are needed
  constexpr int kPa[6] = {2, 0, 1, 1, 0, 0}, kPb[6] = {0, 2, 1, 0, 1, 0}, kOrder[3] = {2, 0, 1};
  // The products are written as assembly, which gives every operand its register file: the output and Q take the AccVGPRs (left to
  // the compiler the output moves between the files around every rescaling).  No hazard recogniser sees into it: wait_products stands
  // wherever the vector ALU may follow a product whose sum it reads or changes.
  auto wait_products = []() SG_INLINE { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); };
  // group g of QK: chunks 2 g and 2 g + 1 of the slots; block b's chunks begin at b * kKK * 2
  auto qk_product = [&](auto g_tag, auto x_tag, const bf16x8 (&a)[3]) SG_INLINE {
    constexpr int g = decltype(g_tag)::value, x = decltype(x_tag)::value, b = g % kPar, kk = g / kPar;
    f32x16& acc = x < 5 ? slo[b] : shi[b];
    const bf16x8 &ka = a[kPa[x]], &qb = qf[kPb[x]][kk];
    if constexpr (kk == 0 && (x == 0 || x == 5)) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(ka), "a"(qb));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(ka), "a"(qb));
  };
  auto qk_chunk = [](int g) SG_INLINE -> int { return (g % kPar) * kKK + g / kPar; };
  auto pv_product = [&](f32x16& acc, const bf16x8& va, const bf16x8& pb) SG_INLINE {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(va), "v"(pb));
  };

  float t[2 * kNP];             // scores of the stage
  auto mask_tail = [&](int stage) SG_INLINE {
#pragma unroll
    for (int i = 0; i < 2 * kNP; ++i) {
      const int r = i & 15, slot = 8 * (r >> 2) + 4 * half + (r & 3);
      if (stage * kKeys + kPar * slot + (i >> 4) >= N) t[i] = -__builtin_inff();
    }
  };
  // over the two lanes of a query
  auto both_halves = [&](float x, auto op) SG_INLINE -> float {
    const uint32_t u = __float_as_uint(x);
    const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return op(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  auto move_reference = [&](float to) SG_INLINE {
    const float alpha = (ref == to) ? 1.f : exp2f(ref - to);
    ref = to;
    l *= alpha;
    wait_products();
#pragma unroll
    for (int db = 0; db < kDB; ++db) {
      ohi[db] *= alpha;
      olo[db] *= alpha;
      asm volatile("" : "+a"(ohi[db]), "+a"(olo[db]));
    }
  };

  // ---- steps of the softmax of a stage, dealt between the products of QK
  u32x4 pw[3][2 * kPar];   // parts of the probabilities, B operand of PV: [part][2 * key of a slot + ks]
  float base = 0.f, mn = 0.f, mxs[2], sum[4];
  Split ps;
  constexpr int kAddSteps = 4 * kPar, kMaxSteps = 2 * kPar, kQuadSteps = 4 + kSplitSteps;
  constexpr int kSoftSteps = kAddSteps + kMaxSteps + 1 + kNP / 2 * kQuadSteps;
  auto soft_step = [&](auto m_tag, int j) SG_INLINE {
    constexpr int m = decltype(m_tag)::value;
    if constexpr (m < kAddSteps) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 4 * m + e;
        t[i] = shi[i >> 4][i & 15] + slo[i >> 4][i & 15];
        asm volatile("" : "+v"(t[i]));
      }
      if (m == 0) mn = t[0];
      mn = fminf(fminf(mn, t[4 * m]), t[4 * m + 1]);
      mn = fminf(fminf(mn, t[4 * m + 2]), t[4 * m + 3]);
      asm volatile("" : "+v"(mn));
      if (m == kAddSteps - 1 && tail && j == n_blocks - 1) mask_tail(j);
    } else if constexpr (m < kAddSteps + kMaxSteps) {
      constexpr int i = 8 * (m - kAddSteps);
      if (i == 0) mxs[0] = mxs[1] = -__builtin_inff();
#pragma unroll
      for (int e = 0; e < 8; e += 4) {
        mxs[0] = fmaxf(fmaxf(mxs[0], t[i + e]), t[i + e + 1]);
        mxs[1] = fmaxf(fmaxf(mxs[1], t[i + e + 2]), t[i + e + 3]);
      }
      asm volatile("" : "+v"(mxs[0]), "+v"(mxs[1]));
    } else if constexpr (m == kAddSteps + kMaxSteps) {
      const float mx = both_halves(fmaxf(mxs[0], mxs[1]), [](float x, float y) { return fmaxf(x, y); });
      if (__builtin_expect(__any(mx > ref + kSlack), 0)) move_reference(fmaxf(ref, mx));
      base = (ref == -__builtin_inff()) ? 0.f : ref;
      gap = fminf(gap, mn - base);
      sum[0] = sum[1] = sum[2] = sum[3] = 0.f;
    } else {
      constexpr int q = (m - kAddSteps - kMaxSteps - 1) / kQuadSteps, i = (m - kAddSteps - kMaxSteps - 1) % kQuadSteps;
      if constexpr (i == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) ps.x[e] = t[4 * q + e] - base;
        asm volatile("" : "+v"(ps.x[0]), "+v"(ps.x[1]), "+v"(ps.x[2]), "+v"(ps.x[3]));
      } else if constexpr (i < 3) {
#pragma unroll
        for (int e = 2 * (i - 1); e < 2 * i; ++e) {
          ps.x[e] = __builtin_amdgcn_exp2f(ps.x[e]);
          asm volatile("" : "+v"(ps.x[e]));
        }
      } else if constexpr (i == 3) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sum[e] += ps.x[e];
          asm volatile("" : "+v"(sum[e]));
        }
      } else {
        ps.step(i - 4);
        if constexpr (i == kQuadSteps - 1) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            pw[0][q >> 1][2 * (q & 1) + e] = ps.h[e];
            pw[1][q >> 1][2 * (q & 1) + e] = ps.m[e];
            pw[2][q >> 1][2 * (q & 1) + e] = ps.l[e];
          }
        }
      }
    }
  };

  // ---- start: K of stages 0 and 1 and V of stage 0 in LDS, K of stage 2 and V of stage 1 in registers
  next_offsets(0);
#pragma unroll
  for (int u = 0; u < 4; ++u) load_k(u);
  for_range<-2, 0>([&](auto j_tag) SG_INLINE {   // K of stage j + 2, V of stage j + 1
    constexpr int j = decltype(j_tag)::value;
    next_offsets(j + 3);
    if (j == -1 && tail && n_blocks == 1) fill_tail_values(0);
    for_range<0, kStageSteps>([&](auto m) SG_INLINE {   // no V in the first: only its requests
      if constexpr (j == -1 || m < kKSteps || m >= kStageSteps - 8) stage_step(m, j);
    });
  });
  tell_range();
  meet();
  bool narrow = out_of_range();
  for_range<0, 8>([&](auto g) SG_INLINE {
    bf16x8 a[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) a[i] = kfrag(kaddr[qk_chunk(g)], i);
    for_range<0, 6>([&](auto x) SG_INLINE { qk_product(g, x, a); });
  });
  wait_products();
  meet();   // all wavefronts have read K of stage 0: the first iteration stores K of stage 2 in its place

  for (int j = 0; j < n_blocks && !narrow; ++j) {
    const int koff = ((j + 1) & 1) * kStageBytes, voff = (j & 1) * kStageBytes;
    bf16x8 a[2][3];
#pragma unroll
    for (int i = 0; i < 3; ++i) a[0][kOrder[i]] = kfrag(kaddr[qk_chunk(0)] + koff, kOrder[i]);
    uint32_t k_at[2], v_at[2];   // of the group to read next
    stage_begin(j);
    // QK of stage j + 1 beside the softmax of stage j.  (Behind the last stage the products are of stale keys and not used.)
    for_range<0, kAddSteps>([&](auto m) SG_INLINE { soft_step(m, j); });
    for_range<0, 48>([&](auto at_tag) SG_INLINE {
      constexpr int at = decltype(at_tag)::value, g = at / 6, x = at % 6, kLeft = kSoftSteps - kAddSteps;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (x == 0 && g < 7) {
        k_at[g & 1] = kaddr[qk_chunk(g + 1)] + koff;
        asm volatile("" : "+v"(k_at[g & 1]));
      }
      if constexpr (x < 3 && g < 7) a[(g + 1) & 1][kOrder[x]] = kfrag(k_at[g & 1], kOrder[x]);
      qk_product(std::integral_constant<int, g>{}, std::integral_constant<int, x>{}, a[g & 1]);
      for_range<kAddSteps + at * kLeft / 48, kAddSteps + (at + 1) * kLeft / 48>([&](auto m) SG_INLINE { soft_step(m, j); });
      __builtin_amdgcn_sched_barrier(0);
    });
    l += (sum[0] + sum[1]) + (sum[2] + sum[3]);
    // PV of stage j beside the staging; group (ks, rb): 16 slots, rows 32 rb .. of V^T
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      v_at[ks] = vaddr[ks] + voff;
      asm volatile("" : "+v"(v_at[ks]));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) a[0][kOrder[i]] = vfrag(v_at[0], 0, kOrder[i]);
    asm volatile("s_nop 4" : "+v"(pw[0][2 * kPar - 1]), "+v"(pw[1][2 * kPar - 1]), "+v"(pw[2][2 * kPar - 1]));
    for_range<0, 48>([&](auto at_tag) SG_INLINE {
      constexpr int at = decltype(at_tag)::value, g = at / 6, x = at % 6, ks = g >> 2, rb = g & 3, acc = rb % kDB, px = 2 * (rb / kDB) + ks;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (x < 3 && g < 7) a[(g + 1) & 1][kOrder[x]] = vfrag(v_at[(g + 1) >> 2], (g + 1) & 3, kOrder[x]);
      pv_product(x < 5 ? olo[acc] : ohi[acc], a[g & 1][kPa[x]], __builtin_bit_cast(bf16x8, pw[kPb[x]][px]));
      for_range<at * kStageSteps / 48, (at + 1) * kStageSteps / 48>([&](auto m) SG_INLINE { stage_step(m, j); });
      __builtin_amdgcn_sched_barrier(0);
    });
    const bool tell = (j & 15) == 15 || j == n_blocks - 1;
    if (tell) tell_range();
    meet();
    if (tell) narrow = out_of_range();
  }
  if (narrow) {   // numbers beyond the parts' range: all over on the fp32 instruction
    for (int i = 0; i < kWaves && qblk * kBR + 32 * i < N; ++i) {   // the same in all wavefronts
      attend_f32<D, 1, 4, MODE, false>(vw, scale, tab, head_bytes, tile, head, qblk * kBR + 32 * i, wy0, wx0, lds);
      __syncthreads();
    }
    return;
  }

  wait_products();
  // ---- output: lane holds query q0 + lq; register r of block db is channel 32 db + 8 (r >> 2) + 4 half + (r & 3)
  const float inv = 1.0f / both_halves(l, [](float x, float y) { return x + y; });
  if (q0 + lq < N) {
    float* const dst = (float*)tab.out[tile] + ((size_t)head * N + q0 + lq) * D + 4 * half;
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (ohi[db][4 * g + e] + olo[db][4 * g + e]) * inv;
        *(f32x4*)(dst + 32 * db + 8 * g) = o;
      }
  }
}

}  // namespace

int launch_attention_f32_split(const View16& vw, bool window, int heads, int head_dim, float scale, int n_tiles, const AttnTable& tab,
                               uint32_t head_bytes, const uint8_t* run_flags, int dev, hipStream_t s) {
  const int n_qblocks = (vw.N + kBR - 1) / kBR;
  constexpr int kMaxDevices = 64;
  static std::atomic<bool> attr_set[kMaxDevices][4];   // zero-initialised; set twice by racing threads is harmless
  const int64_t total = (int64_t)n_tiles * heads * n_qblocks;
  const dim3 grid((unsigned)(((total + kXcd - 1) / kXcd) * kXcd));
  auto launch = [&](auto kern, int slot) -> int {
    if (dev < 0 || dev >= kMaxDevices || !attr_set[dev][slot].load(std::memory_order_acquire)) {
      SG_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
      if (dev >= 0 && dev < kMaxDevices) attr_set[dev][slot].store(true, std::memory_order_release);
    }
    kern<<<grid, kThreads, kLdsBytes, s>>>(vw, scale, (double)scale * 1.4426950408889634, heads, n_qblocks, n_tiles, tab, head_bytes, run_flags);
    return SG_OK;
  };
  if (head_dim == 128) return window ? launch(attention_f32_split_kernel<128, kWindow>, 0) : launch(attention_f32_split_kernel<128, kLinear>, 1);
  return window ? launch(attention_f32_split_kernel<64, kWindow>, 2) : launch(attention_f32_split_kernel<64, kLinear>, 3);
}

}  // namespace sg
