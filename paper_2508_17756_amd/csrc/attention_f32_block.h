// Attention of QB x 32 queries over all keys of a tile, fp32 on the fp32 matrix instruction (see attention_f32.hip): the body of that
// kernel, and what the split kernel (attention_f32_split.hip) does with queries whose tile holds numbers out of its range.
#pragma once
#include "attention_common.h"

namespace sg {
namespace {

#define SG_INLINE __attribute__((always_inline))

constexpr int kBlockKeys = 32;    // keys per block
constexpr float kLog2e = 1.4426950408889634f;
constexpr uint32_t kNowhere8 = 0x07ffff00;   // an offset (32-byte units) beyond every head that is not WIDE, whose bytes still fit 32 bits

constexpr int kWaveBytes = 16384;   // LDS of a wavefront: its K block, after the key loop its partial output
template <int QB, int KS>
constexpr int kBlockLds = KS * kWaveBytes + 2 * KS * QB * 32 * 4;   // and (reference, sum) per wavefront and query

enum { kLinear = 0, kWindow = 1 };   // how a tile token is found

// KS wavefronts = shares of the keys; WIDE: offsets inside a head leave 32 bits; head: the number of it, q0: the first query,
// (wy0, wx0): the canvas position of a window's first token
template <int D, int QB, int KS, int MODE, bool WIDE>
__device__ __forceinline__ void attend_f32(const View16& vw, const float scale, const AttnTable& tab, const uint32_t head_bytes, const int tile,
                                           const int head, const int q0, const int wy0, const int wx0, SG_LDS uint8_t* const lds) {
  static_assert(kBlockKeys * D * 4 <= kWaveBytes && QB * 32 * D * 4 <= kWaveBytes, "K block and partial output");
  constexpr int kPer = D / 32;   // channels a lane holds of one V row: output blocks
  // offset of tile token n from the tile's pointers, in units of 8 elements (32 bytes)
  auto token_off8 = [&](int n) SG_INLINE -> uint32_t {
    return (MODE == kLinear) ? (uint32_t)n * vw.st16 : window_token(vw, n, wy0, wx0).off16;
  };
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lq = lane & 31, half = lane >> 5;
  const int N = vw.N;
  const size_t head_off = (size_t)head * vw.head16 * 32;
  const char* const qh = (const char*)tab.q[tile] + head_off;
  const char* const kh = (const char*)tab.k[tile] + head_off;
  const char* const vh = (const char*)tab.v[tile] + head_off;

  // ---- Q (B operand of S^T): query lq, step (c, j) contracts channel 8 c + j in the lower, 8 c + 4 + j in the upper half
  float qr[QB][D / 8][4];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    int n = q0 + 32 * qb + lq;
    if (n > N - 1) n = N - 1;
    const float4* src = (const float4*)(qh + (size_t)token_off8(n) * 32);
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
      const float4 x = src[2 * c + half];
      qr[qb][c][0] = x.x * scale; qr[qb][c][1] = x.y * scale; qr[qb][c][2] = x.z * scale; qr[qb][c][3] = x.w * scale;
    }
  }

  // ---- loader: one instruction moves 1 KiB = kRows rows; 16-byte chunk c of K row r sits at chunk c ^ (r & 15), so that
  // the 32 rows read side by side (below) fall on different banks
  constexpr int kChunks = D / 4;                 // 16-byte chunks per row
  constexpr int kRows = 64 / kChunks;
  constexpr int kInstr = kBlockKeys / kRows;          // transfers per block: 16 (head_dim 64: 8)
  const int sub = lane / kChunks, slot = lane % kChunks;
  const uint32_t lds_k = (uint32_t)(uintptr_t)lds + wave * kWaveBytes;
  auto block_off8 = [&](int b) SG_INLINE -> uint32_t {   // lane l: where key l % 32 of block b lies (keys >= N: the last one)
    const int n = b * kBlockKeys + lq;
    return token_off8(n < N ? n : N - 1);
  };
  auto issue_k = [&](uint32_t off8) SG_INLINE {
#pragma unroll
    for (int i = 0; i < kInstr; ++i) {
      const int row = kRows * i + sub;
      const uint32_t o = (uint32_t)__shfl((int)off8, row, 64);
      dma16_addr(kh + (size_t)o * 32 + ((slot ^ (row & 15)) << 4), lds_k + i * 1024);
    }
  };
  // V straight into registers, one coalesced load per key pair (k, k + 4): the upper half of the wavefront reads row k + 4.  Keys >= N
  // stand in for the last one with probability 0, and their values have to be zeros, or an infinite last value becomes 0 * inf: they
  // get an offset beyond the head, for which a buffer load returns zeros.  (Selecting zeros for every pair costs 5 %; only heads
  // whose offsets leave 32 bits do.)
  typedef float vrow __attribute__((ext_vector_type(kPer)));
  const __amdgpu_buffer_rsrc_t vbuf = __builtin_amdgcn_make_buffer_rsrc((void*)vh, 0, WIDE ? 0 : (int)head_bytes, 0x00020000);
  auto value_off8 = [&](int b, uint32_t off8) SG_INLINE -> uint32_t { return (WIDE || b * kBlockKeys + lq < N) ? off8 : kNowhere8; };
  auto load_v = [&](uint32_t off8, int r) SG_INLINE -> vrow {
    const uint32_t o = (uint32_t)__shfl((int)off8, 8 * (r >> 2) + (r & 3) + 4 * half, 64);
    if constexpr (WIDE) return *(const vrow*)(vh + (size_t)o * 32 + lq * (kPer * 4));
    else if constexpr (kPer == 4) return __builtin_bit_cast(vrow, __builtin_amdgcn_raw_buffer_load_b128(vbuf, o * 32 + lq * 16, 0, 0));
    else return __builtin_bit_cast(vrow, __builtin_amdgcn_raw_buffer_load_b64(vbuf, o * 32 + lq * 8, 0, 0));
  };
  constexpr int kAhead = 4;   // key pairs whose V rows are in flight: 1,024 cycles of matrix work (head_dim 64, one query block: 512)
  auto reads_done = [&]() SG_INLINE {   // this wavefront's fragment reads have returned: the block may be overwritten
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };

  f32x16 acc[QB][kPer];
  float ref[QB], l[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
    for (int db = 0; db < kPer; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[qb][db][r] = 0.f;
    ref[qb] = -__builtin_inff();
    l[qb] = 0.f;
  }
  uint32_t kaddr[8];   // chunk 2 c + half of row lq; bit 4 of the chunk is not swizzled: chunk 16 and on lie 256 bytes behind
#pragma unroll
  for (int c = 0; c < 8; ++c) kaddr[c] = lds_k + lq * (D * 4) + (((2 * c + half) ^ (lq & 15)) << 4);
  auto kfrag = [&](int c) SG_INLINE -> f32x4 {
    return *(const SG_LDS f32x4*)(uintptr_t)(kaddr[c & 7] + (c >> 3) * 256);
  };

  const int n_blocks = (N + kBlockKeys - 1) / kBlockKeys;
  uint32_t off = 0;   // value_off8 of the block in work
  if (wave < n_blocks) {
    const uint32_t first = block_off8(wave);
    issue_k(first);
    off = value_off8(wave, first);
  }
  for (int b = wave; b < n_blocks; b += KS) {
    const bool more = b + KS < n_blocks;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // K of block b
    __builtin_amdgcn_sched_barrier(0);
    // ---- S^T = K Q^T; the channels in four chains one behind the other, each from zero, whose sums are added while the next one
    // runs.  Two chains have an error against fp64 of 2.4e-7 at 81 tokens of head_dim 128, four 1.9e-7, as four interleaved chains
    // on the vector ALU have; side by side they would keep a fourth accumulator alive (1.28 ms where this takes 1.22, two chains
    // 1.20; 4 tiles of 2,880 tokens).
    constexpr int kChain = D / 32;   // steps of 8 channels per chain
    constexpr int kSlot[4] = {0, 1, 2, 1};
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 s[QB][3];
    f32x4 a[D / 8];   // fragments are read two steps (512 cycles and more) ahead
    a[0] = kfrag(0);
    a[1] = kfrag(1);
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
      if (c + 2 < D / 8) a[c + 2] = kfrag(c + 2);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          f32x16& sum = s[qb][kSlot[c / kChain]];
          if (c % kChain == 0 && j == 0) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][j], qr[qb][c][j], zero, 0, 0, 0);
          else sum = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][j], qr[qb][c][j], sum, 0, 0, 0);
        }
      if (c % kChain == kChain / 2 && c / kChain >= 2) {   // the chain before is done
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          s[qb][0] += s[qb][kSlot[c / kChain - 1]];
          asm volatile("" : "+v"(s[qb][0]));   // here, not behind all chains
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    reads_done();
    uint32_t next = 0;
    if (more) {
      const uint32_t first = block_off8(b + KS);
      issue_k(first);
      next = value_off8(b + KS, first);
    }
    vrow v[16];
#pragma unroll
    for (int r = 0; r < kAhead; ++r) v[r] = load_v(off, r);
    __builtin_amdgcn_sched_barrier(0);
    // ---- softmax against the running maximum: no exponential is above 1, so sums of p v stay finite as long as the values do.  (A
    // reference that lags by up to e^5 saves half of the rescalings and 1.6 % of the time, and overflows from |v| = 2.3e36.)  It
    // is subtracted before the factor log2(e) of the exponent, so that scores up to the largest fp32 number stay finite.
    float p[QB][16];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) p[qb][r] = s[qb][0][r] + s[qb][1][r];   // (the fourth chain)
      if (b == n_blocks - 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (b * kBlockKeys + 8 * (r >> 2) + 4 * half + (r & 3) >= N) p[qb][r] = -__builtin_inff();
      }
      float mx = p[qb][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, p[qb][r]);
      const uint32_t mu = __float_as_uint(mx);
      const auto sw = __builtin_amdgcn_permlane32_swap(mu, mu, false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
      if (__any(!(mx <= ref[qb]))) {   // also the first block, where the reference is -inf
        const float moved = fmaxf(ref[qb], mx);
        const float alpha = (ref[qb] == moved) ? 1.f : exp2f((ref[qb] - moved) * kLog2e);
        ref[qb] = moved;
        l[qb] *= alpha;
#pragma unroll
        for (int db = 0; db < kPer; ++db) acc[qb][db] *= alpha;
      }
      float l0 = 0.f, l1 = 0.f;
      const float base = (ref[qb] == -__builtin_inff()) ? 0.f : ref[qb];   // all scores of this share -inf so far: probabilities 0
      // The exponential instruction returns 0 for results below 2^-126.  Where a score lies that far below the reference (or at -inf), the
      // function that returns them is called: times a value near the largest number they still count.  (Called always it costs
      // 2.5 %, this way 0.7 %.)
      float mn = p[qb][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mn = fminf(mn, p[qb][r]);
      if (__builtin_expect(__any(mn - base < -87.f), 0)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) p[qb][r] = exp2f((p[qb][r] - base) * kLog2e);
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) p[qb][r] = __builtin_amdgcn_exp2f((p[qb][r] - base) * kLog2e);
      }
#pragma unroll
      for (int r = 0; r < 16; r += 2) { l0 += p[qb][r]; l1 += p[qb][r + 1]; }
      l[qb] += l0 + l1;
    }
    // ---- O^T += V^T P^T: row m of output block db is channel kPer m + db
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (r + kAhead < 16) v[r + kAhead] = load_v(off, r + kAhead);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (WIDE) {
        const bool gone = b * kBlockKeys + 8 * (r >> 2) + 4 * half + (r & 3) >= N;
#pragma unroll
        for (int x = 0; x < kPer; ++x) v[r][x] = gone ? 0.f : v[r][x];
      }
#pragma unroll
      for (int db = 0; db < kPer; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) acc[qb][db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[r][db], p[qb][r], acc[qb][db], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    off = next;
  }

  // ---- merge the KS partial states of every query: a wavefront that saw no key has reference -inf, sum 0, output 0
  SG_LDS float* const s_ref = (SG_LDS float*)(lds + KS * kWaveBytes);   // [KS][QB * 32]
  SG_LDS float* const s_sum = s_ref + KS * QB * 32;
  // partial output of (wavefront, query): D floats, kPer-float groups at m ^ (query & 31) so that neither side conflicts
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const uint32_t lu = __float_as_uint(l[qb]);
    const auto sw = __builtin_amdgcn_permlane32_swap(lu, lu, false, false);
    if (half == 0) {
      s_ref[wave * (QB * 32) + 32 * qb + lq] = ref[qb];
      s_sum[wave * (QB * 32) + 32 * qb + lq] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = 8 * (r >> 2) + 4 * half + (r & 3);
      const uint32_t at = lds_k + (32 * qb + lq) * (D * 4) + (m ^ lq) * (kPer * 4);
      if constexpr (kPer == 4) {
        const f32x4 x = {acc[qb][0][r], acc[qb][1][r], acc[qb][2][r], acc[qb][3][r]};
        *(SG_LDS f32x4*)(uintptr_t)at = x;
      } else {
        const f32x2 x = {acc[qb][0][r], acc[qb][1][r]};
        *(SG_LDS f32x2*)(uintptr_t)at = x;
      }
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < QB * 32) {   // weights of the KS states, normalised, in place of the references
    const int q = threadIdx.x;
    float top = s_ref[q];
#pragma unroll
    for (int w = 1; w < KS; ++w) top = fmaxf(top, s_ref[w * (QB * 32) + q]);
    float wgt[KS], sum = 0.f;
#pragma unroll
    for (int w = 0; w < KS; ++w) {
      const float rw = s_ref[w * (QB * 32) + q];
      wgt[w] = (rw == -__builtin_inff()) ? 0.f : exp2f((rw - top) * kLog2e);
      sum += wgt[w] * s_sum[w * (QB * 32) + q];
    }
    const float inv = 1.0f / sum;
#pragma unroll
    for (int w = 0; w < KS; ++w) s_ref[w * (QB * 32) + q] = wgt[w] * inv;
  }
  __syncthreads();
  float* const out = (float*)tab.out[tile] + (size_t)head * N * D;
  for (int e = threadIdx.x; e < QB * 32 * 32; e += 64 * KS) {   // (query, group of kPer channels), group fastest
    const int q = e >> 5, m = e & 31;
    if (q0 + q >= N) break;   // queries rise with e
    float o[kPer];
#pragma unroll
    for (int x = 0; x < kPer; ++x) o[x] = 0.f;
#pragma unroll
    for (int w = 0; w < KS; ++w) {
      const float wgt = s_ref[w * (QB * 32) + q];
      const SG_LDS float* src = (const SG_LDS float*)(lds + w * kWaveBytes + q * (D * 4) + (m ^ (q & 31)) * (kPer * 4));
#pragma unroll
      for (int x = 0; x < kPer; ++x) o[x] = fmaf(wgt, src[x], o[x]);
    }
    float* dst = out + (size_t)(q0 + q) * D + m * kPer;
    if constexpr (kPer == 4) *(float4*)dst = make_float4(o[0], o[1], o[2], o[3]);
    else *(float2*)dst = make_float2(o[0], o[1]);
  }
}

}  // namespace

// The split kernel's launch over one table of tiles (attention_f32_split.hip).
int launch_attention_f32_split(const View16& vw, bool window, int heads, int head_dim, float scale, int n_tiles, const AttnTable& tab,
                               uint32_t head_bytes, const uint8_t* run_flags, int dev, hipStream_t s);

}  // namespace sg
