// Tile attention, fp32 throughout (paper Section 2.1 "full attention" restricted to one tile), for SG_F32
// problems, on the fp32 matrix instruction (32x32x2: fp32 operands, fp32 accumulation, 64 FLOP per cycle and
// SIMD; a large fp32 matrix product reaches 154 TFLOP/s on the same device).
//
// A workgroup owns QB x 32 query rows of one head and its KS wavefronts split the keys (wavefront w takes the
// 32-key blocks w, w + KS, ...), so that even one tile of a few hundred tokens gives every SIMD of its compute
// units work, and no workgroup barrier stands in the key loop: every wavefront moves its own K blocks into
// its own part of LDS (direct global->LDS transfers; K of the next block is requested when QK is done and, as
// transfers complete in order, has to arrive before the first V rows, which are requested behind it: it has the length of
// the softmax), reads its V rows straight into registers a few key pairs ahead, and keeps its own softmax state; the KS
// states of a query are merged through LDS at the end.  Two wavefronts per SIMD cover each other's softmax and waits.  (One
// wavefront per SIMD with 64 queries and V in LDS as well, which halves what is read per FLOP, spills its 512 registers around
// the rescaling of the accumulators: 2.14 ms where this takes 1.22.)
//
// Transposed products, S^T = K Q^T and O^T = V^T P^T, keep the probabilities in their lanes: accumulator register r
// of S^T holds, for the lane's query, key 8 (r >> 2) + (r & 3) in the lower and that key + 4 in the upper half of the
// wavefront, which is what the second product takes as its B operand for the key pair (k, k + 4).  The order of the
// channels inside either product is free, so they are numbered such that a lane's operands of four (head_dim 64: two)
// products are adjacent in LDS, and the results of a query adjacent in memory.
//
// Bound: matrix pipe (per 32 x 32 block and head_dim 128: 128 instructions of 64 cycles against 32 fragment reads
// and 16 exponentials a lane).  Measured, before (vector ALU, keys and values broadcast from LDS) -> now, whole steps:
// 4 tiles of 2,880 tokens, 8 heads x 128: 7.35 -> 1.22 ms (113 TFLOP/s in the kernel); 4 tiles of 300 tokens,
// 2 heads x 64: 75.6 -> 17.6 us.
#include <atomic>
#include "attention_common.h"

namespace sg {
namespace {

#define SG_INLINE __attribute__((always_inline))

constexpr int kKeys = 32;    // keys per block
constexpr int kXcd = 8;
constexpr float kLog2e = 1.4426950408889634f;
constexpr uint32_t kNowhere8 = 0x07ffff00;   // an offset (32-byte units) beyond every head that is not WIDE, whose bytes still fit 32 bits

constexpr int kWaveBytes = 16384;   // LDS of a wavefront: its K block, after the key loop its partial output
template <int QB, int KS>
constexpr int kLds = KS * kWaveBytes + 2 * KS * QB * 32 * 4;   // and (reference, sum) per wavefront and query

enum { kLinear = 0, kWindow = 1 };   // how a tile token is found

// KS wavefronts = shares of the keys; two wavefronts per SIMD either way: one workgroup of 8 per compute unit, or two of 4
// WIDE: offsets inside a head leave 32 bits
template <int D, int QB, int KS, int MODE, bool WIDE>
__global__ __launch_bounds__(64 * KS, 2) void attention_f32_kernel(
    const View16 vw, const float scale, const int heads, const int n_qblocks, const int n_tiles, const AttnTable tab,
    const uint32_t head_bytes, const uint8_t* __restrict__ run_flags) {
  static_assert(kKeys * D * 4 <= kWaveBytes && QB * 32 * D * 4 <= kWaveBytes, "K block and partial output");
  constexpr int kPer = D / 32;   // channels a lane holds of one V row: output blocks
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  SG_LDS uint8_t* const lds = (SG_LDS uint8_t*)smem;

  // (active tile, head, query block), query block fastest; each XCD walks a contiguous range (one head's K/V per L2)
  const uint32_t active = attn_active_mask(run_flags, n_tiles);
  const int per_tile = heads * n_qblocks;
  const int total = __builtin_popcount(active) * per_tile;
  const int per_xcd = (total + kXcd - 1) / kXcd;
  const int slot_x = blockIdx.x / kXcd;
  const int logical = (blockIdx.x % kXcd) * per_xcd + slot_x;
  if (slot_x >= per_xcd || logical >= total) return;
  const int nth = logical / per_tile, in_tile = logical - nth * per_tile;
  const int tile = __builtin_amdgcn_readfirstlane(attn_nth_tile(active, nth));
  const int head = in_tile / n_qblocks, qblk = in_tile - head * n_qblocks;
  const int wy0 = (MODE == kWindow) ? tab.y0[tile] : 0, wx0 = (MODE == kWindow) ? tab.x0[tile] : 0;
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
  const int q0 = qblk * (QB * 32);
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
  constexpr int kInstr = kKeys / kRows;          // transfers per block: 16 (head_dim 64: 8)
  const int sub = lane / kChunks, slot = lane % kChunks;
  const uint32_t lds_k = (uint32_t)(uintptr_t)lds + wave * kWaveBytes;
  auto block_off8 = [&](int b) SG_INLINE -> uint32_t {   // lane l: where key l % 32 of block b lies (keys >= N: the last one)
    const int n = b * kKeys + lq;
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
  auto value_off8 = [&](int b, uint32_t off8) SG_INLINE -> uint32_t { return (WIDE || b * kKeys + lq < N) ? off8 : kNowhere8; };
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

  const int n_blocks = (N + kKeys - 1) / kKeys;
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
          if (b * kKeys + 8 * (r >> 2) + 4 * half + (r & 3) >= N) p[qb][r] = -__builtin_inff();
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
        const bool gone = b * kKeys + 8 * (r >> 2) + 4 * half + (r & 3) >= N;
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

int launch_attention_f32(const TileView& tv, int heads, int head_dim, float scale, const AttnBatch& b, hipStream_t s) {
  if (head_dim != 64 && head_dim != 128) return SG_ERR_UNSUPPORTED;
  if (b.n_tiles <= 0) return SG_OK;
  const View16 vw = make_view16(tv);
  constexpr int kMaxDevices = 64;
  static std::atomic<bool> attr_set[kMaxDevices][20];   // zero-initialised; set twice by racing threads is harmless
  int dev = 0, n_cu = 0;
  SG_HIP_TRY(hipGetDevice(&dev));
  SG_HIP_TRY(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
  if (n_cu < 1) n_cu = 1;
  const int64_t head_units = (int64_t)tv.T * tv.H * tv.W * (tv.stride_token / 8);   // an upper bound of a head's extent, in 32 bytes
  const bool far = head_units > kNowhere8;
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
      tab.refresh[i] = nullptr;   // the cache refresh is not carried by this kernel
    }
    const uint8_t* flags = b.run_flags ? b.run_flags + t0 : nullptr;
    // 64 queries per workgroup (head_dim 64, heads within 32-bit offsets: the registers hold them) read K and V half as often as 32 but make half as many
    // workgroups: taken where their rounds over the device are not longer.  Then 4 shares of the keys, two workgroups per
    // compute unit, where there are that many workgroups: one's start, end and uneven last blocks run beside the other's loop.
    // Fewer workgroups take 8 shares, which halves the time of each.  (4 x 2,880 tokens, 8 heads x 128, 2,880 workgroups: 8 % more
    // a step with 8 shares than with 4.)
    const int64_t wg1 = (int64_t)n * heads * ((tv.N + 31) / 32), wg2 = (int64_t)n * heads * ((tv.N + 63) / 64);
    const bool two_blocks = head_dim == 64 && !far && 2 * ((wg2 + n_cu - 1) / n_cu) <= (wg1 + n_cu - 1) / n_cu;
    const int64_t total = two_blocks ? wg2 : wg1;
    const bool pairs = total >= 2 * n_cu;
    if (total > (1ll << 31) - 2 * kXcd) return SG_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)(((total + kXcd - 1) / kXcd) * kXcd));
    const int n_qblocks = (tv.N + (two_blocks ? 63 : 31)) / (two_blocks ? 64 : 32);
    auto launch = [&](auto kern, int shares, int lds, int slot) -> int {
      if (dev < 0 || dev >= kMaxDevices || !attr_set[dev][slot].load(std::memory_order_acquire)) {
        SG_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        if (dev >= 0 && dev < kMaxDevices) attr_set[dev][slot].store(true, std::memory_order_release);
      }
      kern<<<grid, 64 * shares, lds, s>>>(vw, scale, heads, n_qblocks, n, tab, (uint32_t)(head_units * 32), flags);
      return SG_OK;
    };
    int st;
#define SG_F32_MODES(D, QB, KS, WIDE, SLOT)                                                        \
  (tv.window ? launch(attention_f32_kernel<D, QB, KS, kWindow, WIDE>, KS, kLds<QB, KS>, SLOT)      \
             : launch(attention_f32_kernel<D, QB, KS, kLinear, WIDE>, KS, kLds<QB, KS>, SLOT + 1))
    if (far && head_dim == 128) st = pairs ? SG_F32_MODES(128, 1, 4, true, 0) : SG_F32_MODES(128, 1, 8, true, 2);
    else if (far) st = pairs ? SG_F32_MODES(64, 1, 4, true, 4) : SG_F32_MODES(64, 1, 8, true, 6);
    else if (head_dim == 128) st = pairs ? SG_F32_MODES(128, 1, 4, false, 8) : SG_F32_MODES(128, 1, 8, false, 10);
    else if (two_blocks) st = pairs ? SG_F32_MODES(64, 2, 4, false, 12) : SG_F32_MODES(64, 2, 8, false, 14);
    else st = pairs ? SG_F32_MODES(64, 1, 4, false, 16) : SG_F32_MODES(64, 1, 8, false, 18);
#undef SG_F32_MODES
    if (st != SG_OK) return st;
    SG_HIP_TRY(hipGetLastError());
  }
  return SG_OK;
}

}  // namespace sg
