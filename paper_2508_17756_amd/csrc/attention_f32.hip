// Tile attention, fp32 throughout (paper Section 2.1 "full attention" restricted to one tile), for SG_F32
// problems, on the fp32 matrix instruction (32x32x2: fp32 operands, fp32 accumulation, 64 FLOP per cycle and
// SIMD; a large fp32 matrix product reaches 154 TFLOP/s on the same device): calls of few queries, heads of 4 GiB and more, and
// queries whose tile holds numbers that the split kernel (attention_f32_split.hip), which takes the others, does not.
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
#include "attention_f32_block.h"

namespace sg {
namespace {

constexpr int kXcd = 8;

// KS wavefronts = shares of the keys; two wavefronts per SIMD either way: one workgroup of 8 per compute unit, or two of 4
// WIDE: offsets inside a head leave 32 bits
template <int D, int QB, int KS, int MODE, bool WIDE>
__global__ __launch_bounds__(64 * KS, 2) void attention_f32_kernel(
    const View16 vw, const float scale, const int heads, const int n_qblocks, const int n_tiles, const AttnTable tab,
    const uint32_t head_bytes, const uint8_t* __restrict__ run_flags) {
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
  attend_f32<D, QB, KS, MODE, WIDE>(vw, scale, tab, head_bytes, tile, head, qblk * (QB * 32), wy0, wx0, lds);
}

// Several rounds of tiles of up to 256 tokens: start and end of a round, which nothing runs beside in the split kernel, are as long as three to
// five stages, so that the rounds alone do not tell.  Times in us, fitted to both kernels' at 65 - 1,100 tokens (within 3 to 7 % in the mean
// square, 18 at most): of the split kernel a round and its stages of 32 keys (head_dim 64: 64); here, of two workgroups per compute unit, a round
// of blocks of 32 keys dealt to four shares, and of what stays on average beside it a workgroup and its blocks.  us here and on the split kernel,
// head_dim 64: 342 heads of 65 tokens 18.9 and 26.2, 769 38.2 and 52.7, 512 of 129 58.0 and 64.5, 192 of 192 34.7 and 32.1, 640 of 97 52.1 and 42.4;
// head_dim 128: 769 of 65 62.2 and 74.8, 769 of 97 97.4 and 87.8.  Where this chooses wrongly it costs up to 8 % (wrapped windows of 65 tokens x
// 128 11).  One round and longer tiles go by the rounds alone, which costs them 7 % at most.
bool split_is_faster(int tokens, int head_dim, int64_t heads, int64_t rounds, bool two_blocks, int n_cu) {
  const int blocks = (tokens + 31) / 32, dealt = (blocks + 3) / 4;
  const int64_t workgroups = heads * (two_blocks ? (tokens + 63) / 64 : blocks);
  const double full = (double)((workgroups + 2 * n_cu - 1) / (2 * n_cu)), part = (double)workgroups / (2 * n_cu);
  if (head_dim == 128) return rounds * (11.8 + 2.56 * blocks) < full * 4.1 * dealt + part * (5.9 + blocks) + 6.0;
  const double split = rounds * (8.0 + 2.65 * ((blocks + 1) / 2)) + 1.0;
  return split < (two_blocks ? full * 7.3 * dealt + part * (6.1 + 3.1 * dealt) + 7.0 : full * 2.6 * dealt + part * (3.2 + 0.43 * blocks) + 4.0);
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
    // The split kernel owns 128 queries per workgroup, one workgroup per compute unit, and takes 2.4 times as long for them as this one
    // for 32 (see there): taken where the rounds over the device say so, however many of the tiles the gate lets run.
    bool split = !far;
    for (int a = b.run_flags ? 1 : n; a <= n && split; ++a) {
      const int64_t big = ((int64_t)a * heads * ((tv.N + 127) / 128) + n_cu - 1) / n_cu, small = ((int64_t)a * heads * ((tv.N + 31) / 32) + n_cu - 1) / n_cu;
      split = 12 * big < 5 * small && (big == 1 || tv.N > 256 || split_is_faster(tv.N, head_dim, (int64_t)a * heads, big, two_blocks, n_cu));
    }
    int st;
#define SG_F32_MODES(D, QB, KS, WIDE, SLOT)                                                        \
  (tv.window ? launch(attention_f32_kernel<D, QB, KS, kWindow, WIDE>, KS, kBlockLds<QB, KS>, SLOT)      \
             : launch(attention_f32_kernel<D, QB, KS, kLinear, WIDE>, KS, kBlockLds<QB, KS>, SLOT + 1))
    if (split) st = launch_attention_f32_split(vw, tv.window, heads, head_dim, scale, n, tab, (uint32_t)(head_units * 32), flags, dev, s);
    else if (far && head_dim == 128) st = pairs ? SG_F32_MODES(128, 1, 4, true, 0) : SG_F32_MODES(128, 1, 8, true, 2);
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
