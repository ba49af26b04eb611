// Shared by the tile-attention kernels (paper Sections 2.1 and 3; Algorithm 1 "SliceTile" / "Shift"):
// the table of tiles one launch works on, the mapping of workgroups to (tile, head, query block) that skips
// reused tiles on the device, and the addressing of a tile's tokens inside a canvas tensor.
#pragma once
#include "sg_common.h"

namespace sg {

// vector types of the bf16 matrix-core kernels
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
#define SG_LDS __attribute__((address_space(3)))

// 16 bytes per lane from global memory straight into LDS: lane i fills bytes [16 i, 16 i + 16) of the
// 1 KiB block at LDS byte address `lds_dst` (wave-uniform).  Address = sbase + voff (32-bit byte offset), or
// a 64-bit address per lane.
// Inline assembly keeps the compiler from ordering later LDS reads behind the transfer; completion is
// awaited explicitly on vmcnt.  The statements overwrite m0 and say so.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is a reserved register; naming it as clobbered is the point
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_dst), "v"(voff), "s"(sbase) : "memory", "m0");
}
__device__ __forceinline__ void dma16_addr(const void* addr, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_dst), "v"(addr) : "memory", "m0");
}
#pragma clang diagnostic pop

// ---------------------------------------------------------------------------------------------------
// One launch attends up to kAttnTilesPerLaunch tiles of the same shape (Algorithm 1: for all tiles of the
// partition).  Per tile the table holds the tensors its offsets are relative to (packed tile or canvas), the packed
// output and, for a window of a canvas, the canvas position of its first token.
constexpr int kAttnTilesPerLaunch = 32;
struct AttnTable {
  const void* q[kAttnTilesPerLaunch];
  const void* k[kAttnTilesPerLaunch];
  const void* v[kAttnTilesPerLaunch];
  void* out[kAttnTilesPerLaunch];
  int32_t y0[kAttnTilesPerLaunch], x0[kAttnTilesPerLaunch];   // windows only
  void* refresh[kAttnTilesPerLaunch];   // cache refresh fused into the launch (packed tiles): copy of the tile's input, or unused
};

// Tiles whose run flag is 0 (the cache gate reuses them) are skipped on the device: the workgroups number
// only the work of the active tiles, so that work is spread evenly whichever tiles run, and the rest of the
// grid exits at once.  Returns the 32-bit mask of active tiles among the launch's n_tiles.
__device__ __forceinline__ uint32_t attn_active_mask(const uint8_t* __restrict__ run_flags, int n_tiles) {
  const int lane = threadIdx.x & 63;
  if (!run_flags) return n_tiles >= 32 ? 0xffffffffu : ((1u << n_tiles) - 1u);
  const bool on = lane < n_tiles && run_flags[lane] != 0;
  return (uint32_t)__ballot(on);
}
// index of the a-th set bit of mask (a < popcount(mask))
__device__ __forceinline__ int attn_nth_tile(uint32_t mask, int a) {
  for (int i = 0; i < a; ++i) mask &= mask - 1;
  return __builtin_ctz(mask);
}

// ---------------------------------------------------------------------------------------------------
// Tile addressing on the device, in units of 8 elements (16 bytes of bf16, 32 of fp32), so that offsets inside one
// head fit 32 bits.  A packed tile (a canvas that is one unshifted tile) is walked linearly; any other tile is a window of
// a canvas tensor: token (t, i, j) sits at canvas row (y0 + i) mod H, column (x0 + j) mod W, where (y0, x0) is the
// canvas position of its first token (Algorithm 1 "SliceTile"; "Shift" lets it wrap around the edges).
// Divisions by the tile's width and plane are multiplications: n / d = ((n * mul) >> 32 >> shift) + (n & all) for 0 <= n < 2^31.
struct Divisor {
  uint32_t mul, shift, all;
};
struct View16 {
  uint32_t st16;     // units per canvas token
  uint32_t head16;   // units per head
  int32_t th, tw, N;
  int32_t H, W;      // canvas size
  Divisor by_plane, by_row;   // th * tw, tw
  uint32_t reach;    // kReach* bits
};
constexpr uint32_t kReachLane = 1;   // 16 tokens span less than 4 GiB (16-byte units)
constexpr uint32_t kReachHead = 2;   // so does a whole head

__device__ __forceinline__ uint32_t divide(uint32_t n, const Divisor d) { return (__umulhi(n, d.mul) >> d.shift) + (n & d.all); }

struct WindowToken {
  uint32_t off16;   // offset from the canvas tensor's head
  int32_t x0j, j;   // x0 + column before wrapping, column inside the tile
};
__device__ __forceinline__ WindowToken window_token(const View16& vw, int n, int y0, int x0) {
  const int t = (int)divide((uint32_t)n, vw.by_plane);
  const int r = n - t * (vw.th * vw.tw);
  const int i = (int)divide((uint32_t)r, vw.by_row);
  WindowToken k;
  k.j = r - i * vw.tw;
  k.x0j = x0 + k.j;
  int y = y0 + i, x = k.x0j;
  y -= (y >= vw.H) ? vw.H : 0;
  x -= (x >= vw.W) ? vw.W : 0;
  k.off16 = (uint32_t)((t * vw.H + y) * vw.W + x) * vw.st16;
  return k;
}

// Host side: the divisor of 0 <= n < 2^31 by d >= 1.  With l = ceil(log2 d) the rounded-up reciprocal
// floor(2^(31+l) / d) + 1 is below 2^32 and exact for 31-bit dividends (Granlund and Montgomery, 1994).
inline Divisor make_divisor(uint32_t d) {
  if (d <= 1) return {0u, 0u, 0xffffffffu};
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  return {(uint32_t)((1ull << (31 + l)) / d + 1), l - 1, 0u};
}
inline View16 make_view16(const TileView& tv) {
  View16 vw;
  vw.st16 = (uint32_t)(tv.stride_token / 8);
  vw.head16 = (uint32_t)(tv.stride_head / 8);
  vw.th = tv.th; vw.tw = tv.tw; vw.N = tv.N;
  vw.H = tv.H; vw.W = tv.W;
  vw.by_plane = make_divisor((uint32_t)tv.th * (uint32_t)tv.tw);
  vw.by_row = make_divisor((uint32_t)tv.tw);
  vw.reach = (tv.stride_token / 8 < (1 << 23) ? kReachLane : 0u) |
             ((int64_t)tv.T * tv.H * tv.W * (tv.stride_token / 8) < (1ll << 28) ? kReachHead : 0u);
  return vw;
}

}  // namespace sg
