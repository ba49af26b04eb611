// Internal declarations shared by the HIP translation units of libsupergen_tile.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "supergen_tile.h"

namespace sg {

// Records a failed HIP call for sg_last_hip_error() and maps it to SG_ERR_HIP.
int note_hip_error(hipError_t e);
#define SG_HIP_TRY(expr)                                  \
  do {                                                    \
    hipError_t sg_e_ = (expr);                            \
    if (sg_e_ != hipSuccess) return sg::note_hip_error(sg_e_); \
  } while (0)

// Shape and canvas addressing shared by the tiles of one attention call, in elements, resolved on the host.
struct TileView {
  int64_t stride_token;  // elements between canvas tokens
  int64_t stride_head;
  int32_t T, H, W;       // canvas
  int32_t th, tw;        // tile
  int32_t N;             // T*th*tw tokens
  bool window;           // tiles are windows of canvas tensors (else packed: the canvas is one unshifted tile)
};

// The tiles of one attention call.  q[i], k[i], v[i] are tile i's packed tensors or, for windows, the canvas
// tensors, and (y0[i], x0[i]) is then the canvas position of tile i's first token.
struct AttnBatch {
  int n_tiles;
  const void* const* q;      // host arrays of n_tiles device pointers
  const void* const* k;
  const void* const* v;
  void* const* out;          // packed tile outputs
  const int32_t* y0;         // host arrays, windows only (else nullptr)
  const int32_t* x0;
  const uint8_t* run_flags;  // device, n_tiles bytes: tiles with a 0 are skipped; nullptr = all tiles run
  // Cache refresh of the tiled step, carried out by the same launch where the kernel supports it (*refreshed is
  // then set): for every tile that runs, refresh_dst[i] <- its packed input (Q, K and V of all heads; k[i] and v[i] lie as far
  // behind q[i] as their copies behind refresh_dst[i]) and has_cache[i] <- 1.  All nullptr when no refresh is asked for.
  void* const* refresh_dst;  // host array of n_tiles device pointers
  uint8_t* has_cache;        // device, n_tiles bytes
  bool* refreshed;           // host, out
};

// Launchers (each validates nothing: the API layer has already done so).
int launch_attention_f32(const TileView& tv, int heads, int head_dim, float scale, const AttnBatch& b, hipStream_t s);
int launch_attention_bf16(const TileView& tv, int heads, int head_dim, float scale, const AttnBatch& b, hipStream_t s);
int launch_attention_bf16_short(const TileView& tv, int heads, float scale, const AttnBatch& b, hipStream_t s);   // head_dim 64, windows
int launch_blend(const sg_problem& p, const void* const* tile_out, void* grid_out, const void* latent, float c_latent,
                 float c_noise, hipStream_t s);
int launch_slice(const sg_problem& p, const void* const* src, int n_src, const int* tiles, void* const* dst, int n_tiles,
                 hipStream_t s);
int launch_gate(const void* const* x_cur, const void* const* x_cached, const uint8_t* has_cache,
                int n_tiles, int64_t elems, int dtype, float threshold, float* scores,
                uint8_t* recompute, void* ws, hipStream_t s);
int launch_gain_gate(const void* const* x_cur, const void* const* x_prev, const sg_gain_state& gs, int n_tiles,
                     int64_t elems, int dtype, float threshold, const float* tile_thresholds, float* step_change,
                     float* scores, uint8_t* recompute, void* ws, hipStream_t s);
int launch_gain_refresh(void* const* out_cur, const void* const* out_prev, const void* const* latent,
                        float* const* delta, const uint8_t* recompute, const float* step_change,
                        const sg_gain_state& gs, int n_tiles, int64_t elems, int dtype, void* ws, hipStream_t s);
int launch_tile_std(const void* const* x, int n_tiles, int64_t elems, int dtype, float* tile_std, void* ws, hipStream_t s);
int launch_similarity(const void* const* x_new, const void* const* x_old, int n_tiles, int64_t elems, int dtype,
                      float* l1_rel, float* cos_sim, void* ws, hipStream_t s);
int launch_region_thresholds(const float* tile_std, double* track_mean, int32_t* track_count, int n_tiles,
                             float tau_base, float alpha, int mode, int adjust, float* sigma, float* thresholds,
                             hipStream_t s);
int launch_cache_refresh(const void* const* src, void* const* dst, const uint8_t* recompute,
                         uint8_t* has_cache, int n_tiles, int64_t bytes_per_tile, hipStream_t s);

// Gate scratch: per tile kGateSlots (num, den) fp64 pairs, one per wavefront of the partial-sum kernel.
constexpr int kGateSlots = 1024;
inline size_t gate_workspace_bytes(int n_tiles) {
  return (size_t)(n_tiles > 0 ? n_tiles : 1) * kGateSlots * 2 * sizeof(double);
}

// Grid of the streaming passes over tiles (x: workgroups that share a tile, y: tiles side by side).  Large tiles: one resident
// workgroup per compute unit walks the tiles one after the other, y = 1 (no tail of late workgroups).  A tile with less than
// `vecs` 16-byte vectors for each of those is instead cut into workgroups of that many and all tiles run side by side: walked
// in turn, every small tile costs each workgroup a round trip to memory and a reduction with nothing beside it.
// kPassVecs, the passes that only read.  Measured, walked -> cut (gate, similarity, tile statistics, us a call): 20 tiles of
// 1 MiB 30, 36, 26 -> 14, 14, 12; 9 of 4 MiB 22, 36, 29 -> 16, 17, 12; 9 of 8 MiB 32, 33, 48 -> 27, 27, 16; from 16 MiB (4,096
// vectors for each of 256 compute units) the two are within 2 %.  2,048 vectors leave 8 MiB walked, 16 - 200 % slower.
// kRefreshVecs, the gain refresh, which writes as much as it reads: 20 tiles of 1 MiB 42 -> 22; of 4 MiB 73 -> 69; from
// 8 MiB walked (130; cut into workgroups of 4,096 135).
// In a cut tile a thread takes up to 16 vectors where a walked small tile gave it one: it hands the sums of every vector to fp64
// (PassSum), so that no sum in fp32 is longer than 8 elements; in walked tiles, 16 MiB and larger, it keeps them in fp32 and hands
// over once (fp64 for every vector slows the statistics of such tiles by a sixth: one wavefront per SIMD, nothing beside it).
// Error of cosine and standard deviation against fp64, bf16 tiles of 1 MiB: 4.5e-8 and 6.5e-8 without, 1.9e-8 and 3.8e-8 with
// it, which is the rounding of the result.
template <bool CUT> struct PassSumType { typedef float type; };
template <> struct PassSumType<true> { typedef double type; };
template <bool CUT> using PassSum = typename PassSumType<CUT>::type;

constexpr int64_t kPassVecs = 4096, kRefreshVecs = 2048;
constexpr int kPassThreads = 256;
inline int pass_most(int n_cu, int max_blk) { return n_cu < 1 ? 1 : (n_cu > max_blk ? max_blk : n_cu); }
inline bool pass_cut(int64_t n_vec, int n_cu, int max_blk, int64_t vecs = kPassVecs) { return (n_vec + vecs - 1) / vecs < pass_most(n_cu, max_blk); }
// Workgroups of a tile, one of n_tiles of the call; the grid of a launch that takes n of them.  Where cutting leaves compute units
// without work, the tiles are cut further, down to `least` vectors a workgroup: us a call on one tile of 64 KiB, 1 MiB and 4 MiB, gate
// 6.5, 7.0, 8.9 -> 5.4, 7.3, 7.7, similarity 8.0, 8.5, 9.1 -> 6.2, 6.6, 8.5, gain refresh 8.7, 9.5, 12.2 -> 6.6, 8.7, 11.0; 4 tiles of
// 1 MiB 8.7, 9.1, 11.1 -> 6.7, 7.9, 9.0.  Not the tile statistics, whose threads load 16 vectors at a time: 9 tiles of 1 MiB 7.6 -> 10.2.
inline int pass_blocks(int64_t n_vec, int n_tiles, int n_cu, int max_blk, int64_t vecs = kPassVecs, int64_t least = kPassThreads) {
  const int most = pass_most(n_cu, max_blk);
  if (!pass_cut(n_vec, n_cu, max_blk, vecs)) return most;
  const int64_t cut = (n_vec + vecs - 1) / vecs, full = (n_vec + least - 1) / least;
  const int64_t share = most / n_tiles < full ? most / n_tiles : full;
  const int64_t blocks = cut > share ? cut : share;
  return blocks < 1 ? 1 : (int)blocks;
}
inline dim3 pass_grid(int blocks, int64_t n_vec, int n, int n_cu, int max_blk, int64_t vecs = kPassVecs) {
  return dim3((unsigned)blocks, pass_cut(n_vec, n_cu, max_blk, vecs) ? (unsigned)n : 1u);
}

// bf16 <-> fp32 on the device.
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t bits16) {
  return __uint_as_float(bits16 << 16);
}
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {  // round to nearest even
  __bf16 b = (__bf16)f;
  return (uint32_t)__builtin_bit_cast(unsigned short, b);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

}  // namespace sg
