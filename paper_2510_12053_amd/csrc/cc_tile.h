// Configurations and index arithmetic of the matrix-core condensation
// (prep_tile_body): shared by the kernel and the host, and free of HIP headers,
// so that a host compiler can replay it.
#pragma once
#include <stdint.h>

namespace cc {

// Segments that the dense condensation splits a row's band into where a launch
// is short of workgroups.
constexpr int SEG_MAX = 2;
constexpr int TILE_Q = 8;                    // upper blocks per band row it handles
// Configurations (index + 1; 0: none): 1, ten vertices per workgroup of eight
// waves, chunks of 64 band positions, for band widths up to TILE_RING - 64;
// 2, five vertices per workgroup of sixteen waves, chunks of 256; 3, five
// vertices per workgroup of eight waves, chunks of 128.
constexpr int TILE_N = 3;
constexpr int TILE_G[TILE_N] = {2, 1, 1};            // groups of five vertices
constexpr int TILE_CH[TILE_N] = {64, 256, 128};      // chunks of band positions
constexpr int TILE_WAVES[TILE_N] = {8, 16, 8};
constexpr int TILE_RING = 192;               // ring of the first configuration
constexpr int TILE_PAD = 1024;               // zero band rows after the last one (look-ahead reads)
// LDS ring length (positions, a multiple of the chunk, so that no refill
// wraps), nine words each; the vertices' rings are tile_stride words apart:
// 3 mod 16, so that the 15 columns a row of 16 lanes reads fall into 15
// consecutive banks (mod 16).
__host__ __device__ inline int tile_ring(int cfg, int nf, int band_w) {
  if (cfg == 1) return TILE_RING;
  const int ch = TILE_CH[cfg - 1], need = nf < ch + band_w ? nf : ch + band_w;
  return (need + ch - 1) / ch * ch;
}
__host__ __device__ inline constexpr int tile_stride(int ring) { return ring * 9 + 3; }

// First band row of segment seg of nseg (seg = nseg: past the last segment,
// not clamped to nf): whole rings, so that position p keeps its slot p mod R.
__host__ __device__ inline int tile_segment(int nf, int R, int seg, int nseg) {
  return (nf + R - 1) / R * seg / nseg * R;
}
// Basis rows (nine words a position) are copied into the ring in pieces of
// TILE_PIECE words.  First word in the row of piece k from position pos on:
constexpr int TILE_PIECE = 64;
__host__ __device__ inline uint32_t tile_piece(int pos, int k) { return (uint32_t)(pos * 9 + k * TILE_PIECE); }
// The same for a segment's first fill, which may take a whole ring from close to
// the row's end on: pieces wholly past the end hold no position that is used
// and all read the words right after it.
__host__ __device__ inline uint32_t tile_fill_piece(int pos, int k, int nf) {
  const uint32_t at = tile_piece(pos, k), end = (uint32_t)nf * 9u;
  return at < end ? at : end;
}
// Floats past a float32 dense basis: what the copies read past the end of its
// last row, a piece of the first fill or a chunk whose first position exists.
constexpr int DENSE_F32_PAD = 4096;
static_assert(DENSE_F32_PAD >= 256 * 9 + TILE_PIECE, "the widest chunk's look-ahead");

}  // namespace cc
