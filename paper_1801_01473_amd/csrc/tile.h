// Site traversal orders shared by the force-side kernels.
#pragma once

#include "common.h"

namespace lqcd {

// Half index of the i-th site visited when the (y, z) cross-section is cut
// into tiles of ty rows and tz slices and, inside a tile, x and y run
// fastest, then z, then t (the tiles come last).  Sites whose +-t, +-z and +-y
// neighbours are in the same tile are visited close together in time, so a
// neighbour that one site loads is still in L2 when the next one needs it.
// tz = 0: lexicographic (i itself).  A bijection on [0, Vh) when ty divides Ly
// and tz divides Lz.
__device__ __forceinline__ int tiled_half_index(const KGeom& g, int i, int ty, int tz) {
  if (tz == 0) return i;
  const int row = g.Lxh * ty;
  const int inrow = i % row;
  int r = i / row;
  const int zi = r % tz;
  r /= tz;
  const int t = r % g.Lt;
  const int tile = r / g.Lt;
  const int nty = g.Ly / ty;
  const int y0 = (tile % nty) * ty, z = (tile / nty) * tz + zi;
  return inrow + g.Lxh * y0 + g.sz * z + g.st * t;
}

// A z-slab depth for kernels whose threads are short-lived (every site of a
// slab's t slice in flight at once): the largest of {8, 6, 4, 3, 2} that
// divides L, else 0 (no tiling).
inline int slab_tile(int L) {
  for (int e : {8, 6, 4, 3, 2})
    if (L % e == 0 && L > e) return e;
  return 0;
}

// Thread order of the per-link kernels: a segment (a direction or a side)
// outermost, then chunks of kLinkChunk half indices in which the two halves
// of a workgroup take the same half indices of parity 0 and of parity 1.
// A link's staples and neighbours alternate between the parities, so both
// parities of a region are read while they are in the same XCD's L2.  The
// grid covers link_threads_per_segment() threads per segment; threads whose
// half index i is past Vh do nothing (the return value).
constexpr int kLinkChunk = 64;  // half the per-link workgroup (128 threads)

struct LinkThread {
  int seg, par, i;
};

__host__ __device__ inline int64_t link_threads_per_segment(int Vh) {
  return int64_t(2) * ((Vh + kLinkChunk - 1) / kLinkChunk) * kLinkChunk;
}

__device__ __forceinline__ bool link_thread(const KGeom& g, int64_t idx, LinkThread& t) {
  const int64_t per = link_threads_per_segment(g.Vh);
  t.seg = int(idx / per);
  const int64_t loc = idx % per;
  t.par = int((loc / kLinkChunk) & 1);
  t.i = int((loc / (2 * kLinkChunk)) * kLinkChunk + loc % kLinkChunk);
  return t.i < g.Vh;
}

// Thread order of the kernels whose work at a site splits into a few tasks of
// equal code (directions, planes): a workgroup takes 64 consecutive entries of
// the site order at one parity, and its waves take the tasks, so that links
// several tasks use are read once and shared through LDS; the next workgroup
// of the same XCD takes the other parity of the same entries, whose links the
// first one's staples are made of.  Task and parity are uniform over a wave.
// Lanes past Vh (`in` false) work on the first site and must not store.
struct ChunkSite {
  int par, h, lane, task;
  bool in;
};

inline unsigned chunk_blocks(int Vh) { return unsigned((Vh + 63) / 64 * 2); }

__device__ __forceinline__ ChunkSite chunk_site(const KGeom& g, int ty, int tz) {
  const int w = xcd_block(blockIdx.x, gridDim.x, 1);
  ChunkSite c;
  c.par = w & 1;
  c.lane = threadIdx.x & 63;
  c.task = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = (w >> 1) * 64 + c.lane;
  c.in = i < g.Vh;
  c.h = tiled_half_index(g, c.in ? i : 0, ty, tz);
  return c;
}

// The same with both parities of the 64 entries in one workgroup, its first
// ntask waves taking parity 0: for six tasks, whose 6 waves do not spread evenly
// over the 4 SIMDs of a CU, so that of two such workgroups that would fit by
// registers and LDS only one is ever resident (5.6 waves a CU measured).
inline unsigned chunk_pair_blocks(int Vh) { return unsigned((Vh + 63) / 64); }

__device__ __forceinline__ ChunkSite chunk_pair_site(const KGeom& g, int ntask, int ty, int tz) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  ChunkSite c;
  c.par = w >= ntask;
  c.lane = threadIdx.x & 63;
  c.task = w - c.par * ntask;
  const int i = xcd_block(blockIdx.x, gridDim.x, 1) * 64 + c.lane;
  c.in = i < g.Vh;
  c.h = tiled_half_index(g, c.in ? i : 0, ty, tz);
  return c;
}

// Tile edges for those kernels: the largest divisor of Ly up to 16 and of Lz
// up to 7.  Their sites in flight and the +-2 neighbourhood compete for 4 MB of
// L2: at 48^4 the gauge force takes 7.4 ms with 8 x 6 to 16 x 6 tiles, 7.7 ms
// with 16 x 4, 8.2 ms with whole 48 x 8 slabs.
inline int chunk_tile(int L, int most) {
  for (int e = most; e > 1; --e)
    if (L % e == 0) return e;
  return 1;
}

}  // namespace lqcd
