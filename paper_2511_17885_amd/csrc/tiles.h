// Device-side construction of the grouped-GEMM work lists, shared by the permutation scan (fused
// layer path) and the stand-alone expert-FFN entry point.
#pragma once

#include "common.h"

#define FMOE_TILES_SCRATCH 768

#if defined(__HIPCC__)
// Builds, with one block of 256 threads or a multiple, the two row-tile lists of the expert FFN (`bm` rows per tile):
//   list 1 (gate/up GEMM): the dense shared-expert group (group id E, all n kept tokens, hidden
//     dimension = the N_s experts concatenated) first, then the routed experts;
//   list 2 (down GEMM): one dense group per shared expert (group id E+s) first, then the routed
//     experts.
// Long items go first: the shared groups (every kept token), then the routed experts by
// descending row count (ties: ascending expert id), so that the short tiles are the ones left to
// fill the tail of the launch.  A launch gives every entry `cols1` column tiles; the shared group
// of list 1 may have more (`scols1`): its row tiles are then repeated with a column-tile offset in
// `col0`.  The row tiles of one group (one replica) are consecutive entries, cut into runs of at most
// `run` row tiles (rt / nrt number a tile within its run): a run is the unit within which
// the GEMM kernels order their workgroups.
// counts[0], counts[1] = number of entries in list 1 / list 2; counts[2], counts[3] = how many of them, the first
// ones, belong to groups of several row tiles.  Experts whose offsets are malformed
// (negative, decreasing or past row_cap) are skipped so that no tile can index outside the row
// buffers; without room for rows (row_cap 0) the offsets are not read and may be null.  `scratch` is
// FMOE_TILES_SCRATCH ints of LDS (8-byte aligned); bm and run are powers of two.
template <bool SPLIT>
__device__ __forceinline__ void fmoe_build_tiles(const int32_t* expert_offsets, int E, int row_cap,
                                                 int n, int n_shared, int bm, int run, int tile_cap, int cols1,
                                                 int scols1, fmoe_tile* tiles1, fmoe_tile* tiles2,
                                                 int32_t* counts, int* scratch) {
  const int sh = 31 - __clz(bm);   // bm is a power of two
  // the experts side by side, as often as the block holds them: every share takes its part of an expert's tiles and, with
  // SPLIT, of the comparisons (64 experts, 256 threads, some 1000 tiles at 20000 tokens: the joined scan and scatter,
  // whose longest block this is, 12.3 -> 8.1 us).  Alone in a launch, or for a handful of tokens, it does not split: the
  // code comes from memory, and the additions and the barrier behind them take longer than the comparisons they
  // save (8 experts 1.84 -> 1.56 us, 256 experts 6.40 -> 6.16)
  const int le = E > 1 ? 32 - __clz(E - 1) : 0;
  const int e = threadIdx.x & ((1 << le) - 1), share = threadIdx.x >> le, shares = blockDim.x >> le;
  int* const s_start = scratch + 512;   // of every expert
  int r0 = 0, cnt = 0;
  if (e < E && row_cap > 0) {
    r0 = expert_offsets[e];
    const int r1 = expert_offsets[e + 1];
    cnt = r1 - r0;
    if (r0 < 0 || cnt < 0 || r1 > row_cap) cnt = 0;
  }
  const int nt = (cnt + bm - 1) >> sh;
  __syncthreads();
  // order key: more rows first, then the lower expert id (rows < 2^24, ids < 2^8)
  const unsigned key = ((unsigned)cnt << 8) | (unsigned)(255 - e);
  if (share == 0) {
    scratch[2 * e] = (e < E) ? (int)key : 0;
    scratch[2 * e + 1] = nt;
    if constexpr (SPLIT) s_start[e] = 0;
  }
  __syncthreads();
  // first tile slot of expert e = tiles of all experts ahead of it in that order
  int start = 0;
  {
    const int per = !SPLIT ? E : ((1 << le) > 8 * shares ? (1 << le) / shares : 8);
    const int o0 = SPLIT ? share * per : 0, o1 = o0 + per < E ? o0 + per : E;
#pragma unroll 8
    for (int o = o0; o < o1; ++o) {
      const int2 kn = *reinterpret_cast<const int2*>(&scratch[2 * o]);
      start += ((unsigned)kn.x > key) ? kn.y : 0;
    }
  }
  if constexpr (SPLIT) {
    if (start) atomicAdd(&s_start[e], start);
    __syncthreads();
    start = s_start[e];
  }

  const int ns = (n_shared > 0) ? (n + bm - 1) / bm : 0;
  const int rep1 = (ns > 0 && cols1 > 0) ? (scols1 + cols1 - 1) / cols1 : 0;
  const int sh1 = ns * rep1, sh2 = ns * n_shared;
  for (int j = threadIdx.x; j < ns; j += blockDim.x) {
    fmoe_tile t;
    t.rt = j & (run - 1);
    t.nrt = (ns - (j - t.rt) < run) ? (ns - (j - t.rt)) : run;
    t.row0 = (j - t.rt) * bm;
    t.rows = n - t.row0;
    t.group = E;
    for (int c = 0; c < rep1; ++c) {   // replica-major: the row tiles of one replica are consecutive
      const int slot = c * ns + j;
      if (slot >= tile_cap) break;
      t.col0 = c * cols1;
      tiles1[slot] = t;
    }
    t.col0 = 0;
    for (int s = 0; s < n_shared; ++s) {
      const int slot = s * ns + j;
      if (slot >= tile_cap) break;
      t.group = E + s;
      tiles2[slot] = t;
    }
  }
  if (e < E) {
    for (int j = share; j < nt; j += shares) {
      fmoe_tile t;
      t.group = e;
      t.col0 = 0;
      t.rt = j & (run - 1);
      t.nrt = (nt - (j - t.rt) < run) ? (nt - (j - t.rt)) : run;
      t.row0 = r0 + (j - t.rt) * bm;
      t.rows = cnt - (j - t.rt) * bm;
      if (sh1 + start + j < tile_cap) tiles1[sh1 + start + j] = t;
      if (sh2 + start + j < tile_cap) tiles2[sh2 + start + j] = t;
    }
  }
  if (threadIdx.x >= blockDim.x - 64) {   // the last wavefront, which has the fewest tiles to write
    const int lane = threadIdx.x & 63;
    int all = 0, more = 0;   // entries of the routed experts, of those with several tiles
    for (int o = lane; o < E; o += 64) {
      const int v = scratch[2 * o + 1];
      all += v;
      more += v > 1 ? v : 0;
    }
    const int routed = wave_scan(all), several = wave_scan(more);
    if (lane == 63) {
      const int t1 = routed + sh1, t2 = routed + sh2;
      counts[0] = t1 < tile_cap ? t1 : tile_cap;
      counts[1] = t2 < tile_cap ? t2 : tile_cap;
      const int s1 = several + (ns > 1 ? sh1 : 0), s2 = several + (ns > 1 ? sh2 : 0);
      counts[2] = s1 < tile_cap ? s1 : tile_cap;
      counts[3] = s2 < tile_cap ? s2 : tile_cap;
    }
  }
}
#endif
