// The deal of the dense expert-GEMM shape: which work item a workgroup takes.  Integers only, so that a host program
// can walk a whole launch.
#pragma once

#if defined(__HIPCC__)
#define FMOE_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define FMOE_HOST_DEVICE inline
#endif

// Work items of the dense shape.  The items of a list (entries in order, each entry's column groups) are cut into
// eight contiguous shares, one per XCD (consecutive workgroups go round the XCDs), separately for the entries of
// groups with several row tiles, the first n_several of the list, and for the single tiles behind them; a share
// of each is walked by one XCD, evenly mixed.
//  * Contiguous: a group of several row tiles sits on one XCD, or two where a cut falls into it, and every XCD has as
//    much to do.  What the down GEMM reads past L2 fell by it (4096 tokens, 64 experts of 1408: 15 % less; 8192, 128 of
//    768: 31 %).  Gate/up reads 10 % less at the latter, but 3 % more at the former and 11 % more with hundreds of rows
//    per expert, since its items wait for each other less and walk the reduction out of step: there the gain
//    in time is the balance.
//  * Mixed: groups of many rows keep the matrix pipes busy, single tiles the memory; one kind after the other left
//    the pipes idle in the second half.
//  * Inside a run the items go down the row tiles in strips of DENSE_STRIP column groups: neighbours in time
//    share an activation tile or a weight tile while it still is in L2.
//  * The weights of a single tile are not asked for again and bypass the L2's recency order (non-temporal), if the
//    layer's weights are more than the memory-side cache (256 MB) keeps for the next call: non-temporal loads miss that
//    too.  Layer after layer, or 440 MB and more of weights, with / without the hint: 1600 tokens, d 1280, 64 experts of
//    896 115.5 / 121.2 us, 4096 tokens, d 2048, 64 experts of 1408 347 / 356.  One layer over and over, very uneven rows:
//    1200 tokens, d 1288, 16 experts of 904 and a shared one (119 MB) 94 / 78, 1600 tokens, d 4096, 8 experts of 1536 (302 MB) 156 / 138.
//    The line is drawn between, at one and a half times the cache.
// Measured, gate/up and down us, entries dealt round-robin before: 4096 tokens d 2048 64 experts of 1408, half kept
// 193 + 106 -> 177 + 103; the same size, nothing dropped and every token six experts 270 + 158 -> 243 + 140;
// 8192 tokens, 128 experts of 768 160 + 97 -> 149 + 90; 22016 tokens, six experts 1526 + 883 -> 1493 + 864.  Strips of
// one or two groups and runs of 8 or 16 row tiles: within 1 % of this, one group 1 % slower at 22016 tokens.
constexpr int DENSE_STRIP = 3;
// Up to so many items, a round and a half of two workgroups a CU, the launch takes as long as its fullest XCD: entries go
// round the XCDs, long and short ones alike, and a run's items in strips of one column group, so that a weight
// tile enters one or two L2s (layer of 1600 tokens, d 1280, 64 experts of 896, half kept: 118.1 -> 114.9 us).
// Contiguous shares / entry by entry, us, gate/up and down; below the line: 1920 tokens of that layer 51/48 and 38/35;
// 1440 tokens, d 2048, 32 experts of 1024, half kept 66/62 and 40/37; 1066 tokens, 64 experts of 1408, half kept 119/115
// and 63/56; 960 tokens, d 1024, 72 of 768, all kept 38/36 and 22/22; above it: 2666 tokens, 64 of 1408, half kept 137/145
// and 81/84, all kept 245/251 and 142/149; 4000 tokens, 128 of 768, half kept 100/107 and 63/63, all kept 204/221 and
// 127/143; 3200 tokens of the first layer, all kept 123/125 and 80/84.
constexpr int DENSE_ONE_ROUND = 768;

// workgroups of a launch whose list has at most tile_cap entries (an XCD's share of either kind rounds up)
FMOE_HOST_DEVICE unsigned dense_blocks(int tile_cap, int cols) { return (((unsigned)tile_cap + 7) / 8 * cols + 2) * 8; }

FMOE_HOST_DEVICE int eighth(int n, int x) { return (n >> 3) * x + (((n & 7) * x) >> 3); }   // n*x/8

// list entry of workgroup `block` in a list of n entries of `cols` column groups, -1: none; its column group; whether
// the entry counts as a single tile; columns per strip
FMOE_HOST_DEVICE int dense_entry(int block, int n, int n_several, int cols, int& group, bool& single, int& strip) {
  const int xcd = block & 7, b = block >> 3;
  if (n * cols <= DENSE_ONE_ROUND) {
    const int batch = b / cols, e = batch * 8 + xcd;
    group = b - batch * cols;
    single = e >= n_several;
    strip = 1;
    return e < n ? e : -1;
  }
  strip = DENSE_STRIP;
  const int i0 = n_several * cols, i1 = (n - n_several) * cols;   // items of the two kinds
  const int f0 = eighth(i0, xcd), nf = eighth(i0, xcd + 1) - f0;
  const int s0 = eighth(i1, xcd), ns = eighth(i1, xcd + 1) - s0;
  if (b >= nf + ns) return -1;
  int done = b < nf ? 0 : b - nf;   // single-tile items ahead of item b of this XCD
  single = b >= nf;
  if (nf + ns < 32768) {            // (beyond, where the products would overflow: one kind after the other)
    done = b * ns / (nf + ns);
    single = (b + 1) * ns / (nf + ns) > done;
  }
  const int item = single ? i0 + s0 + done : f0 + (b - done);
  const int e = item / cols;
  group = item - e * cols;
  return e;
}

// Item `group` of row tile rt of a run of nrt row tiles with c_eff column groups -> the row tile and column group it
// is in the run's order (strips of `strip` column groups, each down the row tiles).
FMOE_HOST_DEVICE void dense_run_order(int rt, int nrt, int c_eff, int strip, int& row_tile, int& group) {
  const int w = rt * c_eff + group;
  const int s = w / (strip * nrt), in_strip = w - s * (strip * nrt);
  const int left = c_eff - s * strip;
  const int width = left < strip ? left : strip;
  row_tile = in_strip / width;
  group = s * strip + (in_strip - row_tile * width);
}
