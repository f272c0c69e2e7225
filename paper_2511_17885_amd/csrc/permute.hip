// Token permutation by expert: histogram, prefix sums, stable scatter.  The paper leaves the
// dispatch to the framework; this build fixes the order as (expert ascending, kept position
// ascending) so that the permutation is unique and reproducible.
//
// No slot is claimed with an atomic counter (that would make the order depend on scheduling).
// A block of 256 kept positions records, per expert, a 256-bit membership mask in LDS (the
// bitwise OR is order-free); a slot's rank inside the block is the population count of the mask
// bits below its position, per-block counts are scanned in block order, and the destination row
// is expert_offset + block_base + rank.

#include "common.h"
#include "prune_dev.h"
#include "tiles.h"

namespace {

constexpr int PB = FMOE_PERM_BLOCK;
constexpr int PW = PB / 32;  // mask words per expert

// ---- P1: per-block expert masks -> in-block ranks and per-block counts.  KM slots: one or few blocks fetch the code from
// memory, so that code for slots that are not there, or a copy of it for each wavefront's pairs of words, costs more
// than what it computes (16 positions, 256 experts, sixteen slots 5.3 -> 2.6 us; 256 positions, one slot 1.84 -> 1.44).
// all (where its kept_idx is not null): every position is kept, and what the pruning would have written comes from here,
// behind the loads of the slots (a launch less in a layer that drops nothing: 5000 tokens of d 1280 247.5 -> 245.7 us, 8900 of
// d 2048 491.9 -> 490.0).
template <int KM>
__global__ __launch_bounds__(PB) void permute_count_kernel(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ kept_idx, int n_cap,
    const int32_t* __restrict__ n_dev, int E, int32_t* __restrict__ slot_rank, int32_t* __restrict__ blk_count,
    fmoe_keep_all_job all) {
  __shared__ __align__(16) uint32_t mask[FMOE_MAX_EXPERTS * PW];
  static_assert(PB == 256 && PW == 8, "a wavefront's 64 positions end with a pair of words");
  const int n = resolve_count(n_cap, n_dev);
  const int blk = blockIdx.x;
  for (int i = threadIdx.x; i < E * PW; i += PB) mask[i] = 0u;
  __syncthreads();
  const int lp = threadIdx.x;
  const int p = blk * PB + lp;
  int ex[KM];
#pragma unroll
  for (int s = 0; s < KM; ++s) ex[s] = -1;
  if (p < n) {
    const int t = kept_idx ? kept_idx[p] : p;
    // all slots' experts on their way at once: asked for where they are used, each was a memory latency of its own
#pragma unroll
    for (int s = 0; s < KM; ++s) ex[s] = topk_idx[(size_t)t * KM + s];
#pragma unroll
    for (int s = 0; s < KM; ++s) {
      if (ex[s] < 0 || ex[s] >= E) ex[s] = -1;
      else atomicOr(&mask[ex[s] * PW + (lp >> 5)], 1u << (lp & 31));
    }
  }
  if (all.kept_idx != nullptr) keep_all(all, n_cap, p, gridDim.x * PB);
  __syncthreads();
  // set bits below the position, in pairs of words: its own up to it, those before it whole
  if (p < n) {
    const int pair = __builtin_amdgcn_readfirstlane(lp >> 6);
    const uint32_t below = (1u << (lp & 31)) - 1u;
    int rank[KM];
#pragma unroll
    for (int s = 0; s < KM; ++s) {
      const uint2 w = reinterpret_cast<const uint2*>(&mask[(ex[s] >= 0 ? ex[s] : 0) * PW])[pair];
      rank[s] = (lp & 32) ? __popc(w.x) + __popc(w.y & below) : __popc(w.x & below);
    }
    for (int i = 0; i < pair; ++i) {
#pragma unroll
      for (int s = 0; s < KM; ++s) {
        const uint2 w = reinterpret_cast<const uint2*>(&mask[(ex[s] >= 0 ? ex[s] : 0) * PW])[i];
        rank[s] += __popc(w.x) + __popc(w.y);
      }
    }
#pragma unroll
    for (int s = 0; s < KM; ++s) slot_rank[(size_t)p * KM + s] = ex[s] >= 0 ? rank[s] : -1;
  }
  for (int e = threadIdx.x; e < E; e += PB) {
    int c = 0;
#pragma unroll
    for (int w = 0; w < PW; ++w) c += __popc(mask[e * PW + w]);
    blk_count[(size_t)blk * E + e] = c;
  }
}

// Exclusive scan of the E (at most 256) totals into offsets[0..E] by the block's first wavefront, four per lane.
__device__ __forceinline__ void scan_totals(const int* total, int E, int32_t* offsets) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    int c[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 4 * lane + q;
      c[q] = (i < E) ? total[i] : 0;
      sum += c[q];
    }
    const int incl = wave_scan(sum);
    int excl = incl - sum;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 4 * lane + q;
      if (i < E) offsets[i] = excl;
      excl += c[q];
    }
    if (lane == 63) offsets[E] = incl;
  }
}

// ---- P2 + P3 in one launch: every block sums the per-block counts itself (totals over all blocks, bases over
// those before it; E counts per block, from L2), scans the totals and scatters its own positions.  One more block
// writes the offsets and builds the GEMM work lists, so that neither waits for the other.  A launch less and no
// walk by a single block: inside a layer, scan + scatter -> this, 22016 tokens / 64 experts 20.7 + 5.8 -> 19.9 us;
// 4224 of 8192 tokens / 128 experts 9.7 + 5.5 -> 10.2; 2176 of 4096 / 64 6.9 + 4.8 -> 7.5; with the work lists shared
// out over the whole block (tiles.h) 11.7, 9.0 and 6.7.  (Every row's loads before the first store: 12.2 -> 12.9.)
__global__ __launch_bounds__(PB) void permute_scan_scatter_kernel(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ kept_idx, int n_cap,
    const int32_t* __restrict__ n_dev, int E, int Kmax, const int32_t* __restrict__ slot_rank,
    const int32_t* __restrict__ blk_count, int32_t* __restrict__ expert_offsets,
    int32_t* __restrict__ perm_src, int32_t* __restrict__ inv_perm, fmoe_ffn_geom geom, int build, int n_shared,
    fmoe_tile* __restrict__ tiles1, fmoe_tile* __restrict__ tiles2, int32_t* __restrict__ tile_count) {
  __shared__ int s_tot[PB], s_pre[PB], s_off[FMOE_MAX_EXPERTS + 1];
  __shared__ __align__(8) int scratch[FMOE_TILES_SCRATCH];
  const int n = resolve_count(n_cap, n_dev);
  const int nblk = (n + PB - 1) / PB;
  const int blk = blockIdx.x;
  const bool lists = blk == (int)gridDim.x - 1;   // the extra block
  if (!lists && blk >= nblk) return;
  const int tid = threadIdx.x;
  int ep = 1;
  while (ep < E) ep <<= 1;                        // experts side by side, PB/ep shares of the blocks
  const int e = tid & (ep - 1), share = tid / ep, shares = PB / ep;
  int tot = 0, pre = 0;
  if (e < E) {
    constexpr int SC = 8;                         // independent loads at a time
    for (int b0 = share; b0 < nblk; b0 += SC * shares) {
      int c[SC];
#pragma unroll
      for (int i = 0; i < SC; ++i) {
        const int b = b0 + i * shares;
        c[i] = b < nblk ? blk_count[(size_t)b * E + e] : 0;
      }
#pragma unroll
      for (int i = 0; i < SC; ++i) {
        tot += c[i];
        pre += b0 + i * shares < blk ? c[i] : 0;
      }
    }
  }
  // the block's own positions meanwhile
  const int p = blk * PB + tid;
  const bool mine = !lists && p < n;
  int ex[FMOE_MAX_TOPK], rank[FMOE_MAX_TOPK];
  if (mine) {
    const int t = kept_idx ? kept_idx[p] : p;
#pragma unroll
    for (int s = 0; s < FMOE_MAX_TOPK; ++s) {
      if (s < Kmax) {
        ex[s] = topk_idx[(size_t)t * Kmax + s];
        rank[s] = slot_rank[(size_t)p * Kmax + s];
      }
    }
  }
  s_tot[tid] = tot;
  s_pre[tid] = pre;
  __syncthreads();
  if (tid < ep) {
    for (int q = 1; q < shares; ++q) {
      tot += s_tot[q * ep + tid];
      pre += s_pre[q * ep + tid];
    }
  }
  __syncthreads();
  if (tid < ep) {
    s_tot[tid] = tot;
    s_pre[tid] = pre;
  }
  __syncthreads();
  scan_totals(s_tot, E, s_off);
  __syncthreads();
  if (lists) {
    for (int i = tid; i <= E; i += PB) expert_offsets[i] = s_off[i];
    if (build)   // fused layer path
      fmoe_build_tiles<true>(s_off, E, n_cap * Kmax, n, n_shared, geom.bm, geom.run, geom.tile_cap, geom.cols1,
                             geom.scols1, tiles1, tiles2, tile_count, scratch);
    return;
  }
  if (!mine) return;
#pragma unroll
  for (int s = 0; s < FMOE_MAX_TOPK; ++s) {
    if (s < Kmax) {
      int row = -1;
      if (ex[s] >= 0 && ex[s] < E) {
        row = s_off[ex[s]] + s_pre[ex[s]] + rank[s];
        perm_src[row] = p;
      }
      inv_perm[(size_t)p * Kmax + s] = row;
    }
  }
}

// Up to which size the joined launch is the faster one.  Every block walks all counts, a thread at least
// nblk / (256 / E rounded up to a power of two) of them, while the scan's one block walks nblk a thread whatever E is.
// Whole permutation (without work lists, ten calls in a graph), two launches after the count -> one, us:
//   experts 64, 8 slots:   8192 positions 15.4 -> 12.6, 22016 18.4 -> 14.1, 65536 27.7 -> 18.8
//   experts 128, 8 slots:  8192 15.7 -> 13.4, 22016 19.0 -> 15.9, 65536 28.7 -> 24.1; 16 slots, 65536: 40.7 -> 36.7
//   experts 256, 1 slot:   8192 9.0 -> 8.75, 16384 10.7 -> 11.1, 65536 20.9 -> 25.8
//   experts 256, 8 slots:  16384 18.0 -> 17.3, 22016 19.5 -> 19.2, 32768 21.9 -> 22.5, 65536 29.7 -> 33.9
//   experts 256, 16 slots: 32768 32.8 -> 32.2, 49152 37.3 -> 38.9
// With more than 128 experts a thread walks all blocks, and the lines cross where a position's own slots (whose
// loads the walk hides) no longer pay for it: some 40 / 100 / 150 blocks at 1 / 8 / 16 slots.
bool join_scan_scatter(int nblk, int E, int Kmax) {
  return nblk <= (E <= 128 ? 256 : 32 + 8 * Kmax);
}

// ---- P2: one block; thread e scans its expert's per-block counts (turning them into block
// bases in place), then the per-expert totals are scanned into expert_offsets.  n_cap / n_dev: the positions that
// have been counted, none if no slot is routed anywhere (Kmax == 0); rows_cap / rows_dev: those kept, which is what
// the work lists give the shared experts.
__global__ __launch_bounds__(256) void permute_scan_kernel(int n_cap, const int32_t* __restrict__ n_dev,
                                                           int E, int32_t* __restrict__ blk_count,
                                                           int32_t* __restrict__ expert_offsets,
                                                           fmoe_ffn_geom geom, int build, int n_shared,
                                                           int row_cap, int rows_cap,
                                                           const int32_t* __restrict__ rows_dev,
                                                           fmoe_tile* __restrict__ tiles1,
                                                           fmoe_tile* __restrict__ tiles2,
                                                           int32_t* __restrict__ tile_count) {
  __shared__ int total[FMOE_MAX_EXPERTS];
  __shared__ __align__(8) int scratch[FMOE_TILES_SCRATCH];
  const int n = resolve_count(n_cap, n_dev);
  const int nblk = (n + PB - 1) / PB;
  const int e = threadIdx.x;
  if (e < E) {
    // SC blocks at a time: their counts are fetched together (independent loads), then turned into
    // bases -- one memory latency per SC blocks instead of one per block
    constexpr int SC = 16;
    int running = 0;
    for (int b0 = 0; b0 < nblk; b0 += SC) {
      int c[SC];
#pragma unroll
      for (int i = 0; i < SC; ++i) c[i] = (b0 + i < nblk) ? blk_count[(size_t)(b0 + i) * E + e] : 0;
#pragma unroll
      for (int i = 0; i < SC; ++i) {
        if (b0 + i < nblk) blk_count[(size_t)(b0 + i) * E + e] = running;
        running += c[i];
      }
    }
    total[e] = running;
  }
  __syncthreads();
  scan_totals(total, E, expert_offsets);
  if (build) {   // fused layer path: the grouped-GEMM work lists come out of the same scan
    __threadfence_block();
    __syncthreads();
    fmoe_build_tiles<true>(expert_offsets, E, row_cap, resolve_count(rows_cap, rows_dev), n_shared, geom.bm,
                           geom.run, geom.tile_cap, geom.cols1, geom.scols1, tiles1, tiles2, tile_count, scratch);
  }
}

// ---- P3: scatter
__global__ __launch_bounds__(PB) void permute_scatter_kernel(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ kept_idx, int n_cap,
    const int32_t* __restrict__ n_dev, int E, int Kmax, const int32_t* __restrict__ slot_rank,
    const int32_t* __restrict__ blk_base, const int32_t* __restrict__ expert_offsets,
    int32_t* __restrict__ perm_src, int32_t* __restrict__ inv_perm) {
  const int n = resolve_count(n_cap, n_dev);
  const int blk = blockIdx.x;
  const int p = blk * PB + threadIdx.x;
  if (p >= n) return;
  const int t = kept_idx ? kept_idx[p] : p;
  for (int s = 0; s < Kmax; ++s) {
    const int e = topk_idx[(size_t)t * Kmax + s];
    int row = -1;
    if (e >= 0 && e < E) {
      row = expert_offsets[e] + blk_base[(size_t)blk * E + e] + slot_rank[(size_t)p * Kmax + s];
      perm_src[row] = p;
    }
    inv_perm[(size_t)p * Kmax + s] = row;
  }
}

template <int KM = 1>
void launch_count(int Kmax, int nblk, hipStream_t stream, const int32_t* topk_idx, const int32_t* kept_idx, int n_cap,
                  const int32_t* n_dev, int E, int32_t* slot_rank, int32_t* blk_count, const fmoe_keep_all_job& all) {
  if constexpr (KM < FMOE_MAX_TOPK) {
    if (Kmax > KM)
      return launch_count<KM + 1>(Kmax, nblk, stream, topk_idx, kept_idx, n_cap, n_dev, E, slot_rank, blk_count, all);
  }
  hipLaunchKernelGGL(permute_count_kernel<KM>, dim3(nblk), dim3(PB), 0, stream, topk_idx, kept_idx, n_cap, n_dev, E,
                     slot_rank, blk_count, all);
}

}  // namespace

int launch_permute(const fmoe_ctx* ctx, const int32_t* topk_idx, const int32_t* kept_idx, int n_cap,
                   const int32_t* n_dev, int32_t* expert_offsets, int32_t* perm_src,
                   int32_t* inv_perm, void* ws, const fmoe_ws_layout& L, bool build_tiles,
                   hipStream_t stream, const fmoe_keep_all_job* all) {
  char* base = static_cast<char*>(ws);
  int32_t* slot_rank = reinterpret_cast<int32_t*>(base + L.slot_rank);
  int32_t* blk_count = reinterpret_cast<int32_t*>(base + L.blk_count);
  const int E = ctx->cfg.n_experts, Kmax = ctx->kmax;
  const int nblk = (n_cap + PB - 1) / PB;
  if (nblk > 0 && Kmax > 0) {
    fmoe_prof_scope prof(ctx, SLOT_PERM_COUNT, stream);
    launch_count(Kmax, nblk, stream, topk_idx, kept_idx, n_cap, n_dev, E, slot_rank, blk_count,
                 all != nullptr ? *all : fmoe_keep_all_job{});
  } else if (all != nullptr) {
    const int rc = launch_identity_kept(all->is_visual, all->cu, all->B, n_cap, all->kept_idx, all->new_cu,
                                        all->is_visual_out, stream);
    if (rc != FMOE_OK) return rc;
  }
  if (nblk > 0 && Kmax > 0 && join_scan_scatter(nblk, E, Kmax)) {
    fmoe_prof_scope prof(ctx, SLOT_PERM_SCATTER, stream);
    hipLaunchKernelGGL(permute_scan_scatter_kernel, dim3(nblk + 1), dim3(PB), 0, stream, topk_idx, kept_idx,
                       n_cap, n_dev, E, Kmax, slot_rank, blk_count, expert_offsets, perm_src, inv_perm,
                       fmoe_geom(ctx, n_cap), build_tiles ? 1 : 0, ctx->cfg.n_shared,
                       reinterpret_cast<fmoe_tile*>(base + L.tiles), reinterpret_cast<fmoe_tile*>(base + L.tiles2),
                       reinterpret_cast<int32_t*>(base + L.tile_count));
    FMOE_HIP_CHECK(hipGetLastError());
    return FMOE_OK;
  }
  {
    fmoe_prof_scope prof(ctx, SLOT_PERM_SCAN, stream);
    hipLaunchKernelGGL(permute_scan_kernel, dim3(1), dim3(256), 0, stream, Kmax > 0 ? n_cap : 0,
                       Kmax > 0 ? n_dev : nullptr, E, blk_count, expert_offsets,
                       fmoe_geom(ctx, n_cap), build_tiles ? 1 : 0, ctx->cfg.n_shared,
                       n_cap * Kmax, n_cap, n_dev, reinterpret_cast<fmoe_tile*>(base + L.tiles),
                       reinterpret_cast<fmoe_tile*>(base + L.tiles2),
                       reinterpret_cast<int32_t*>(base + L.tile_count));
  }
  if (nblk > 0 && Kmax > 0) {
    fmoe_prof_scope prof(ctx, SLOT_PERM_SCATTER, stream);
    hipLaunchKernelGGL(permute_scatter_kernel, dim3(nblk), dim3(PB), 0, stream, topk_idx, kept_idx,
                       n_cap, n_dev, E, Kmax, slot_rank, blk_count, expert_offsets, perm_src,
                       inv_perm);
  }
  FMOE_HIP_CHECK(hipGetLastError());
  return FMOE_OK;
}
