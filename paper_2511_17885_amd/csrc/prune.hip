// Routing-aware sliding-window pruning of visual tokens (paper Sec. 3.2): per-sequence visual
// ordinals, window similarity scores (Eq.8-10), attention term (Eq.11-13), budget, drop
// selection and compaction.
//
// The kept-token set is a decision, so every float here follows the same fixed-order fp32
// arithmetic as the router (compiled with contraction off): a dot product over the E routing
// probabilities is taken with one partial per lane (element e in lane e mod 64, ascending e,
// fmaf from +0) and the 6-level xor butterfly; means, cosines and the window average are plain
// sequential fp32 operations in window order; '/' and sqrtf are correctly rounded.
//
// Indexing trick: window i of sequence b lives at slot cu_seqlens[b] + i (a sequence has fewer
// windows than tokens), so no per-sequence window offsets have to be scanned; a slot finds its
// sequence by binary search over cu_seqlens.

#include "common.h"
#include "prune_dev.h"
#include "tiles.h"

namespace {

// v of the lane `ROT` places on in the row of 16
template <int ROT>
__device__ __forceinline__ float row_rotate(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + ROT, 0xf, 0xf, false));
}
// The xor butterfly 32, 16, 8, 4, 2, 1 without the LDS crossbar: the halves and the rows of 16 are exchanged by lane
// swaps (a swap of v with itself leaves v of the lower partner in one result and of the upper one in the other),
// and once the values repeat every 8 lanes, a rotation inside the row pairs what the exclusive-or would.
// (Eleven sums one after the other per window of five: 7936 tokens, 128 experts 11.0 -> 10.2 us; 48 tokens 4.9 -> 4.2.)
__device__ __forceinline__ float wave_sum_butterfly(float p) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(p), false, false);
  p = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(p), false, false);
  p = __uint_as_float(q[0]) + __uint_as_float(q[1]);
  p = p + row_rotate<8>(p);
  p = p + row_rotate<4>(p);
  p = p + row_rotate<2>(p);
  return p + row_rotate<1>(p);
}

__device__ __forceinline__ uint32_t wave_or(uint32_t v) {   // over all lanes, in every lane
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  v = h[0] | h[1];
  const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = q[0] | q[1];
  v |= __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, false);
  return v | __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, false);
}

// ---- A: visual ordinals.  One block per sequence.
// vis_ord[t] = number of visual tokens before t in its sequence, as ~(that number) < 0 for text;
// vis_tok[cu[b] + j] = global index of the j-th visual token of sequence b; seq_nv[b] = N_v.
__global__ __launch_bounds__(256) void seq_ordinals_kernel(
    const uint8_t* __restrict__ is_visual, const int32_t* __restrict__ cu, int T,
    int32_t* __restrict__ vis_ord, int32_t* __restrict__ vis_tok, int32_t* __restrict__ seq_nv) {
  __shared__ int wave_tot[4 * ORD_ROWS];
  seq_ordinals_block(is_visual, cu, blockIdx.x, T, vis_ord, vis_tok, seq_nv, wave_tot);
}

// ---- B: window scores.  One wavefront per window; lanes <-> experts.
// win_s[g] = S_i (Eq.10 or Eq.8), win_a[g] = raw window attention sum (Eq.11) if attn, g = the window's slot.
// Launch over window units: sequence b owns the units cu[b]/W + b ... (it has at most
// floor(cu[b+1]/W) - floor(cu[b]/W) + 1 windows, so consecutive sequences never overlap and
// floor(T/W) + B units cover every window); a unit finds its sequence by binary search.
// STAGED: the wavefront copies the window's routing-probability rows into its own LDS tile once (coalesced
// row reads) and both passes over the window -- the mean row, then the cosines (Eq.9-10), or all pairs
// (Eq.8) -- read the tile; a lane only ever reads back the columns it stored itself, so no
// synchronisation is involved.  Windows whose rows do not fit the tile (W*E > WS_TILE) take the
// instantiation that re-reads global memory.  The arithmetic and its order are the same either way.
constexpr int WS_TILE = 2048;   // floats of LDS per wavefront
__device__ __forceinline__ int unit_base(const int32_t* cu, int b, int T, int W) {
  return clampi(cu[b], 0, T) / W + b;
}
template <bool STAGED>
__global__ __launch_bounds__(256) void window_score_kernel(
    const float* __restrict__ probs, const int32_t* __restrict__ cu, int B, int T, int E, int W,
    int sim_mode, const int32_t* __restrict__ vis_tok, const int32_t* __restrict__ seq_nv,
    const float* __restrict__ attn, float* __restrict__ win_s, float* __restrict__ win_a) {
  __shared__ float tile_all[STAGED ? 4 * WS_TILE : 1];
  const int lane = threadIdx.x & 63;
  const int u = blockIdx.x * 4 + (threadIdx.x >> 6);
  int lo = 0, hi = B - 1;   // largest b with unit_base(b) <= u
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (unit_base(cu, mid, T, W) <= u) lo = mid; else hi = mid - 1;
  }
  const int b = lo;
  int s, e;
  seq_range(cu, b, T, s, e);
  const int i = u - unit_base(cu, b, T, W);
  int nv = seq_nv[b];
  nv = nv < e - s ? nv : e - s;                 // a sequence has no more visual tokens than tokens
  if (i < 0 || (long long)i * W >= nv) return;  // not a window of this sequence
  const int g = s + i;                          // < s + nv <= T
  const int first = i * W;
  const int w = __builtin_amdgcn_readfirstlane((nv - first < W) ? (nv - first) : W);
  const int32_t* toks = vis_tok + s + first;

  // One load for all rows (w <= 64).  The token ids are read across the lanes, so that from here on every loop and
  // branch is uniform: all lanes stay on, those without an expert take the last one's column and add nothing.
  const int tok = toks[lane < w ? lane : w - 1];
  if (attn != nullptr) {
    const float mine = attn[tok];
    float a = 0.0f;
    for (int j = 0; j < w; ++j) a = a + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), j));
    if (lane == 0) win_a[g] = a;
  }
  if (w == 1) {
    if (lane == 0) win_s[g] = 1.0f;
    return;
  }
  float* tile = tile_all + (STAGED ? (threadIdx.x >> 6) * WS_TILE : 0);
  if (STAGED) {
    // eight rows at a time: one after the other, index and row, each was two memory latencies (7936 tokens in
    // windows of five, 128 experts 10.6 -> 6.9 us; 1536 in windows of three, 64 experts 5.2 -> 4.9)
    for (int e0 = 0; e0 < E; e0 += 64) {
      const int ex = e0 + lane < E ? e0 + lane : E - 1;
      for (int j0 = 0; j0 < w; j0 += 8) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {   // (past the window the last row again)
          const int j = j0 + q < w ? j0 + q : w - 1;
          v[q] = probs[(size_t)__builtin_amdgcn_readlane(tok, j) * E + ex];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) tile[(j0 + q < w ? j0 + q : w - 1) * E + ex] = v[q];
      }
    }
  }
  // element ex of the window's row j, 0 past the experts
  auto row = [&](int j, int ex) -> float {
    const int e = ex < E ? ex : E - 1;
    const float v = STAGED ? tile[j * E + e] : probs[(size_t)__builtin_amdgcn_readlane(tok, j) * E + e];
    return ex < E ? v : 0.0f;
  };
  float S;
  if (sim_mode == 0) {
    // Eq.9: mean row (sequential over the window, one divide), Eq.10: mean cosine to it
    float mean[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ex = lane + 64 * r;
      float acc = 0.0f;
      if (64 * r < E) {
        acc = row(0, ex);
        for (int j = 1; j < w; ++j) acc = acc + row(j, ex);
        acc = acc / (float)w;
      }
      mean[r] = acc;
    }
    float pm = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (64 * r < E) pm = fmaf(mean[r], mean[r], pm);
    const float norm_mean = sqrtf(wave_sum_butterfly(pm));
    float acc = 0.0f;
    for (int j = 0; j < w; ++j) {
      float pd = 0.0f, pn = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ex = lane + 64 * r;
        if (64 * r < E) {
          const float v = row(j, ex);
          pd = fmaf(v, mean[r], pd);
          pn = fmaf(v, v, pn);
        }
      }
      const float dot = wave_sum_butterfly(pd);
      const float nrm = sqrtf(wave_sum_butterfly(pn));
      const float c = dot / (nrm * norm_mean);
      acc = acc + c;
    }
    S = acc / (float)w;
  } else {
    // Eq.8: mean cosine over all pairs q < j
    float acc = 0.0f;
    for (int j = 1; j < w; ++j) {
      float rj[4];
      float pn = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ex = lane + 64 * r;
        rj[r] = 64 * r < E ? row(j, ex) : 0.0f;
        if (64 * r < E) pn = fmaf(rj[r], rj[r], pn);
      }
      const float nj = sqrtf(wave_sum_butterfly(pn));
      for (int q = 0; q < j; ++q) {
        float pd = 0.0f, pq = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ex = lane + 64 * r;
          if (64 * r < E) {
            const float v = row(q, ex);
            pd = fmaf(rj[r], v, pd);
            pq = fmaf(v, v, pq);
          }
        }
        const float dot = wave_sum_butterfly(pd);
        const float nq = sqrtf(wave_sum_butterfly(pq));
        const float c = dot / (nj * nq);
        acc = acc + c;
      }
    }
    S = acc / (float)(w * (w - 1) / 2);
  }
  if (lane == 0) win_s[g] = S;
}

// ---- C: drop order, merged set, budget and compaction in one launch over blocks of CP_BLOCK positions.
// The drop order (normalised attention asc, score desc, index asc) and the merge order (score desc, index asc) are
// total, and of the places in them only two matters: where merging ends and where the drop budget ends.  So nobody
// ranks the windows: every block finds, for the sequences that its positions belong to, those two windows by a radix
// selection over integer keys, after which a window's fate is one comparison, and counts what is dropped ahead of its
// first position; sequences before that have dropped exactly their budget.  Blocks need nothing from each other.
// Bound: latency, a dozen barriers between LDS passes over a few keys a thread; the uniform arithmetic is paid once per
// wavefront of a SIMD, hence 512 threads and not 1024 (12.6 -> 8.9 us inside the kernel at 4096 tokens; 256: 9.6).
// In place of counting all pairs of windows, deciding, flagging and writing (three launches, five with merging and
// attention), average kernel times: 4096 tokens, 1280 windows 17.0 -> 10.4 us; 8192 tokens, 1588 windows 17.5 -> 9.8; three
// ragged sequences of 5003 tokens, one of them short, 15.0 -> 9.8; eight of 22016 24.4 -> 10.1; 1600 tokens, merging and
// attention 24.8 -> 14.0.
// Without attention both orders are one: the two windows are found together.  fmoe_prune of one sequence of 7000 tokens in
// windows of two, merging: two searches 35.7 us, one 32.8, three launches 32.7.
// A block takes the sequences that it touches one after the other, so in batches of up to CP_CUT_SEQS sequences no block
// has positions of two: its place is looked up first, in one load of a wavefront.  fmoe_prune in us, three to five
// launches / blocks of CP_BLOCK positions throughout / ending with their sequence: 7000 tokens in three sequences, windows
// of two, 22.4 / 22.6 / 20.1, with merging 31.7 / 38.5 / 31.8, with attention 25.1 / 26.9 / 23.0; in sixteen 23.0 / 25.2 /
// 16.6, 32.2 / 44.9 / 28.0, 25.1 / 30.7 / 18.6; 1000 tokens in eight 22.6 / 24.6 / 14.7, 30.1 / 43.7 / 22.2, 25.9 / 29.5 / 15.3.
// Larger batches gain more from the one launch than that costs (4000 tokens in 64 sequences 36.1 -> 20.7, 12000 in 150
// 43.1 -> 22.8).
// Sequences of up to CP_WAVE_N windows are decided by a wavefront each (lane = window, ranks by counting), so that a
// block with many short ones does not walk them one barrier at a time.
constexpr int CP_BLOCK = 512;
constexpr int CP_WAVES = CP_BLOCK / 64;
constexpr int CP_KEYS = 4096;     // windows of a sequence whose keys stay in LDS; those past it are formed again
constexpr int CP_WAVE_N = 64;     // windows of a sequence that one wavefront decides
constexpr int CP_RANK = 8;        // candidates of a selection that are ranked by counting
constexpr int CP_SEQS = 512;      // sequences whose bounds stay in LDS
constexpr int CP_CUT_SEQS = 62;   // sequences of a batch whose blocks end with them: with what lies ahead and behind a lane each

struct CompactArgs {
  const uint8_t* is_visual;
  const int32_t* cu;
  int B, T, W;
  float retention, gamma, alpha;
  const int32_t* vis_ord;
  const int32_t* seq_nv;
  const float* win_s;
  const float* win_a;             // nullptr without attention importance
  float* scores_out;              // or nullptr
  int32_t* kept_idx;
  int32_t* new_cu;
  uint8_t* is_visual_out;         // or nullptr
  uint8_t* is_merged_out;         // or nullptr
  unsigned long long window_rcp;  // ceil(2^37 / W)
  bool cut;                       // blocks end where a sequence ends (B <= CP_CUT_SEQS)
};
// v / W, exactly: W <= 64 and 0 <= v < 2^24, so the error of the product is below 2^24 in 2^37, less than 1 / W
__device__ __forceinline__ int per_window(const CompactArgs& a, int v) {
  return (int)(((unsigned long long)(uint32_t)v * a.window_rcp) >> 37);
}

// Sort key of a window: attention (0 without), then score; ascending = drop order.  The score alone, ascending = merge
// order.  Ties by index.
struct fmoe_window_key {
  uint32_t att, sc;
  __device__ __forceinline__ unsigned long long both() const { return (unsigned long long)att << 32 | sc; }
};
__device__ __forceinline__ bool key_before(fmoe_window_key a, int i, fmoe_window_key b, int j) {
  return (int)(a.both() < b.both()) | ((int)(a.both() == b.both()) & (int)(i < j));   // without branches
}

// What becomes of the windows of a sequence (uniform).
struct fmoe_window_cut {
  int n_full;                // windows of W tokens; one more if the last is shorter
  int last_merged, last_keeps;
  uint32_t merge_sc;         // of the full ones, merged: those ahead of this one in the merge order
  int merge_i;
  fmoe_window_key drop_key;  // of the others, dropped: those ahead of this one in the drop order, and the last `part` tokens
  int drop_i, part;          // of this one
  __device__ __forceinline__ bool merged(int i, fmoe_window_key K) const {
    const bool m = (int)(K.sc < merge_sc) | ((int)(K.sc == merge_sc) & (int)(i < merge_i));
    return i < n_full ? m : last_merged != 0;
  }
  __device__ __forceinline__ int lead(int i, fmoe_window_key K, int W) const {   // leading tokens of an unmerged one that stay
    const int l = i == drop_i ? W - part : (key_before(K, i, drop_key, drop_i) ? 0 : W);
    return i < n_full ? l : last_keeps;
  }
};
constexpr int CP_ALL = 0x7fffffff;   // index of a cut behind all windows (with the largest key), -1 of one ahead of all (with 0)

// The drop walk over the unmerged windows with a budget of u tokens: q full windows go whole and `part` tokens of the
// next; a shorter last window that takes part in it (`last`) has its turn behind `ahead` full ones.
__device__ __forceinline__ void drop_walk(const CompactArgs& a, int u, bool last, int w_last, int ahead, int& q, int& part,
                                          int& last_keeps) {
  q = per_window(a, u);
  part = u - q * a.W;
  last_keeps = w_last;
  if (last && q >= ahead) {
    const int v = u - ahead * a.W, rest = v < w_last ? 0 : v - w_last, more = per_window(a, rest);
    last_keeps = v < w_last ? w_last - v : 0;
    q = ahead + more;
    part = rest - more * a.W;
  }
}

template <bool MERGE, bool ATTN>
__global__ __launch_bounds__(CP_BLOCK) void compact_kernel(CompactArgs a) {
  __shared__ uint32_t s_sc[CP_KEYS], s_att[ATTN ? CP_KEYS : 1];
  __shared__ unsigned long long s_red[2][CP_WAVES];
  constexpr int NT = MERGE && !ATTN ? 2 : 1;   // windows that one search finds
  constexpr int TABLE = NT * 256;
  __shared__ __align__(16) int hist[3 * TABLE];
  // fates of the short sequences' windows, leading tokens that stay or ~0 for merged: of the sequence that the block
  // begins inside at i, of one that starts at position s at CP_WAVE_N + s - p0 + i (a sequence has no more windows
  // than tokens, so they don't overlap)
  __shared__ int s_fate[CP_WAVE_N + CP_BLOCK + CP_WAVE_N];
  __shared__ int s_few[CP_BLOCK], s_many[CP_BLOCK / CP_WAVE_N + 2];
  __shared__ int s_count[2 + NT], s_first;   // sequences in the two lists, candidates; dropped of the first sequence before p0
  __shared__ uint32_t s_cand_att[NT * CP_RANK], s_cand_sc[NT * CP_RANK];
  __shared__ int s_cand[NT * CP_RANK];
  __shared__ int s_cu[CP_SEQS + 1], s_nv[CP_SEQS], s_ahead[CP_WAVES];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = a.T, W = a.W, B = a.B;
  int p0 = blockIdx.x * CP_BLOCK, p1 = p0 + CP_BLOCK < T ? p0 + CP_BLOCK : T;
  if (a.cut) {   // lane = part of the batch: ahead of the sequences, each of them, behind them; a block's is the last to begin by it
    const int begin = lane == 0 ? 0 : clampi(a.cu[lane <= B + 1 ? lane - 1 : B], 0, T);
    const int first = begin / CP_BLOCK + lane;   // block; ascending in a partition (of bounds that decrease nothing below is used)
    const int j = __popcll(__ballot(lane <= B + 1 && first <= (int)blockIdx.x)) - 1;
    p0 = __builtin_amdgcn_readlane(begin, j) + ((int)blockIdx.x - __builtin_amdgcn_readlane(first, j)) * CP_BLOCK;
    const int end = j == B + 1 ? T : __builtin_amdgcn_readlane(begin, j + 1);
    p1 = p0 + CP_BLOCK < end ? p0 + CP_BLOCK : end;
  }
  const int t = p0 + tid, tc = t < T ? (t < 0 ? 0 : t) : T - 1;
  const float one_minus_alpha = 1.0f - a.alpha;
  if (tid < 2 + NT) s_count[tid] = 0;
  if (tid == 2 + NT) s_first = 0;
  __syncthreads();   // (while the first loads are on their way)

  // ---- the sequences: which of them have windows and positions in this block, what those before it have dropped
  const int ord = a.vis_ord[tc], ord_p0 = a.vis_ord[clampi(p0, 0, T - 1)];   // (meaningless outside the sequences)
  const uint8_t vis = a.is_visual_out != nullptr ? a.is_visual[tc] : 0;
  const bool cached = B <= CP_SEQS;
  bool bad = false;
  int gone = 0;
  for (int b = tid; b < B; b += CP_BLOCK) {
    const int s = clampi(a.cu[b], 0, T), e = clampi(a.cu[b + 1], 0, T), nv = clampi(a.seq_nv[b], 0, e - s);
    bad |= e < s;
    if (e <= p0) {
      gone += nv - token_budget(nv, a.retention);
    } else if (s < p1 && p0 < p1 && nv > 0) {
      if (nv > W * CP_WAVE_N) {
        const int at = atomicAdd(&s_count[1], 1);   // (a bound that decreases could make them more than there is room for)
        if (at < CP_BLOCK / CP_WAVE_N + 2) s_many[at] = b;
      } else {
        const int at = atomicAdd(&s_count[0], 1);
        if (at < CP_BLOCK) s_few[at] = b;
      }
    }
    if (cached) {
      s_cu[b] = s;
      s_nv[b] = nv;
      if (b == B - 1) s_cu[B] = e;
    }
  }
  gone = wave_scan(gone);
  const bool wave_bad = __ballot(bad) != 0ull;
  if (lane == 63) s_red[0][wave] = (unsigned long long)(uint32_t)gone | (wave_bad ? 1ull << 63 : 0ull);
  __syncthreads();
  unsigned long long before_block = 0;
#pragma unroll
  for (int w = 0; w < CP_WAVES; ++w) {
    before_block += s_red[0][w] & ~(1ull << 63);
    bad |= (s_red[0][w] >> 63) != 0;
  }
  if (__builtin_expect(bad, 0)) {   // uniform: bounds that decrease are no partition into sequences; nothing is pruned
    const int own = blockIdx.x * CP_BLOCK + tid;
    if (own < T) {
      a.kept_idx[own] = own;
      if (a.is_visual_out != nullptr) a.is_visual_out[own] = a.is_visual[own];
      if (a.is_merged_out != nullptr) a.is_merged_out[own] = 0;
    }
    for (int b = own; b <= B; b += gridDim.x * CP_BLOCK) a.new_cu[b] = clampi(a.cu[b], 0, T);
    return;
  }
  if (p0 >= p1 && blockIdx.x + 1 != gridDim.x) return;   // uniform: no positions, and the bounds are the last block's
  const int32_t* cu = cached ? s_cu : a.cu;
  const int32_t* seq_nv = cached ? s_nv : a.seq_nv;
  auto visual_tokens = [&](int b) {
    int s, e;
    seq_range(cu, b, T, s, e);
    return clampi(seq_nv[b], 0, e - s);
  };
  // sums over the block: two sets of slots in turn, one barrier
  int phase = 1;
  auto block_sum = [&](int v) -> int {
    v = wave_scan(v);
    if (lane == 63) s_red[phase][wave] = (unsigned long long)(uint32_t)v;
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < CP_WAVES; ++w) total += (int)(uint32_t)s_red[phase][w];
    phase ^= 1;
    return total;
  };
  int bits = t < p1 ? 1 : 0;   // bit 0: the token stays, bit 1: a merged window collapses into it
  const int n_few = s_count[0], n_many = s_count[1];
  // visual tokens of the sequence from s on ahead of p0
  auto ahead_of_block = [&](int s) { return s < p0 ? (ord_p0 >= 0 ? ord_p0 : ~ord_p0) : 0; };
  auto key_from = [&](float ws, float wa, float amax) {
    float A;
    const float c = redundancy_score(ws, ATTN, wa, amax, a.alpha, one_minus_alpha, A);
    return fmoe_window_key{ATTN ? float_order_key(A) : 0u, ~float_order_key(c)};
  };
  auto write_score = [&](int g, float ws, float wa, float amax) {
    float A;
    a.scores_out[g] = redundancy_score(ws, ATTN, wa, amax, a.alpha, one_minus_alpha, A);
  };

  // ---- sequences of more than CP_WAVE_N windows, one after the other over the whole block
  for (int k = 0; k < n_many; ++k) {   // uniform
    const int b = __builtin_amdgcn_readfirstlane(s_many[k]);
    const int s = __builtin_amdgcn_readfirstlane(clampi(cu[b], 0, T)), nv = __builtin_amdgcn_readfirstlane(visual_tokens(b));
    const int n = per_window(a, nv + W - 1);
    const int w_last = nv - (n - 1) * W, o0 = ahead_of_block(s);
    auto win_a = [&](int i) { return ATTN ? a.win_a[s + i] : 0.0f; };
    float amax = 0.0f;
    if constexpr (ATTN) {   // per-sequence attention maximum (Eq.12)
      for (int i = tid; i < n; i += CP_BLOCK) {
        const float v = a.win_a[s + i];
        amax = v > amax ? v : amax;
      }
#pragma unroll
      for (int sh = 32; sh >= 1; sh >>= 1) {
        const float o = __shfl_xor(amax, sh, 64);
        amax = o > amax ? o : amax;
      }
      if (lane == 0) s_red[phase][wave] = __float_as_uint(amax);
      __syncthreads();
#pragma unroll
      for (int w = 0; w < CP_WAVES; ++w) {
        const float o = __uint_as_float((uint32_t)s_red[phase][w]);
        amax = o > amax ? o : amax;
      }
      phase ^= 1;
    }
    auto key_of = [&](int i) { return key_from(a.win_s[s + i], win_a(i), amax); };
    const fmoe_window_key K_first = key_of(0), K_last = key_of(n - 1);
    uint32_t diff_sc = 0, diff_att = 0;   // bits in which the keys are not all alike
    int ahead_of_last = 0;                // windows ahead of the last one in the merge order, without merging in the drop order
    auto take_in = [&](int i, fmoe_window_key K) {
      diff_sc |= K.sc ^ K_first.sc;
      diff_att |= K.att ^ K_first.att;
      ahead_of_last += (int)(i < n - 1) & (int)(MERGE ? K.sc <= K_last.sc : K.both() <= K_last.both());
    };
    for (int i0 = 0; i0 < n && i0 < CP_KEYS; i0 += 4 * CP_BLOCK) {   // four loads at a time (past the end the last window)
      fmoe_window_key K[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + r * CP_BLOCK + tid;
        K[r] = key_of(i < n ? i : n - 1);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s_sc[i0 + r * CP_BLOCK + tid] = K[r].sc;
        if (ATTN) s_att[i0 + r * CP_BLOCK + tid] = K[r].att;
        take_in(i0 + r * CP_BLOCK + tid, K[r]);
      }
    }
    static_assert(CP_KEYS % (4 * CP_BLOCK) == 0, "whole rounds of keys");
    for (int i = CP_KEYS + tid; i < n; i += CP_BLOCK) take_in(i, key_of(i));
    diff_sc = wave_or(diff_sc);
    if (ATTN) diff_att = wave_or(diff_att);
    ahead_of_last = wave_scan(ahead_of_last);
    if (lane == 63) {
      s_red[phase][wave] = (unsigned long long)diff_att << 32 | diff_sc;
      s_ahead[wave] = ahead_of_last;
    }
    ahead_of_last = 0;
    for (int h = tid; h < TABLE; h += CP_BLOCK) hist[h] = 0;
    fmoe_window_cut cut{};
    const int n_full = w_last < W ? n - 1 : n;
    cut.n_full = n_full;
    const int eps = nv - token_budget(nv, a.retention);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < CP_WAVES; ++w) {
      diff_sc |= (uint32_t)s_red[phase][w];
      if (ATTN) diff_att |= (uint32_t)(s_red[phase][w] >> 32);
      ahead_of_last += s_ahead[w];
    }
    phase ^= 1;
    // this thread's windows, and up to the end of a round some past the last; their keys are its own
    auto each = [&](auto f) {
      for (int i0 = 0; i0 < n && i0 < CP_KEYS; i0 += 4 * CP_BLOCK) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = i0 + r * CP_BLOCK + tid;
          const fmoe_window_key K{ATTN ? s_att[i] : 0u, s_sc[i]};
          f(i, K);
        }
      }
#pragma unroll 1
      for (int i = CP_KEYS + tid; i < n; i += CP_BLOCK) f(i, key_of(i));
    };
    fmoe_merge_plan p{0, 0, eps};
    if constexpr (MERGE) p = merge_plan(nv, W, a.retention, a.gamma, n_full < n ? ahead_of_last : n);
    cut.last_merged = p.last_m;
    cut.last_keeps = w_last;
    const int index_bits = 32 - __clz(n);
    // The windows at `place` of the drop order (by_att: with the attention keys) among the candidates: digits of eight bits of
    // the attention key, then of the score's, then of the index, each from the highest bit on that is not the same in all,
    // until the candidates are few enough to rank.  Counts of the candidates per digit are summed by every wavefront for
    // itself; a barrier a digit, the tables take turns.  Two windows of one order share a table until their digits part.
    auto find = [&](bool by_att, int (&place)[NT], const bool (&wanted)[NT], auto candidate, fmoe_window_key (&found)[NT],
                    int (&found_i)[NT]) {
      struct { int level, fixed; uint32_t chosen, tied_sc, tied_att, att_counts, sc_counts; bool open; } st[NT];
      bool shared = NT == 2;
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        const int level = by_att && diff_att != 0 ? 0 : (diff_sc != 0 ? 1 : 2);
        st[q].level = level;
        st[q].chosen = level == 0 ? K_first.att : (level == 1 ? K_first.sc : 0u);
        st[q].fixed = level == 2 ? index_bits : 32 - __clz(level == 0 ? diff_att : diff_sc);   // bits from here on are those of `chosen`
        // what the levels before have settled (the keys' common attention, if it takes part in the order at all)
        st[q].tied_att = K_first.att;
        st[q].tied_sc = K_first.sc;
        st[q].att_counts = by_att && level > 0 ? ~0u : 0u;
        st[q].sc_counts = level == 2 ? ~0u : 0u;
        st[q].open = wanted[q];
        shared = shared && wanted[q];
      }
      int table = 0;
      for (;;) {   // uniform; ends because indices differ
        int* const h = hist + table * TABLE;
        table = table == 2 ? 0 : table + 1;
        for (int z = tid; z < TABLE; z += CP_BLOCK) hist[table * TABLE + z] = 0;
        auto live_digit = [&](int q, int i, fmoe_window_key K, uint32_t& digit) {
          const int shift = st[q].fixed > 8 ? st[q].fixed - 8 : 0;
          const uint32_t v = st[q].level == 1 ? K.sc : (st[q].level == 0 ? K.att : (uint32_t)i);
          digit = (v >> shift) & 255u;
          const uint32_t off = ((K.att ^ st[q].tied_att) & st[q].att_counts) | ((K.sc ^ st[q].tied_sc) & st[q].sc_counts) |
                               (st[q].fixed < 32 ? (v ^ st[q].chosen) >> st[q].fixed : 0u);
          return (int)(off == 0u) & candidate(i, K);
        };
        each([&](int i, fmoe_window_key K) {
#pragma unroll
          for (int q = 0; q < NT; ++q) {
            uint32_t digit;
            if (st[q].open && !(q == 1 && shared) && live_digit(q, i, K, digit)) atomicAdd(&h[q * 256 + digit], 1);
          }
        });
        __syncthreads();
        uint32_t digits[NT];
        int4 c4{};
        int sum4 = 0, excl = 0;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
          digits[q] = 0;
          if (!st[q].open) continue;   // uniform
          if (q == 0 || !shared) {     // uniform
            c4 = *reinterpret_cast<const int4*>(&h[q * 256 + 4 * lane]);
            sum4 = c4.x + c4.y + c4.z + c4.w;
            excl = wave_scan(sum4) - sum4;
          }
          const int src = __builtin_ctzll(__ballot(excl <= place[q] && place[q] < excl + sum4));   // exactly one lane
          int before = excl, val = 4 * lane, here = c4.x;
          if (before + here <= place[q]) { before += here; here = c4.y; ++val; }
          if (val > 4 * lane && before + here <= place[q]) { before += here; here = c4.z; ++val; }
          if (val > 4 * lane + 1 && before + here <= place[q]) { before += here; here = c4.w; ++val; }
          place[q] -= __builtin_amdgcn_readlane(before, src);
          digits[q] = (uint32_t)__builtin_amdgcn_readlane(val, src);
          here = __builtin_amdgcn_readlane(here, src);
          if (here <= CP_RANK) {
            each([&](int i, fmoe_window_key K) {
              uint32_t digit;
              if (live_digit(q, i, K, digit) & (int)(digit == digits[q])) {
                const int at = q * CP_RANK + atomicAdd(&s_count[2 + q], 1);
                if (ATTN) s_cand_att[at] = K.att;
                s_cand_sc[at] = K.sc;
                s_cand[at] = i;
              }
            });
            st[q].open = false;
            continue;
          }
          const int shift = st[q].fixed > 8 ? st[q].fixed - 8 : 0;
          const uint32_t mask = (0xffu << shift) & (st[q].fixed < 32 ? (1u << st[q].fixed) - 1u : ~0u);
          st[q].chosen = (st[q].chosen & ~mask) | ((digits[q] << shift) & mask);
          st[q].fixed = shift;
          if (shift == 0) {   // alike so far: by what comes next
            if (st[q].level == 0) {
              st[q].tied_att = st[q].chosen;
              st[q].att_counts = ~0u;
            } else {
              st[q].tied_sc = st[q].chosen;
              st[q].sc_counts = ~0u;
            }
            st[q].level = st[q].level == 0 && diff_sc != 0 ? 1 : 2;
            st[q].chosen = st[q].level == 1 ? K_first.sc : 0u;
            st[q].fixed = st[q].level == 1 ? 32 - __clz(diff_sc) : index_bits;
          }
        }
        bool open = false;
#pragma unroll
        for (int q = 0; q < NT; ++q) open |= st[q].open;
        if (!open) break;
        if (NT == 2) shared = shared && digits[0] == digits[NT - 1];
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        if (!wanted[q]) continue;   // uniform
        const int here = s_count[2 + q], mine = q * CP_RANK + (lane < here ? lane : 0);
        const fmoe_window_key K{ATTN ? s_cand_att[mine] : 0u, s_cand_sc[mine]};
        const int i = s_cand[mine];
        int rank = 0;
#pragma unroll 4
        for (int j = 0; j < here; ++j) {   // uniform
          const fmoe_window_key o{by_att ? (uint32_t)__builtin_amdgcn_readlane(K.att, j) : 0u,
                                  (uint32_t)__builtin_amdgcn_readlane(K.sc, j)};
          rank += (int)key_before(o, __builtin_amdgcn_readlane(i, j), fmoe_window_key{by_att ? K.att : 0u, K.sc}, i);
        }
        const int src = __builtin_ctzll(__ballot(lane < here && rank == place[q]));   // exactly one
        found[q] = fmoe_window_key{ATTN ? (uint32_t)__builtin_amdgcn_readlane(K.att, src) : 0u,
                                   (uint32_t)__builtin_amdgcn_readlane(K.sc, src)};
        found_i[q] = __builtin_amdgcn_readlane(i, src);
      }
    };
    // where merging ends: the full window at place q_full of the merge order
    const bool find_merge = MERGE && p.q_full > 0 && p.q_full < n_full;
    if constexpr (MERGE) {
      cut.merge_sc = p.q_full == 0 ? 0u : ~0u;
      cut.merge_i = p.q_full == 0 ? -1 : CP_ALL;
    }
    if constexpr (MERGE && ATTN) {
      if (find_merge) {   // uniform; a search of its own, the drop order is another one
        int place[NT] = {p.q_full}, i[NT];
        const bool wanted[NT] = {true};
        fmoe_window_key found[NT];
        find(false, place, wanted, [&](int w, fmoe_window_key) { return (int)(w < n_full); }, found, i);
        cut.merge_sc = found[0].sc;
        cut.merge_i = i[0];
        for (int z = tid; z < TABLE; z += CP_BLOCK) hist[z] = 0;   // for the next search
        __syncthreads();   // all have read the number of candidates
        if (tid == 0) s_count[2] = 0;
      }
    }
    // where the budget ends: of the full windows that are not merged, the one at place q of the drop order
    {
      const bool last = n_full < n && !p.last_m;
      int ahead = 0, q, place[NT], i[NT];
      if (last) {   // uniform
        if constexpr (MERGE && ATTN) {
          int v = 0;
          each([&](int w, fmoe_window_key K) { v += (int)(w < n_full) & (int)!cut.merged(w, K) & (int)(K.both() <= K_last.both()); });
          ahead = block_sum(v);
        } else {   // one order, in which the merged ones come first
          ahead = ahead_of_last > p.q_full ? ahead_of_last - p.q_full : 0;
        }
      }
      drop_walk(a, p.u_rem, last, w_last, ahead, q, cut.part, cut.last_keeps);
      const bool none = q == 0 && cut.part == 0, find_drop = !none && q < n_full - p.q_full;
      cut.drop_key = none ? fmoe_window_key{0u, 0u} : fmoe_window_key{ATTN ? ~0u : 0u, ~0u};
      cut.drop_i = none ? -1 : CP_ALL;
      bool wanted[NT];
      wanted[NT - 1] = find_drop;
      place[NT - 1] = NT == 2 ? p.q_full + q : q;
      if constexpr (NT == 2) {
        wanted[0] = find_merge;
        place[0] = p.q_full;
      }
      if (find_drop || (NT == 2 && find_merge)) {   // uniform
        fmoe_window_key found[NT];
        find(ATTN, place, wanted,
             [&](int w, fmoe_window_key K) { return (int)(w < n_full) & (int)!(MERGE && ATTN && cut.merged(w, K)); }, found, i);
        if (find_drop) {
          cut.drop_key = found[NT - 1];
          cut.drop_i = i[NT - 1];
        }
        if (NT == 2 && find_merge) {
          cut.merge_sc = found[0].sc;
          cut.merge_i = i[0];
        }
      }
    }
    if (ord >= 0 && ord < nv && t >= s && t < clampi(cu[b + 1], 0, T)) {
      const int i = per_window(a, ord);
      const fmoe_window_key K = i < CP_KEYS ? fmoe_window_key{ATTN ? s_att[i] : 0u, s_sc[i]} : key_of(i);   // (barriers behind the writers)
      const int in_win = ord - i * W;
      if (MERGE && cut.merged(i, K)) bits = in_win == 0 ? 3 : 0;
      else bits = in_win < cut.lead(i, K, W) ? 1 : 0;
    }
    if (a.scores_out != nullptr && t >= s && t < s + n) write_score(t, a.win_s[t], win_a(t - s), amax);
    if (s < p0) {   // uniform: what is dropped of it ahead of this block
      const int i0 = per_window(a, o0), j0 = o0 - i0 * W;
      int v = 0;
      each([&](int i, fmoe_window_key K) {
        const int lead = cut.lead(i, K, W), stays = MERGE && cut.merged(i, K) ? 1 : lead;
        const int size = i < i0 ? (i < n_full ? W : w_last) : (i == i0 ? j0 : 0);
        v += size > stays ? size - stays : 0;
      });
      v = block_sum(v);
      if (tid == 0) s_first = v;
    }
    __syncthreads();   // keys, candidates and their number are read no more
    if (tid < NT) s_count[2 + tid] = 0;   // (the next use is behind another barrier)
  }

  // ---- the others, a wavefront each (lane = window)
  if (__builtin_expect(n_few > 0, 0)) {   // uniform
    for (int k = wave; k < n_few; k += CP_WAVES) {   // uniform over the wavefront
      const int b = __builtin_amdgcn_readfirstlane(s_few[k]);
      const int s = clampi(cu[b], 0, T), nv = visual_tokens(b), n = per_window(a, nv + W - 1);
      const int w_last = nv - (n - 1) * W, n_full = w_last < W ? n - 1 : n;
      const int i = lane < n ? lane : n - 1;   // lanes past the windows repeat the last one and are not counted
      const float ws = a.win_s[s + i], wa = ATTN ? a.win_a[s + i] : 0.0f;
      float amax = wa > 0.0f ? wa : 0.0f;
      if constexpr (ATTN) {
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) {
          const float o = __shfl_xor(amax, sh, 64);
          amax = o > amax ? o : amax;
        }
      }
      const fmoe_window_key K = key_from(ws, wa, amax);
      auto key_at = [&](int j) {
        return fmoe_window_key{ATTN ? (uint32_t)__builtin_amdgcn_readlane(K.att, j) : 0u, (uint32_t)__builtin_amdgcn_readlane(K.sc, j)};
      };
      const fmoe_window_key K_last = key_at(n - 1);
      const bool full = lane < n_full;
      fmoe_merge_plan p{0, 0, nv - token_budget(nv, a.retention)};
      bool merged = false;
      int place = 0;
      if constexpr (MERGE) {
        const int L = n_full < n ? __popcll(__ballot(full && K.sc <= K_last.sc)) : n;
        p = merge_plan(nv, W, a.retention, a.gamma, L);
#pragma unroll 4
        for (int j = 0; j < n_full; ++j) {
          const uint32_t o = __builtin_amdgcn_readlane(K.sc, j);
          place += (int)(o < K.sc) | ((int)(o == K.sc) & (int)(j < lane));
        }
        merged = full ? place < p.q_full : p.last_m != 0;
      }
      const bool takes_part = full && !merged;
      const unsigned long long part_mask = __ballot(takes_part);
      const int ahead = __popcll(__ballot(takes_part && K.both() <= K_last.both()));
      int q, part, last_keeps;
      drop_walk(a, p.u_rem, n_full < n && !p.last_m, w_last, ahead, q, part, last_keeps);
      if constexpr (MERGE && !ATTN) {
        place -= p.q_full;   // one order, in which the merged ones come first
      } else {
        place = 0;
#pragma unroll 4
        for (int j = 0; j < n_full; ++j) {
          place += (int)key_before(key_at(j), j, K, lane) & (int)((part_mask >> j) & 1);
        }
      }
      const int lead = full ? (place < q ? 0 : (place == q ? W - part : W)) : last_keeps;
      if (lane < n) {
        s_fate[(s < p0 ? 0 : CP_WAVE_N + s - p0) + lane] = merged ? ~0 : lead;
        const int g = s + lane;
        if (a.scores_out != nullptr && g >= p0 && g < p1) write_score(g, ws, wa, amax);
      }
      if (s < p0) {   // uniform: what is dropped of it ahead of this block
        const int o0 = ahead_of_block(s), i0 = per_window(a, o0), j0 = o0 - i0 * W;
        const int stays = merged ? 1 : lead, size = full ? W : w_last;
        int v = 0;
        if (lane < n) v = lane < i0 ? size - stays : (lane == i0 && j0 > stays ? j0 - stays : 0);
        v = wave_scan(v);
        if (lane == 63) s_first = v;
      }
    }
    __syncthreads();
    if (ord >= 0 && t < p1 && t >= clampi(cu[0], 0, T) && t < clampi(cu[B], 0, T)) {
      const int b = find_seq(cu, B, t), s = clampi(cu[b], 0, T), nv = visual_tokens(b);
      if (ord < nv && nv <= W * CP_WAVE_N) {
        const int i = per_window(a, ord), fate = s_fate[(s < p0 ? 0 : CP_WAVE_N + s - p0) + i];
        const int in_win = ord - i * W;
        bits = fate < 0 ? (in_win == 0 ? 3 : 0) : (in_win < fate ? 1 : 0);
      }
    }
  }

  // ---- positions of the kept tokens
  const unsigned long long kept = __ballot(bits & 1);
  if (lane == 0) s_red[phase][wave] = (unsigned long long)__popcll(kept);
  __syncthreads();
  int pos = p0 - (int)before_block - s_first + __popcll(kept & ((1ull << lane) - 1ull));
#pragma unroll
  for (int w = 0; w < CP_WAVES; ++w) pos += w < wave ? (int)s_red[phase][w] : 0;
  phase ^= 1;
  if ((bits & 1) && pos >= 0 && pos < T) {   // pos <= t by construction
    a.kept_idx[pos] = t;
    if (a.is_visual_out != nullptr) a.is_visual_out[pos] = vis;
    if (a.is_merged_out != nullptr) a.is_merged_out[pos] = (bits >> 1) & 1;
  }
  if (blockIdx.x == gridDim.x - 1) {   // sequence bounds of the kept tokens
    int before = 0;
    for (int b0 = 0; b0 <= B; b0 += CP_BLOCK) {   // uniform
      const int b = b0 + tid;
      int v = 0;
      if (b < B) {   // a sequence loses its budget exactly
        const int nv = visual_tokens(b);
        v = nv - token_budget(nv, a.retention);
      }
      const int incl = wave_scan(v);
      if (lane == 63) s_red[phase][wave] = (unsigned long long)(uint32_t)incl;
      __syncthreads();
      int mine = before + incl - v;
#pragma unroll
      for (int w = 0; w < CP_WAVES; ++w) {
        const int c = (int)(uint32_t)s_red[phase][w];
        mine += w < wave ? c : 0;
        before += c;
      }
      phase ^= 1;
      if (b <= B) a.new_cu[b] = clampi(cu[b], 0, T) - mine;
    }
  }
}

// ---- D2: the layer input after merging (Eq.16-18).  One block per kept position: an ordinary token's
// row is copied, 16 bytes a thread; a merged token becomes the mean of its window's rows, rescaled to the
// largest row norm of the window.  The few merged rows are computed in fp64 with one rounding to the storage
// type, so that the routing decisions taken on them afterwards see the correctly rounded token; a thread
// keeps the columns' sums in registers between the norm and the store (columns past MG_COLS * 256 are summed
// a second time), and the row norms share one block reduction, since it is the chain of reductions and row
// reads that a merged row costs.  1216 kept rows of d 1280, 57 merged: 13.6 -> 10.4 us; 4250 of d 2048: 23.9 ->
// 15.6 (element copies, three passes over a window and a reduction per row before).
constexpr int MG_COLS = 8;
constexpr int MG_ROWS = 4;    // rows of the window whose norms are reduced together
template <int NV>
__device__ __forceinline__ void block_sums_f64(double (&v)[NV], double* red) {   // red: 4 * NV
#pragma unroll
  for (int q = 0; q < NV; ++q)
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) v[q] += __shfl_xor(v[q], sh, 64);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q)
    if ((threadIdx.x & 63) == 0) red[q * 4 + (threadIdx.x >> 6)] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = (red[q * 4] + red[q * 4 + 1]) + (red[q * 4 + 2] + red[q * 4 + 3]);
}

template <typename T>
__global__ __launch_bounds__(256) void merge_gather_kernel(
    const T* __restrict__ x, int d, const int32_t* __restrict__ kept_idx, const int32_t* __restrict__ n_dev,
    const uint8_t* __restrict__ is_merged, const int32_t* __restrict__ cu, int B, int Ttot, int W,
    const int32_t* __restrict__ vis_ord, const int32_t* __restrict__ vis_tok,
    const int32_t* __restrict__ seq_nv, T* __restrict__ x_merged, int mean_only) {
  __shared__ double red[4 * MG_ROWS];
  const int p = blockIdx.x;
  const int t = kept_idx[p];
  const bool merged = is_merged[p] != 0;
  if (p >= *n_dev) return;
  const T* src = x + (size_t)t * d;
  T* dst = x_merged + (size_t)p * d;
  if (!merged) {
    constexpr int N = 16 / (int)sizeof(T);   // rows are 16-byte aligned: d is a multiple of 8
    for (int c = threadIdx.x * N; c < d; c += 256 * N)
      *reinterpret_cast<uint4*>(dst + c) = *reinterpret_cast<const uint4*>(src + c);
    return;
  }
  const int b = find_seq(cu, B, t);
  const int s = clampi(cu[b], 0, Ttot);
  const int ord = vis_ord[t];
  const int nv = seq_nv[b];
  const int w = (nv - ord < W) ? (nv - ord) : W;
  const int32_t* toks = vis_tok + s + ord;
  double max_row_sq = 0.0;   // Eq.18: the largest token norm of the window
  double sum[MG_COLS];       // Eq.16: of this thread's first columns
#pragma unroll
  for (int i = 0; i < MG_COLS; ++i) sum[i] = 0.0;
  for (int j0 = 0; j0 < w; j0 += MG_ROWS) {
    double part[MG_ROWS];
#pragma unroll
    for (int q = 0; q < MG_ROWS; ++q) {
      part[q] = 0.0;
      if (j0 + q < w) {   // uniform
        const T* row = x + (size_t)toks[j0 + q] * d;
#pragma unroll
        for (int i = 0; i < MG_COLS; ++i) {
          const int c = threadIdx.x + i * 256;
          const double v = c < d ? (double)to_f32(row[c]) : 0.0;
          part[q] += v * v;
          sum[i] += v;
        }
        for (int c = threadIdx.x + MG_COLS * 256; c < d; c += 256) {
          const double v = (double)to_f32(row[c]);
          part[q] += v * v;
        }
      }
    }
    block_sums_f64(part, red);
#pragma unroll
    for (int q = 0; q < MG_ROWS; ++q) max_row_sq = part[q] > max_row_sq ? part[q] : max_row_sq;
  }
  auto column_mean = [&](int c) -> double {   // Eq.16-17 with the window's real size
    double acc = 0.0;
    for (int j = 0; j < w; ++j) acc += (double)to_f32(x[(size_t)toks[j] * d + c]);
    return acc / (double)w;
  };
  double mean_sq[1] = {0.0};
#pragma unroll
  for (int i = 0; i < MG_COLS; ++i) {
    sum[i] = sum[i] / (double)w;
    mean_sq[0] += sum[i] * sum[i];
  }
  for (int c = threadIdx.x + MG_COLS * 256; c < d; c += 256) {
    const double mu = column_mean(c);
    mean_sq[0] += mu * mu;
  }
  block_sums_f64(mean_sq, red);
  const double mean_norm = sqrt(mean_sq[0]);
  // mean_only: the plain mean of the merge-method ablation instead of MLERP's rescaling
  const double scale = mean_only ? 1.0 : (mean_norm > 0.0 ? sqrt(max_row_sq) / mean_norm : 0.0);
#pragma unroll
  for (int i = 0; i < MG_COLS; ++i) {
    const int c = threadIdx.x + i * 256;
    if (c < d) dst[c] = from_f64<T>(sum[i] * scale);
  }
  for (int c = threadIdx.x + MG_COLS * 256; c < d; c += 256) dst[c] = from_f64<T>(column_mean(c) * scale);
}

__global__ void identity_kept_kernel(fmoe_keep_all_job job, int T) {
  keep_all(job, T, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// ---- E: small batches.  Two 1024-thread blocks take the whole chain after the window scores:
// drop order, budget, compaction, permutation by expert and the grouped-GEMM tile lists, with the
// intermediate arrays in LDS.  At a few thousand tokens each of those steps is a few microseconds
// of work and the launches between them cost more than the steps themselves.
//   * both blocks come to the same expert offsets; then one writes the token lists and the other the tile lists, neither
//     behind the other (1600 tokens 15.3 -> 13.5 us, permutation only 10.7 -> 9.8, a 64-token batch 8.9 -> 8.4).  Where
//     the new sequence bounds replace the old ones in place, one block does both: two would race on them;
//   * every global input is fetched up front (thread i owns tokens i, i+1024, ...), every global
//     output is stored at the very end, so no barrier in between waits on memory;
//   * drop order: the order (normalised attention asc, score desc, index asc) is total, and of the places in it
//     only one matters, that of the window at which the budget ends: a radix selection finds it, one window
//     per thread (with a bitonic sort for all places 1600 tokens took 19.9 us in this kernel, so they take 16.9);
//   * permutation: as in the stand-alone kernels (per-expert position masks, popcount ranks), one
//     pass per 1024 tokens, one 64-bit mask word per wavefront.
constexpr int SB_THREADS = 1024;
constexpr int SB_MAX_TP = 4;                       // tokens per thread, at most
constexpr int SB_MAX_T = SB_THREADS * SB_MAX_TP;   // tokens
constexpr int SB_MAX_NW = 1024;                // windows of one sequence: one per thread
constexpr int SB_MROW = 17;                    // 64-bit mask words per expert (16 + 1 against bank conflicts)
constexpr int SB_MAX_B = 512;                  // sequences whose bounds are cached in LDS

struct SmallArgs {
  int prune;                       // 0: keep every token
  const int32_t* T_dev;            // PERM_ONLY instantiation: device count of the tokens present (<= T)
  const uint8_t* is_visual;
  const int32_t* cu;
  int B, T, W;
  float retention, alpha;
  const int32_t* vis_ord;
  const int32_t* seq_nv;
  const float* win_s;
  const float* win_a;              // null without attention importance
  int32_t* kept_idx;
  int32_t* new_cu;
  uint8_t* is_visual_out;          // may be null
  const int32_t* topk_idx;
  int E, Kmax;
  int32_t* expert_offsets;
  int32_t* perm_src;
  int32_t* inv_perm;
  fmoe_ffn_geom geom;
  int n_shared, row_cap;
  fmoe_tile* tiles1;
  fmoe_tile* tiles2;
  int32_t* tile_count;
};

// SB_TP tokens per thread, at most KM experts per token (both fix the size of register arrays).
// PERM_ONLY: every token up to the device count *T_dev is kept (a.prune is 0); only the permutation
// and the tile lists are produced, kept_idx / new_cu / is_visual_out stay untouched.
template <int SB_TP, int KM, bool PERM_ONLY>
__global__ __launch_bounds__(SB_THREADS) void prune_dispatch_small_kernel(SmallArgs a) {
  __shared__ uint16_t s_before[SB_MAX_T];   // kept tokens ahead of each
  // phase 1: leading tokens kept per window u16[SB_MAX_T] | 3 x counts per byte value [256]
  // phase 2: position masks u64[FMOE_MAX_EXPERTS][SB_MROW]
  constexpr int U_BYTES = FMOE_MAX_EXPERTS * SB_MROW * 8;
  static_assert(SB_MAX_T * 2 + 3 * 256 * 4 <= U_BYTES, "phase-1 arrays fit");
  __shared__ __align__(16) unsigned char s_u[U_BYTES];
  __shared__ int s_off[FMOE_MAX_EXPERTS + 1], s_base[FMOE_MAX_EXPERTS];
  __shared__ int s_cu[SB_MAX_B + 1], s_nv[SB_MAX_B];
  __shared__ __align__(8) int s_scr[FMOE_TILES_SCRATCH];
  __shared__ uint16_t s_pfx[FMOE_MAX_EXPERTS * 16];   // rows of an expert ahead of each wavefront's tokens
  __shared__ int wave_tot[16];
  __shared__ float red[16];
  __shared__ uint32_t s_last[2], s_cut[3];   // keys of a shorter last window; of the window at which the budget ends
  uint16_t* s_pre = reinterpret_cast<uint16_t*>(s_u);
  int* const hist = reinterpret_cast<int*>(s_u + SB_MAX_T * 2);
  unsigned long long* mask = reinterpret_cast<unsigned long long*>(s_u);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int W = a.W, E = a.E, Kmax = a.Kmax, B = a.B;
  int T = a.T;
  if constexpr (PERM_ONLY) {
    const int Td = *a.T_dev;
    T = Td < T ? (Td > 0 ? Td : 0) : T;
  }

  // ---- all global inputs of this thread's tokens
  const int t_end = a.prune ? clampi(a.cu[B], 0, T) : T;
  int ord_r[SB_TP];
  uint8_t vis_r[SB_TP];
  int ex[SB_TP][KM];   // expert per slot, later (expert << 16 | row within the expert)
#pragma unroll
  for (int k = 0; k < SB_TP; ++k) {
    const int t = k * SB_THREADS + tid;
    ord_r[k] = (a.prune && t < t_end) ? a.vis_ord[t] : -1;   // past the last sequence: no ordinal, text
    vis_r[k] = (t < T && a.is_visual_out != nullptr) ? a.is_visual[t] : 0;
#pragma unroll
    for (int sl = 0; sl < KM; ++sl) {
      int e = -1;
      if (sl < Kmax && t < T) e = a.topk_idx[(size_t)t * Kmax + sl];
      ex[k][sl] = (e >= 0 && e < E) ? e : -1;
    }
  }
  // Under bounds that decrease a token's ordinal can be another sequence's and name a window that none has.  What stands
  // there has to be the same in both blocks, or their lists would not fit together.
  static_assert(SB_MAX_T * 4 == SB_THREADS * 16 && SB_MAX_T * 4 <= U_BYTES, "2 * SB_MAX_T entries");
  if (a.prune) *reinterpret_cast<uint4*>(s_u + tid * 16) = make_uint4(0, 0, 0, 0);
  const bool cached = B <= SB_MAX_B;
  if (cached) {
    for (int b = tid; b <= B; b += SB_THREADS) s_cu[b] = clampi(a.cu[b], 0, T);
    if (a.prune)
      for (int b = tid; b < B; b += SB_THREADS) s_nv[b] = a.seq_nv[b];
  }
  __syncthreads();
  const int32_t* cu = cached ? s_cu : a.cu;   // clamping a clamped bound changes nothing
  const int32_t* seq_nv = cached ? s_nv : a.seq_nv;

  // ---- drop order per sequence
  if (a.prune) {
    const bool has_attn = (a.win_a != nullptr);
    const float one_minus_alpha = 1.0f - a.alpha;
    for (int b = 0; b < B; ++b) {   // uniform over the block
      int s, e;
      seq_range(cu, b, T, s, e);
      const int nv = seq_nv[b];
      int n = (nv + W - 1) / W;
      n = n < SB_MAX_NW ? n : SB_MAX_NW;   // the launcher only takes batches where this holds
      if (n <= 0) continue;
      const float ws_r = (tid < n) ? a.win_s[s + tid] : 0.0f;
      const float wa_r = (has_attn && tid < n) ? a.win_a[s + tid] : 0.0f;
      float amax = 0.0f;
      if (has_attn) {   // per-sequence attention maximum (Eq.12)
        float m = (wa_r > 0.0f) ? wa_r : 0.0f;
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) {
          const float o = __shfl_xor(m, sh, 64);
          m = (o > m) ? o : m;
        }
        __syncthreads();
        if (lane == 0) red[wave] = m;
        __syncthreads();
        amax = red[0];
#pragma unroll
        for (int w = 1; w < 16; ++w) amax = (red[w] > amax) ? red[w] : amax;
      }
      uint32_t ka = 0u, kc = 0u;   // sort keys, ascending = drop order (ties: lower index)
      if (tid < n) {
        float A;
        const float c = redundancy_score(ws_r, has_attn, wa_r, amax, a.alpha, one_minus_alpha, A);
        kc = ~float_order_key(c);
        ka = float_order_key(A);
      }
      // How many full-size windows are dropped whole (q), what the next one loses (part), what the last window
      // keeps if it is shorter: that one's turn comes behind `ahead` full windows.
      const int w_last = nv - (n - 1) * W, n_full = w_last < W ? n - 1 : n;
      const bool full = tid < n_full;
      const int eps = nv - token_budget(nv, a.retention);
      int q = eps / W, part = eps - q * W, last_keeps = w_last;
      if (n_full < n) {   // uniform
        if (tid == n - 1) {
          s_last[0] = ka;
          s_last[1] = kc;
        }
        __syncthreads();
        const unsigned long long m = __ballot(full && (ka < s_last[0] || (ka == s_last[0] && kc <= s_last[1])));
        if (lane == 0) wave_tot[wave] = __popcll(m);
        __syncthreads();
        int ahead = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) ahead += wave_tot[w];
        if (q >= ahead) {
          const int u = eps - ahead * W;
          last_keeps = u < w_last ? w_last - u : 0;
          q = u < w_last ? ahead : ahead + (u - w_last) / W;
          part = u < w_last ? 0 : (u - w_last) % W;
        }
      }
      // The full window at place q, by its key's bytes from the highest on: counts of the candidates per byte value,
      // summed by every wavefront for itself; one barrier a byte, the tables take turns.
      bool candidate = full;
      int place = q;
      bool single = false;
      if (q < n_full) {   // uniform
        for (int i = tid; i < 256; i += SB_THREADS) hist[i] = 0;
        __syncthreads();
        int table = 0;
        for (int byte = has_attn ? 0 : 4; byte < 8 && !single; ++byte) {   // uniform
          int* const h = hist + table * 256;
          table = table == 2 ? 0 : table + 1;
          for (int i = tid; i < 256; i += SB_THREADS) hist[table * 256 + i] = 0;
          const int digit = (int)((byte < 4 ? ka : kc) >> (24 - 8 * (byte & 3))) & 255;
          if (candidate) atomicAdd(&h[digit], 1);
          __syncthreads();
          const int4 c4 = *reinterpret_cast<const int4*>(&h[4 * lane]);
          const int sum4 = c4.x + c4.y + c4.z + c4.w;
          const int excl = wave_scan(sum4) - sum4;
          const int src = __builtin_ctzll(__ballot(excl <= place && place < excl + sum4));   // exactly one lane
          int before = excl, val = 4 * lane, here = c4.x;
          if (before + here <= place) { before += here; here = c4.y; ++val; }
          if (val > 4 * lane && before + here <= place) { before += here; here = c4.z; ++val; }
          if (val > 4 * lane + 1 && before + here <= place) { before += here; here = c4.w; ++val; }
          place -= __builtin_amdgcn_readlane(before, src);
          candidate = candidate && digit == __builtin_amdgcn_readlane(val, src);
          single = __builtin_amdgcn_readlane(here, src) == 1;
        }
        if (!single) {   // equal keys: by index
          const unsigned long long m = __ballot(candidate);
          if (lane == 0) wave_tot[wave] = __popcll(m);
          __syncthreads();
          int pos = __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
          for (int w = 0; w < 16; ++w) pos += w < wave ? wave_tot[w] : 0;
          candidate = candidate && pos == place;
        }
        if (candidate) {
          s_cut[0] = ka;
          s_cut[1] = kc;
          s_cut[2] = (uint32_t)tid;
        }
      }
      __syncthreads();
      if (tid < n) {   // leading tokens that stay
        int lead = last_keeps;
        if (full && q < n_full) {
          const uint32_t ca = s_cut[0], cc = s_cut[1];
          const int ci = (int)s_cut[2];
          const bool ahead = ka != ca ? ka < ca : (kc != cc ? kc < cc : tid < ci);
          lead = ahead ? 0 : (tid == ci ? W - part : W);
        } else if (full) {
          lead = 0;
        }
        s_pre[s + tid] = (uint16_t)lead;
      }
      __syncthreads();
    }
  }

  // ---- budget: text tokens and the leading tokens of each window stay
  bool keep_r[SB_TP];
#pragma unroll
  for (int k = 0; k < SB_TP; ++k) {
    const int t = k * SB_THREADS + tid;
    bool keep = false;
    if (t < T) {
      const int ord = ord_r[k];
      if (ord < 0) {
        keep = true;
      } else {
        const int b = find_seq(cu, B, t);
        const int s = clampi(cu[b], 0, T);
        const unsigned w = (unsigned)(s + ord / W);
        keep = (ord % W) < s_pre[w < 2 * SB_MAX_T ? w : 0];
      }
    }
    keep_r[k] = keep;
  }
  __syncthreads();   // s_pre is dead from here on: the masks take its place

  // ---- compaction + per-expert ranks, one pass per 1024 tokens
  if (tid < FMOE_MAX_EXPERTS) s_base[tid] = 0;
  int pos_r[SB_TP];
  int running = 0;
#pragma unroll
  for (int k = 0; k < SB_TP; ++k) {
    pos_r[k] = -1;
    if (k * SB_THREADS < T) {   // uniform
      const int t = k * SB_THREADS + tid;
      const bool keep = keep_r[k];
      const unsigned long long m = __ballot(keep);
      const int before = __popcll(m & ((1ull << lane) - 1ull));
      if (lane == 0) wave_tot[wave] = __popcll(m);
      for (int i = tid; i < E * SB_MROW; i += SB_THREADS) mask[i] = 0ull;
      __syncthreads();
      int wave_base = 0, total = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        if (w < wave) wave_base += wave_tot[w];
        total += wave_tot[w];
      }
      if (t < T) s_before[t] = (uint16_t)(running + wave_base + before);
      if (keep) {
        pos_r[k] = running + wave_base + before;
#pragma unroll
        for (int sl = 0; sl < KM; ++sl)
          if (sl < Kmax && ex[k][sl] >= 0)   // a half of the word
            atomicOr(reinterpret_cast<uint32_t*>(&mask[ex[k][sl] * SB_MROW + wave]) + (lane >> 5), 1u << (lane & 31));
      }
      running += total;
      __syncthreads();
      // item (expert, wavefront w): rows of the expert so far = earlier passes + wavefronts below w
      for (int it = tid; it < E * 16; it += SB_THREADS) {   // 16 consecutive lanes share an expert
        const int e = it >> 4, w = it & 15;
        const int c = __popcll(mask[e * SB_MROW + w]);
        const int base = s_base[e];
        const int incl = row_scan(c);
        s_pfx[it] = (uint16_t)(base + incl - c);
        if (w == 15) s_base[e] = base + incl;   // same wavefront: every lane has read the old value
      }
      __syncthreads();
      if (keep) {
#pragma unroll
        for (int sl = 0; sl < KM; ++sl) {
          if (sl < Kmax && ex[k][sl] >= 0) {
            const int e = ex[k][sl];
            const int rank = (int)s_pfx[e * 16 + wave] +
                             __popcll(mask[e * SB_MROW + wave] & ((1ull << lane) - 1ull));
            ex[k][sl] = (e << 16) | rank;
          }
        }
      } else {
#pragma unroll
        for (int sl = 0; sl < KM; ++sl) ex[k][sl] = -1;
      }
      __syncthreads();
    }
  }
  const int n = running;

  // ---- expert offsets: exclusive scan of the (at most 256) totals, four per lane
  __syncthreads();
  if (wave == 0) {
    int c[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = 4 * lane + q;
      c[q] = (e < E) ? s_base[e] : 0;
      sum += c[q];
    }
    const int incl = wave_scan(sum);
    int excl = incl - sum;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s_off[4 * lane + q] = excl;
      excl += c[q];
    }
    if (lane == 63) s_off[FMOE_MAX_EXPERTS] = incl;
  }
  __syncthreads();

  // ---- grouped-GEMM tile lists, by the last block
  if (blockIdx.x + 1 == gridDim.x) {
    fmoe_build_tiles<true>(s_off, E, a.row_cap, n, a.n_shared, a.geom.bm, a.geom.run, a.geom.tile_cap, a.geom.cols1,
                           a.geom.scols1, a.tiles1, a.tiles2, a.tile_count, s_scr);
    if (tid <= E) a.expert_offsets[tid] = s_off[tid];
  }
  if (blockIdx.x != 0) return;

  // ---- token lists
  for (int b = tid; b <= B && !PERM_ONLY; b += SB_THREADS) {   // new_cu[b] = kept tokens before the sequence start
    const int c = clampi(cu[b], 0, T);
    a.new_cu[b] = c < T ? s_before[c] : n;
  }
#pragma unroll
  for (int k = 0; k < SB_TP; ++k) {
    const int p = pos_r[k];
    if (p >= 0) {
      if constexpr (!PERM_ONLY) {
        a.kept_idx[p] = k * SB_THREADS + tid;
        if (a.is_visual_out != nullptr) a.is_visual_out[p] = vis_r[k];
      }
#pragma unroll
      for (int sl = 0; sl < KM; ++sl) {
        if (sl < Kmax) {
          int row = -1;
          if (ex[k][sl] >= 0) {
            row = s_off[ex[k][sl] >> 16] + (ex[k][sl] & 0xffff);
            if (row < a.row_cap) a.perm_src[row] = p;
          }
          a.inv_perm[(size_t)p * Kmax + sl] = row;
        }
      }
    }
  }
}

// Do the sequence bounds before and after share memory?
bool same_bounds(const int32_t* cu, const int32_t* new_cu, int B) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(cu), b = reinterpret_cast<uintptr_t>(new_cu), n = ((uintptr_t)B + 1) * 4;
  return a < b + n && b < a + n;
}

// One wavefront per window unit (floor(T/W) + B units cover every window), four per block.
void launch_window_scores(const float* probs, const int32_t* cu_seqlens, int B, int T, int E, int W,
                          int sim_mode, const int32_t* vis_tok, const int32_t* seq_nv, const float* attn,
                          float* win_s, float* win_a, hipStream_t stream) {
  const int n_units = T / W + B;
  const dim3 grid((n_units + 3) / 4);
  if ((long long)W * E <= WS_TILE)
    hipLaunchKernelGGL(window_score_kernel<true>, grid, dim3(256), 0, stream, probs, cu_seqlens, B, T, E, W,
                       sim_mode, vis_tok, seq_nv, attn, win_s, win_a);
  else
    hipLaunchKernelGGL(window_score_kernel<false>, grid, dim3(256), 0, stream, probs, cu_seqlens, B, T, E, W,
                       sim_mode, vis_tok, seq_nv, attn, win_s, win_a);
}

}  // namespace

int launch_prune(const fmoe_ctx* ctx, const fmoe_prune_params* pp, const float* probs,
                 const uint8_t* is_visual, const int32_t* cu_seqlens, int B, int T,
                 const float* attn, int32_t* kept_idx, int32_t* new_cu_seqlens, float* scores_out,
                 uint8_t* is_visual_out, const void* x_in, void* x_merged, uint8_t* is_merged_out,
                 void* ws, const fmoe_ws_layout& L, hipStream_t stream, bool ordinals_ready) {
  char* base = static_cast<char*>(ws);
  int32_t* vis_tok = reinterpret_cast<int32_t*>(base + L.vis_tok);
  int32_t* vis_ord = reinterpret_cast<int32_t*>(base + L.vis_ord);
  int32_t* seq_nv = reinterpret_cast<int32_t*>(base + L.seq_nv);
  float* win_s = reinterpret_cast<float*>(base + L.win_s);
  float* win_a = attn ? reinterpret_cast<float*>(base + L.win_a) : nullptr;
  const bool merging = pp->gamma > 0.0f;
  uint8_t* is_merged = is_merged_out;
  if (merging && is_merged == nullptr) is_merged = reinterpret_cast<uint8_t*>(base + L.is_merged);
  // blocks of the compaction and the gather behind it read the bounds while one block writes the new ones: if these are
  // to take their place, they wait in the workspace
  const bool in_place = same_bounds(cu_seqlens, new_cu_seqlens, B);
  int32_t* const new_cu = in_place ? reinterpret_cast<int32_t*>(base + L.new_cu) : new_cu_seqlens;
  const int E = ctx->cfg.n_experts;
  if (T == 0 || B == 0) return launch_identity_kept(is_visual, cu_seqlens, B, T, kept_idx,
                                                    new_cu_seqlens, is_visual_out, stream);

  if (!ordinals_ready) {
    fmoe_prof_scope prof(ctx, SLOT_ORDINALS, stream);
    hipLaunchKernelGGL(seq_ordinals_kernel, dim3(B), dim3(256), 0, stream, is_visual, cu_seqlens, T,
                       vis_ord, vis_tok, seq_nv);
  }
  {
    fmoe_prof_scope prof(ctx, SLOT_SCORES, stream);
    launch_window_scores(probs, cu_seqlens, B, T, E, pp->window, pp->sim_mode, vis_tok, seq_nv, attn, win_s,
                         win_a, stream);
  }
  {
    fmoe_prof_scope prof(ctx, SLOT_COMPACT, stream);
    CompactArgs ca;
    ca.is_visual = is_visual; ca.cu = cu_seqlens; ca.B = B; ca.T = T; ca.W = pp->window;
    ca.retention = pp->retention; ca.gamma = pp->gamma; ca.alpha = pp->alpha;
    ca.vis_ord = vis_ord; ca.seq_nv = seq_nv; ca.win_s = win_s; ca.win_a = win_a;
    ca.scores_out = scores_out; ca.kept_idx = kept_idx; ca.new_cu = new_cu; ca.is_visual_out = is_visual_out;
    ca.is_merged_out = merging ? is_merged : nullptr;
    ca.window_rcp = ((1ull << 37) + pp->window - 1) / pp->window;
    ca.cut = B > 1 && B <= CP_CUT_SEQS;
    // cut: part j of the batch begins at block (its first position) / CP_BLOCK + j
    const dim3 grid(ca.cut ? T / CP_BLOCK + B + 2 : (T + CP_BLOCK - 1) / CP_BLOCK), block(CP_BLOCK);
    if (merging && attn) hipLaunchKernelGGL((compact_kernel<true, true>), grid, block, 0, stream, ca);
    else if (merging) hipLaunchKernelGGL((compact_kernel<true, false>), grid, block, 0, stream, ca);
    else if (attn) hipLaunchKernelGGL((compact_kernel<false, true>), grid, block, 0, stream, ca);
    else hipLaunchKernelGGL((compact_kernel<false, false>), grid, block, 0, stream, ca);
  }
  if (merging) {
    if (ctx->cfg.dtype == FMOE_BF16)
      hipLaunchKernelGGL(merge_gather_kernel<bf16_t>, dim3(T), dim3(256), 0, stream,
                         static_cast<const bf16_t*>(x_in), ctx->cfg.d_model, kept_idx, new_cu + B,
                         is_merged, cu_seqlens, B, T, pp->window, vis_ord, vis_tok, seq_nv,
                         static_cast<bf16_t*>(x_merged), pp->merge_mode);
    else
      hipLaunchKernelGGL(merge_gather_kernel<float>, dim3(T), dim3(256), 0, stream,
                         static_cast<const float*>(x_in), ctx->cfg.d_model, kept_idx, new_cu + B,
                         is_merged, cu_seqlens, B, T, pp->window, vis_ord, vis_tok, seq_nv,
                         static_cast<float*>(x_merged), pp->merge_mode);
  }
  FMOE_HIP_CHECK(hipGetLastError());
  if (in_place) return launch_identity_kept(nullptr, new_cu, B, T, nullptr, new_cu_seqlens, nullptr, stream);
  return FMOE_OK;
}

int launch_identity_kept(const uint8_t* is_visual, const int32_t* cu_seqlens, int B, int T,
                         int32_t* kept_idx, int32_t* new_cu_seqlens, uint8_t* is_visual_out,
                         hipStream_t stream) {
  const int n = (T > B + 1) ? T : B + 1;
  hipLaunchKernelGGL(identity_kept_kernel, dim3((n + 255) / 256), dim3(256), 0, stream,
                     fmoe_keep_all_job{is_visual, cu_seqlens, B, kept_idx, new_cu_seqlens, is_visual_out}, T);
  FMOE_HIP_CHECK(hipGetLastError());
  return FMOE_OK;
}

bool dispatch_small_fits(int T, int window, bool prune) {
  if (T <= 0 || T > SB_MAX_T) return false;
  return !prune || (T + window - 1) / window <= SB_MAX_NW;
}

int launch_prune_dispatch_small(const fmoe_ctx* ctx, const fmoe_prune_params* pp, bool prune,
                                const float* probs, const uint8_t* is_visual, const int32_t* cu_seqlens,
                                int B, int T, const float* attn, const int32_t* topk_idx,
                                int32_t* kept_idx, int32_t* new_cu_seqlens, uint8_t* is_visual_out,
                                int32_t* expert_offsets, int32_t* perm_src, int32_t* inv_perm, void* ws,
                                const fmoe_ws_layout& L, hipStream_t stream, const int32_t* T_dev,
                                bool write_kept) {
  char* base = static_cast<char*>(ws);
  int32_t* vis_tok = reinterpret_cast<int32_t*>(base + L.vis_tok);
  int32_t* vis_ord = reinterpret_cast<int32_t*>(base + L.vis_ord);
  int32_t* seq_nv = reinterpret_cast<int32_t*>(base + L.seq_nv);
  float* win_s = reinterpret_cast<float*>(base + L.win_s);
  float* win_a = attn ? reinterpret_cast<float*>(base + L.win_a) : nullptr;
  const int E = ctx->cfg.n_experts;
  if (prune) {   // the visual ordinals were produced in the router's launch
    fmoe_prof_scope prof(ctx, SLOT_SCORES, stream);
    launch_window_scores(probs, cu_seqlens, B, T, E, pp->window, pp->sim_mode, vis_tok, seq_nv, attn, win_s,
                         win_a, stream);
  }
  SmallArgs a;
  a.prune = prune ? 1 : 0;
  a.T_dev = T_dev;
  a.is_visual = is_visual;
  a.cu = cu_seqlens;
  a.B = B; a.T = T; a.W = prune ? pp->window : 1;
  a.retention = prune ? pp->retention : 1.0f;
  a.alpha = prune ? pp->alpha : 1.0f;
  a.vis_ord = vis_ord; a.seq_nv = seq_nv; a.win_s = win_s; a.win_a = win_a;
  a.kept_idx = kept_idx; a.new_cu = new_cu_seqlens; a.is_visual_out = is_visual_out;
  a.topk_idx = topk_idx;
  a.E = E; a.Kmax = ctx->kmax;
  a.expert_offsets = expert_offsets; a.perm_src = perm_src; a.inv_perm = inv_perm;
  a.geom = fmoe_geom(ctx, T);
  a.n_shared = ctx->cfg.n_shared;
  a.row_cap = T * ctx->kmax;
  a.tiles1 = reinterpret_cast<fmoe_tile*>(base + L.tiles);
  a.tiles2 = reinterpret_cast<fmoe_tile*>(base + L.tiles2);
  a.tile_count = reinterpret_cast<int32_t*>(base + L.tile_count);
  {
    fmoe_prof_scope prof(ctx, SLOT_DISPATCH, stream);
    if (!write_kept && (prune || T_dev == nullptr))
      return fmoe_fail(FMOE_ERR_INVALID_ARG, "small dispatch: the permutation-only form needs a device token count and no pruning");
    const dim3 grid(write_kept && same_bounds(cu_seqlens, new_cu_seqlens, B) ? 1 : 2);
#define FMOE_DISPATCH_LAUNCH(TP, KM)                                                                         \
  do {                                                                                                       \
    if (write_kept)                                                                                          \
      hipLaunchKernelGGL((prune_dispatch_small_kernel<TP, KM, false>), grid, dim3(SB_THREADS), 0, stream, a); \
    else                                                                                                     \
      hipLaunchKernelGGL((prune_dispatch_small_kernel<TP, KM, true>), grid, dim3(SB_THREADS), 0, stream, a);  \
  } while (0)
    // the register arrays as small as the call allows: with those for sixteen experts per token a batch of 3000
    // tokens and six took 34.6 us (pruning, the drop order then still sorted) and 25.8 us (not), with those for eight
    // 29.2 and 20.8
    if (ctx->kmax > 8) FMOE_DISPATCH_LAUNCH(SB_MAX_TP, FMOE_MAX_TOPK);
    else if (T > 2 * SB_THREADS) FMOE_DISPATCH_LAUNCH(SB_MAX_TP, 8);
    else FMOE_DISPATCH_LAUNCH(2, 8);
#undef FMOE_DISPATCH_LAUNCH
  }
  FMOE_HIP_CHECK(hipGetLastError());
  return FMOE_OK;
}

