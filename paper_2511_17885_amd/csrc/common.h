// Internal declarations shared by the library's translation units (host side + device helpers).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fmoe.h"

#define FMOE_MAX_EXPERTS 256
#define FMOE_MAX_TOPK 16
#define FMOE_MAX_WINDOW 64
#define FMOE_PERM_BLOCK 256   // kept positions per block in the permutation kernels
#define FMOE_ROUTE_DISPATCH_TOKENS 16   // tokens up to which the router's one block does the dispatch too
#define FMOE_TILE_M 64        // rows per grouped-GEMM tile (tile list granularity)
#define FMOE_TILE_RUN 8       // row tiles per run of a group in the tile lists
#define FMOE_DENSE_TILE_RUN 64   // the same for the dense shape
#define FMOE_SEG_MIN_TILES 256   // tile entries from which each XCD takes a contiguous segment of the list
// Routed-row capacity per expert from which the expert GEMMs take their dense shape, by how much there is to do with one
// row tile an expert: work items (column groups of the narrower GEMM) and length of the shorter reduction.  The dense
// shape's items are twice as long and half as many; where they leave the chip half idle the weight-stream shape wins
// until experts have several row tiles.  Gate/up + down, stream / dense, us, layer after layer: half of the visual tokens
// kept, all kept (both half of the experts a token), all kept with all experts; the lines lie between the layers measured:
//   704 gate/up, 512 down items (d 2048, 64 experts of 1408, two shared): capacity 80 158/152, 199/195, 243/226;
//     120 189/181, 234/218, 287/269
//   768 and 1024 (d 2048, 128 of 768): 100 121/118, 146/148, 213/199; 120 125/123, 156/159, 232/207; 150 144/142, 188/181
//   448 and 320 (d 1280, 64 of 896, two shared): 120 78/81, 102/96, 129/125; 150 85/83, 110/103, 145/140
//   420 and 300 (d 1280, 60 of 896): 150 70/76, 84/82, 114/114; 215 75/81, 97/96, 141/135; 250 82/83, 105/103, 155/148
//   288 (d 2048, 36 of 1024): 150 90/99, 117/107, 143/138; 180 103/101, 124/114; 256: 150 87/97, 105/101; 215 105/101
//   96 and 128 (d 4096, 8 of 1536): 215 76/100, 103/101, 142/152; 300 101/102, 110/103, 145/151
//   short reductions: 704 (d 2048, 112 experts, 672 and 896 items) 120 139/142, 168/167, 220/207; 150 153/163, 183/179;
//     215 174/176, 212/199; 640 (128 experts) 150 155/158, 189/192, 267/237; 576 215 154/157, 198/185; 512 (d 1024) 180
//     67/68, 85/84, 122/113; 250 77/75, 103/104, 149/136
// One decision for both GEMMs: alone the down product of 64 experts of 896 at capacity 150, half kept, is faster in the
// weight-stream shape (33 against 35 us), but behind a gate/up product in the dense shape that gains nothing (layer of
// 1600 tokens, runs of 8 / 64 row tiles: half kept 114.4 -> 115.3 / 113.9 -> 113.1 us, three quarters with merging
// 167.5 -> 169.7 / 168.1 -> 170.3).
#define FMOE_DENSE_MIN_ROWS 112        // from FMOE_DENSE_ITEMS items on
#define FMOE_DENSE_MIN_ROWS_SOME 144   // from FMOE_DENSE_ITEMS_SOME on
#define FMOE_DENSE_MIN_ROWS_FEW 256    // fewer, or shorter reductions than FMOE_DENSE_MIN_K
#define FMOE_DENSE_ITEMS 480
#define FMOE_DENSE_ITEMS_SOME 310
#define FMOE_DENSE_MIN_K 736

// ---- optional per-kernel timing (instrumentation; off by default)
enum fmoe_kernel_slot {
  SLOT_ROUTE = 0, SLOT_ORDINALS, SLOT_SCORES, SLOT_COMPACT, SLOT_DISPATCH,
  SLOT_PERM_COUNT, SLOT_PERM_SCAN, SLOT_PERM_SCATTER, SLOT_TILES, SLOT_GEMM1, SLOT_GEMM2,
  SLOT_COMBINE, SLOT_GEMM1_DENSE, SLOT_GEMM2_DENSE, SLOT_COUNT
};
struct fmoe_prof {
  bool on;
  hipEvent_t beg[SLOT_COUNT], end[SLOT_COUNT];
  bool used[SLOT_COUNT];
};

struct fmoe_ctx {
  fmoe_config cfg;
  int device;
  int kmax;
  const void* router_w;      // caller's [E,H] in dtype
  float* router_wp;          // private fp32 copy of router_w in the router kernel's operand order
  const float* router_bias;
  const void *w_gate, *w_up, *w_down;
  const void *ws_gate, *ws_up, *ws_down;
  // bf16 contexts: private copies of the expert weights in matrix-core operand order (ffn.hip)
  void *pk_gate_up, *pk_down, *pk_sgate_up, *pk_sdown;
  bool weights_set;
  int sel_strategy, sel_k_base;   // selection-strategy ablation (fmoe_set_selection); 0 = off
  unsigned long long sel_seed;
  int ffn_shape;                  // fmoe_set_ffn_shape: 0 by size, 1 weight-stream, 2 dense
  fmoe_prof* prof;           // nullptr unless fmoe_profile_enable was called
};

// Brackets one kernel launch with events when profiling is on (host-side cost only then).
struct fmoe_prof_scope {
  fmoe_prof* p; int slot; hipStream_t s;
  fmoe_prof_scope(const fmoe_ctx* ctx, int slot_, hipStream_t s_) : p(ctx->prof), slot(slot_), s(s_) {
    if (p && p->on) { (void)hipEventRecord(p->beg[slot], s); } else { p = nullptr; }
  }
  ~fmoe_prof_scope() {
    if (p) { (void)hipEventRecord(p->end[slot], s); p->used[slot] = true; }
  }
};

// ---- error reporting (api.cpp)
int fmoe_fail(int code, const char* fmt, ...);
#define FMOE_HIP_CHECK(expr)                                                              \
  do {                                                                                    \
    hipError_t _e = (expr);                                                               \
    if (_e != hipSuccess)                                                                 \
      return fmoe_fail(FMOE_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(_e));      \
  } while (0)

// ---- workspace layout: one carve-up used by every entry point
struct fmoe_ws_layout {
  size_t probs, topk_idx, topk_gate;            // layer_forward intermediates
  size_t vis_tok, vis_ord, seq_nv;              // prune
  size_t win_s, win_a, new_cu;                  // prune
  size_t is_merged, vis_out, x_merged;          // layer_forward with window merging
  size_t slot_rank, blk_count;                  // permute
  size_t expert_offsets, perm_src, inv_perm;    // layer_forward intermediates
  size_t tiles, tiles2, tile_count;             // grouped GEMM tile lists (gate/up, down)
  size_t h, h_shared, y, y_shared;              // FFN intermediates
  size_t total;
};
fmoe_ws_layout fmoe_layout(const fmoe_ctx* ctx, int32_t max_tokens, int32_t max_seqs);

struct fmoe_tile {  // one M-tile of the grouped GEMM.  The rows are given for its run of consecutive entries (row tiles
                    // of one group), so that every tile of the run follows from any of the run's entries
  int32_t group;    // expert id
  int32_t row0;     // first row of the run (in the permuted row space)
  int32_t rows;     // valid rows from there to the end of the group
  int32_t col0;     // first column tile this entry covers (shared group split over entries)
  int32_t rt;       // index of this row tile within the run
  int32_t nrt;      // number of row tiles in the run
};

// launch geometry of the two grouped GEMMs for a call with capacity n_cap
struct fmoe_ffn_geom {
  int bm;              // rows per tile
  int run;             // row tiles per run
  bool dense;          // bf16: by size, the dense shape of the expert GEMMs
  int cols1, scols1;   // column tiles per launch entry / of the shared group, gate-up GEMM
  int cols2, scols2;   // same, down GEMM
  int tile_cap;        // capacity of each tile list
};
fmoe_ffn_geom fmoe_geom(const fmoe_ctx* ctx, int n_cap);
size_t fmoe_packed_bytes(const fmoe_ctx* ctx, int which);   // 0 gate/up, 1 down, 2 shared gate/up, 3 shared down
int launch_pack_experts(fmoe_ctx* ctx, hipStream_t stream);

// ---- kernel launchers (each returns a fmoe_status; all work goes to `stream`)
size_t router_pack_floats(const fmoe_ctx* ctx);
int launch_pack_router(const fmoe_ctx* ctx, const void* router_w, float* wp, hipStream_t stream);

// Visual ordinals to be produced by extra blocks of the router's launch (Sec. 3.2 needs them before
// the window scores; they do not depend on the routing).  cu == nullptr: none.
struct fmoe_ordinals_job {
  const int32_t* cu;
  int B;
  int32_t *vis_ord, *vis_tok, *seq_nv;
};
// What the dispatch step writes when every token is kept, for a router launch of one block to write as well
// (at most FMOE_ROUTE_DISPATCH_TOKENS tokens, default selection strategy).
struct fmoe_dispatch_job {
  const int32_t* cu;
  int B;
  int32_t *kept_idx, *new_cu;
  uint8_t* is_visual_out;      // or nullptr
  int32_t *expert_offsets, *perm_src, *inv_perm;
  fmoe_ffn_geom geom;
  int n_shared, row_cap;
  fmoe_tile *tiles1, *tiles2;
  int32_t* tile_count;
};
// T_dev (nullable): device count of the tokens actually present (<= T, the capacity).  dispatch (nullable): see above.
int launch_route(const fmoe_ctx* ctx, const void* x, const uint8_t* is_visual, int T, float* probs,
                 int32_t* topk_idx, float* topk_gate, const fmoe_ordinals_job& ord, hipStream_t stream,
                 const int32_t* T_dev = nullptr, const fmoe_dispatch_job* dispatch = nullptr);

int launch_prune(const fmoe_ctx* ctx, const fmoe_prune_params* pp, const float* probs,
                 const uint8_t* is_visual, const int32_t* cu_seqlens, int B, int T,
                 const float* attn, int32_t* kept_idx, int32_t* new_cu_seqlens, float* scores_out,
                 uint8_t* is_visual_out, const void* x_in, void* x_merged, uint8_t* is_merged_out,
                 void* ws, const fmoe_ws_layout& L, hipStream_t stream, bool ordinals_ready = false);

// Small batches: window scores, then ONE launch for drop order, compaction, permutation by expert and
// the grouped-GEMM tile lists (prune == false: every token is kept).  Expects the visual ordinals in
// the workspace (fmoe_ordinals_job) when pruning.  T_dev (nullable): device count of the tokens present;
// write_kept = false: permutation and tile lists only (kept_idx / new_cu_seqlens / is_visual_out untouched).
bool dispatch_small_fits(int T, int window, bool prune);
int launch_prune_dispatch_small(const fmoe_ctx* ctx, const fmoe_prune_params* pp, bool prune,
                                const float* probs, const uint8_t* is_visual, const int32_t* cu_seqlens,
                                int B, int T, const float* attn, const int32_t* topk_idx,
                                int32_t* kept_idx, int32_t* new_cu_seqlens, uint8_t* is_visual_out,
                                int32_t* expert_offsets, int32_t* perm_src, int32_t* inv_perm, void* ws,
                                const fmoe_ws_layout& L, hipStream_t stream, const int32_t* T_dev = nullptr,
                                bool write_kept = true);

int launch_identity_kept(const uint8_t* is_visual, const int32_t* cu_seqlens, int B, int T,
                         int32_t* kept_idx, int32_t* new_cu_seqlens, uint8_t* is_visual_out,
                         hipStream_t stream);

// What the pruning writes where every token is kept (kept list, sequence bounds, modality mask; any output may be null).
struct fmoe_keep_all_job {
  const uint8_t* is_visual;
  const int32_t* cu;
  int B;
  int32_t *kept_idx, *new_cu;
  uint8_t* is_visual_out;
};
// build_tiles: also write the grouped-GEMM tile lists (geometry from fmoe_geom(ctx, n_cap)).  all (nullable; with its
// kept_idx): all n_cap positions are kept, write that as well.
int launch_permute(const fmoe_ctx* ctx, const int32_t* topk_idx, const int32_t* kept_idx, int n_cap,
                   const int32_t* n_dev, int32_t* expert_offsets, int32_t* perm_src,
                   int32_t* inv_perm, void* ws, const fmoe_ws_layout& L, bool build_tiles,
                   hipStream_t stream, const fmoe_keep_all_job* all = nullptr);



int launch_expert_ffn(const fmoe_ctx* ctx, const void* x, const int32_t* kept_idx, int n_cap,
                      const int32_t* n_dev, const int32_t* expert_offsets, const int32_t* perm_src,
                      void* y, void* y_shared, void* ws, const fmoe_ws_layout& L, bool tiles_ready,
                      hipStream_t stream);

int launch_combine(const fmoe_ctx* ctx, const void* y, const void* y_shared, const int32_t* inv_perm,
                   const float* topk_gate, const int32_t* kept_idx, int n_cap, const int32_t* n_dev,
                   int n_expected, const void* residual, void* out, hipStream_t stream);

// ---- diagnostics (diag.hip)
int launch_adjacent_similarity(const float* probs, const uint8_t* is_visual, const int32_t* cu, int B, int T,
                               int E, float* pair_sim, float* mean, int32_t* count, hipStream_t stream);
int launch_magnitude_stability(const fmoe_ctx* ctx, const void* y, int M, const int32_t* M_dev,
                               const int32_t* perm_src, const int32_t* kept_idx, const uint8_t* is_visual,
                               float* row_norm, float* stats, hipStream_t stream);
int launch_row_cosine(const fmoe_ctx* ctx, const void* a, const void* b, int n, const int32_t* n_dev, float* out,
                      hipStream_t stream);
int launch_gate_cosine(const float* gates, int T, int K, int m, float* out, hipStream_t stream);

// ---- device helpers
#if defined(__HIPCC__)
typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even; inputs are finite in this library's data paths
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return bf16_to_f32(v); }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return f32_to_bf16(v); }

// One rounding from fp64 to the storage type.  bf16 goes through an fp32 value rounded to odd (the
// truncated value with a sticky last bit), from which the nearest-even rounding to 8 significant
// bits is the same as from the double itself.
template <typename T> __device__ __forceinline__ T from_f64(double v);
template <> __device__ __forceinline__ float from_f64<float>(double v) { return (float)v; }
template <> __device__ __forceinline__ bf16_t from_f64<bf16_t>(double v) {
  const float f = (float)v;
  const double back = (double)f;
  uint32_t u = __float_as_uint(f);
  if (back != v) {
    if (fabs(back) > fabs(v)) u -= 1u;   // step back towards zero: the truncated value
    u |= 1u;
  }
  return f32_to_bf16(__uint_as_float(u));
}

// Inclusive prefix sum over the wavefront's lanes, inside the vector unit: within rows of 16, then the rows' totals.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or_zero(int v) {   // lanes without a source, or in other rows, get 0
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int row_scan(int v) {   // over the lanes of each row of 16
  v += dpp_or_zero<0x111, 0xf>(v);   // row_shr:1
  v += dpp_or_zero<0x112, 0xf>(v);   // row_shr:2
  v += dpp_or_zero<0x114, 0xf>(v);   // row_shr:4
  return v + dpp_or_zero<0x118, 0xf>(v);   // row_shr:8
}
__device__ __forceinline__ int wave_scan(int v) {
  v = row_scan(v);
  v += dpp_or_zero<0x142, 0xa>(v);   // the last lane of rows 0 and 2 to rows 1 and 3
  return v + dpp_or_zero<0x143, 0xc>(v);   // lane 31 to rows 2 and 3
}

// number of valid entries: the device-side count if given (clamped to the capacity), else cap
__device__ __forceinline__ int resolve_count(int cap, const int32_t* n_dev) {
  if (n_dev == nullptr) return cap;
  int n = *n_dev;
  return n < 0 ? 0 : (n > cap ? cap : n);
}
#endif
