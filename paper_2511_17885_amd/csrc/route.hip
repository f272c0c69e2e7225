// Router: logits (Eq.1), softmax (Eq.2), modality-dependent top-k (Eq.3), gates (Eq.5).
//
// Every float here feeds a decision (which experts a token uses), so the arithmetic follows a
// fixed order that any IEEE-754 machine reproduces bit for bit.  This file is compiled with
// floating-point contraction off; fused multiply-adds appear only where fmaf is written.
//
//  logit:  the plain fp32 dot product in index order, acc = fmaf(x[k], w[k], acc) for k = 0..d-1
//          from +0.  The fp32 matrix-core instruction v_mfma_f32_16x16x4_f32 performs exactly this
//          chain (its four k per instruction are applied in ascending order, one rounding each;
//          verified bit for bit on gfx950), so a 16-token x 16-expert tile of logits costs one
//          instruction per four k and the chain is reproduced by a scalar fmaf loop anywhere else.
//  exp:    range reduction by rint(x*log2 e) with a two-constant ln 2, degree-7 Taylor polynomial
//          in Horner form, exact scaling by 2^n; flushed to 0 once 2^n leaves the normal range.
//  sum:    lane l adds q[l], q[l+64], ... in that order from +0, then a 6-level xor butterfly
//          (p[l] += p[l xor s], s = 32,16,..,1).
//
// Work split: a 256-thread block owns 16 tokens; its 4 wavefronts split the
// experts (NB blocks of 16 experts each).  The fp32 matrix instruction runs on the vector pipe: a chain of
// dependent ones issues every 32 cycles (so one wavefront can fill a SIMD), but every vector instruction
// between two of them adds its own 4 cycles and a dozen more for the change-over.  The reduction is therefore
// built to need almost none:
//   weights: a private fp32 copy that fmoe_set_weights lays out in exactly the per-lane order the
//            instruction consumes; one 16-byte buffer load per four instructions, scalar offsets, a register
//            ring many groups deep;
//   x:       staged through LDS in chunks of 128 k, widened to fp32 and de-interleaved on the way in (eight
//            vector instructions per thread and chunk), so that one 16-byte LDS read feeds four
//            instructions; two LDS buffers and one barrier per chunk, taken while the operands of the
//            chunk's last group already sit in registers, so that the next chunk's first read flies behind
//            that group's instructions.
// Logits meet in LDS, then a wavefront does softmax / top-k for four tokens at once, sixteen lanes each
// (one token at a time over all 64 lanes took 4.6 us a block, this takes 2.0).
// Measured against single-buffered staging with two barriers a chunk and the one-token epilogue (average kernel
// times under the profiler): 8 tokens, d 2048, 64 experts 18.5 -> 13.1 us; 1600 tokens, d 1280 17.3 -> 12.3; 8192
// tokens, d 2048, 128 experts 63.0 -> 49.2; 22016 tokens, d 2048, 64 experts 84.8 -> 74.6; 256 experts, 8 tokens
// 55.3 -> 41.4, 8192 101 -> 83, 22016 278 -> 224.  Bound: the chain itself, 44 cycles per instruction where 32
// are needed (the rest is the staging's vector work and the barrier).

#include <type_traits>

#include "common.h"
#include "prune_dev.h"
#include "tiles.h"

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int TOKB = 16;           // tokens per block
constexpr int KC = 128;            // k per LDS chunk
constexpr int NG = KC / 16;        // groups of four matrix instructions per chunk
constexpr int RS = KC / 4 + 4;     // LDS row stride in floats (rows = kq*16 + token): 16 rows on 16 bank groups
constexpr int XPF = 4;             // chunks of x in flight in registers

__host__ __device__ inline int router_chunks(int d) { return (d + KC - 1) / KC; }

// v of the lane `ROT` places on in the row of 16
template <int ROT>
__device__ __forceinline__ float row_rotate(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + ROT, 0xf, 0xf, false));
}
template <int ROT>
__device__ __forceinline__ int row_rotate(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + ROT, 0xf, 0xf, false);
}
// Over the 16 lanes of a row, the result in every lane.  After the step by 8 all values repeat with period 8,
// so the step by 4 pairs what an exclusive-or by 4 would, and so on: the sum is the xor butterfly 8, 4, 2, 1.
__device__ __forceinline__ float row_sum_butterfly(float v) {
  v = v + row_rotate<8>(v);
  v = v + row_rotate<4>(v);
  v = v + row_rotate<2>(v);
  return v + row_rotate<1>(v);
}
__device__ __forceinline__ float larger(float v, float o) { return (o > v) ? o : v; }
__device__ __forceinline__ float row_max(float v) {
  v = larger(v, row_rotate<8>(v));
  v = larger(v, row_rotate<4>(v));
  v = larger(v, row_rotate<2>(v));
  return larger(v, row_rotate<1>(v));
}
__device__ __forceinline__ int row_min(int v) {
  v = min(v, row_rotate<8>(v));
  v = min(v, row_rotate<4>(v));
  v = min(v, row_rotate<2>(v));
  return min(v, row_rotate<1>(v));
}

__device__ __forceinline__ float exp_fixed(float x) {
  const float kLog2e = 0x1.715476p+0f;
  const float kLn2Hi = 0x1.62e400p-1f;
  const float kLn2Lo = 0x1.7f7d1cp-20f;
  float n = rintf(x * kLog2e);
  float r = fmaf(-n, kLn2Hi, x);
  r = fmaf(-n, kLn2Lo, r);
  float p = 0x1.a01a02p-13f;
  p = fmaf(p, r, 0x1.6c16c2p-10f);
  p = fmaf(p, r, 0x1.111112p-7f);
  p = fmaf(p, r, 0x1.555556p-5f);
  p = fmaf(p, r, 0x1.555556p-3f);
  p = fmaf(p, r, 0.5f);
  p = fmaf(p, r, 1.0f);
  p = fmaf(p, r, 1.0f);
  const bool in = n >= -125.0f;   // not for NaN
  const float scale = __uint_as_float((uint32_t)((int)(in ? n : 0.0f) + 127) << 23);
  return in ? p * scale : 0.0f;
}

// Private router-weight layout: for expert block eb (16 experts) and k group g (16 k), lane l
// holds the float4 { w[eb*16 + l%16][16g + 4j + l/16] : j = 0..3 } at ((eb*G + g)*64 + l).
// Experts >= E and k >= d are zero (a zero product leaves the chain's value unchanged); G covers
// d rounded up to whole 128-wide chunks, so the kernel's loads need no bounds predicate.
template <typename WT>
__global__ void pack_router_kernel(const WT* __restrict__ w, float* __restrict__ wp, int E, int d,
                                   int Eb, int G) {
  const size_t n = (size_t)Eb * G * 256;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    const int j = (int)(i & 3), l = (int)((i >> 2) & 63);
    const size_t eg = i >> 8;
    const int g = (int)(eg % G), eb = (int)(eg / G);
    const int e = eb * 16 + (l & 15), k = 16 * g + 4 * j + (l >> 4);
    wp[i] = (e < E && k < d) ? to_f32(w[(size_t)e * d + k]) : 0.0f;
  }
}

// One thread's share of a chunk of x (16 tokens x 128 k): 16-byte units, widened and de-interleaved into LDS
// rows kq*16 + token, k = 4*step + kq at position step.
template <typename XT> struct XStage;
template <> struct XStage<bf16_t> {
  static constexpr int UNITS = 1;
  static __device__ __forceinline__ int token(int tid, int) { return tid >> 4; }
  static __device__ __forceinline__ int k(int tid, int) { return 8 * (tid & 15); }
  static __device__ __forceinline__ void store(float* xs, int tid, int, u32x4_t v) {
    const int tok = tid >> 4, cu = tid & 15;
    float f[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(v[i] << 16);
      f[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
    }
    // element i of the unit has k = 8cu + i: kq = i%4, step = 2cu + i/4
#pragma unroll
    for (int kq = 0; kq < 4; ++kq)
      *reinterpret_cast<float2*>(&xs[(kq * 16 + tok) * RS + 2 * cu]) = make_float2(f[kq], f[kq + 4]);
  }
};
template <> struct XStage<float> {
  static constexpr int UNITS = 2;
  static __device__ __forceinline__ int token(int tid, int u) { return (tid + u * 256) >> 5; }
  static __device__ __forceinline__ int k(int tid, int) { return 4 * (tid & 31); }
  static __device__ __forceinline__ void store(float* xs, int tid, int u, u32x4_t v) {
    const int tok = token(tid, u), cu = tid & 31;
#pragma unroll
    for (int kq = 0; kq < 4; ++kq) xs[(kq * 16 + tok) * RS + cu] = __uint_as_float(v[kq]);
  }
};

struct fmoe_no_job {};

// Selection-strategy ablation (Sec. 4): which k of a token's k_base highest experts stay active.
struct fmoe_selection {
  int strategy;              // 0 the k highest (the method), 1 k at random, 2 the k lowest
  int k_base;
  unsigned long long seed;
};

// n-th output of the SplitMix64 generator started at `seed` (the key of a candidate position for
// the random strategy)
__device__ __forceinline__ unsigned long long splitmix64_nth(unsigned long long seed, unsigned long long n) {
  unsigned long long z = seed + n * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// R = groups of weights in flight.  (Two token tiles per block, which halve the weight loads, measured the same
// at 22016 tokens / 64 experts and 3 % slower at 8192 / 128.)
// DISPATCH: one block has all tokens and none is dropped, so it goes on to write what the dispatch step would
// (kept list, permutation by expert, GEMM work lists): an expert's rows are the set bits of its token mask.  A
// launch less for a decoding step, where the dispatch kernel took 9 us for a few hundred bytes (8 tokens, 64
// experts: router 13.1 + dispatch 9.3 us, together 19.2, now 17.6; the layer 108.0 -> 102.9 us).
template <typename XT, int NB, int R, bool SEL, bool DISPATCH>
__global__ __launch_bounds__(256) void route_kernel(
    const XT* __restrict__ x, const float* __restrict__ wp, const float* __restrict__ bias,
    const uint8_t* __restrict__ is_visual, int T, int d, int E, int Eb, int k_text,
    int k_visual, int Kmax, int renorm, float* __restrict__ probs, int32_t* __restrict__ topk_idx,
    float* __restrict__ topk_gate, int route_blocks, fmoe_ordinals_job ord, const int32_t* __restrict__ T_dev,
    fmoe_selection selp, std::conditional_t<DISPATCH, fmoe_dispatch_job, fmoe_no_job> job) {
  typedef XStage<XT> XS;
  constexpr int UNITS = XS::UNITS, PER_UNIT = 16 / (int)sizeof(XT);
  constexpr int ES = 4 * NB * 16 + 4;   // row stride of the logits
  constexpr int XS_FLOATS = 2 * 64 * RS, ZS_FLOATS = TOKB * ES;
  __shared__ __align__(16) float smem[XS_FLOATS > ZS_FLOATS ? XS_FLOATS : ZS_FLOATS];   // x chunks, later the logits
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if ((int)blockIdx.x >= route_blocks) {   // rider blocks: per-sequence visual ordinals for the pruning stage
    seq_ordinals_block(is_visual, ord.cu, (int)blockIdx.x - route_blocks, T, ord.vis_ord, ord.vis_tok,
                       ord.seq_nv, reinterpret_cast<int*>(smem));
    return;
  }
  const int t0 = blockIdx.x * TOKB;
  if (T_dev != nullptr) {   // the batch holds fewer tokens than its capacity
    const int Td = *T_dev;
    T = Td < T ? Td : T;
    if (t0 >= T) return;
  }

  f32x4_t acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Loads go through buffer descriptors over the block's token rows and the wavefront's weights: a lane offset
  // that never changes and a scalar one per load.  All indices are clamped (tokens past T re-read the last
  // token, whose logits are then not used; k past d re-reads the end of the row, where the packed weights are
  // zero; chunks past the last re-read it).
  const int nch = router_chunks(d), G = nch * NG;
  const int eb0 = wave * NB < Eb ? wave * NB : Eb - 1;
  const __amdgpu_buffer_rsrc_t w_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wp) + (size_t)eb0 * G * 256, 0, 0xffffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t x_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<XT*>(x) + (size_t)t0 * d, 0, 0xffffffff, 0x00020000);
  uint32_t wbase[NB];   // scalar
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {   // expert blocks past E recompute the last one; never read back
    const int eb = wave * NB + nb < Eb ? wave * NB + nb : Eb - 1;
    wbase[nb] = (uint32_t)(eb - eb0) * (uint32_t)G * 1024u;
  }
  const uint32_t lane16 = (uint32_t)lane * 16u;
  uint32_t xrow[UNITS];
#pragma unroll
  for (int u = 0; u < UNITS; ++u) {
    const int row = XS::token(tid, u), last = T - 1 - t0;
    xrow[u] = (uint32_t)(row < last ? row : last) * (uint32_t)d;
  }
  u32x4_t xbuf[XPF][UNITS];
  f32x4_t wbuf[R][NB];
  auto load_x = [&](int slot, int c) {
    const int k0 = (c < nch ? c : nch - 1) * KC;   // scalar
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      int k = k0 + XS::k(tid, u);
      k = k < d ? k : d - PER_UNIT;
      xbuf[slot][u] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, (xrow[u] + (uint32_t)k) * (uint32_t)sizeof(XT), 0, 0);
    }
  };
  auto load_w = [&](int slot, int g) {
    const uint32_t off = (uint32_t)(g < G ? g : G - 1) * 1024u;   // scalar
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      wbuf[slot][nb] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, lane16, wbase[nb] + off, 0));
  };
  auto store_x = [&](int buf, int slot) {
#pragma unroll
    for (int u = 0; u < UNITS; ++u) XS::store(smem + buf * (64 * RS), tid, u, xbuf[slot][u]);
  };
  f32x4_t xa[2];
  const int xlane = ((lane >> 4) * 16 + (lane & 15)) * RS;
  auto read_x = [&](int o, int buf, int gl) {
    xa[o] = *reinterpret_cast<const f32x4_t*>(&smem[buf * (64 * RS) + xlane + gl * 4]);
  };
  // Four tokens per wavefront side by side, token q of them in lanes 16q .. 16q+15; lane j of a token holds the
  // experts 16r + j, r = 0 .. NR-1.
  constexpr int NR = 4 * NB;
  const int j = lane & 15;
  const int tok = wave * 4 + (lane >> 4);
  const bool tv = (t0 + tok) < T;
  const int t = tv ? t0 + tok : T - 1;
  const bool visual = is_visual[t] != 0;
  const bool biased = bias != nullptr;
  // Chunk c is multiplied while chunk c+1 goes into the other LDS buffer, chunks up to c+XPF and R groups of
  // weights are in flight.
  static_assert(XPF % 2 == 0 && (XPF * NG) % R == 0, "ring indices are compile-time");
#pragma unroll
  for (int u = 0; u < XPF; ++u) load_x(u, u);
#pragma unroll
  for (int r = 0; r < R; ++r) {   // in ring order: the waits in the loop count on it
    load_w(r, r);
    __builtin_amdgcn_sched_barrier(0);
  }
  store_x(0, 0);
  load_x(0, XPF);
  __syncthreads();
  read_x(0, 0, 0);
  for (int c0 = 0; c0 < nch; c0 += XPF) {
#pragma unroll
    for (int u = 0; u < XPF; ++u) {
      const int c = c0 + u;
      if (c >= nch) break;   // uniform
#pragma unroll
      for (int gl = 0; gl < NG; ++gl) {
        const int o = gl & 1, slot = (u * NG + gl) % R;
        if (gl == NG - 1) {
          // every wavefront has its operands of this chunk's last group and has stored its part of the next chunk
          __syncthreads();
          read_x(o ^ 1, (u + 1) & 1, 0);
        } else {
          read_x(o ^ 1, u & 1, gl + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i)   // each chain in ascending k; the chains alternate
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[o][i], wbuf[slot][nb][i], acc[nb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_w(slot, c * NG + gl + R);
        if (gl == 0) {
          store_x((u + 1) & 1, (u + 1) % XPF);
          load_x((u + 1) % XPF, c + 1 + XPF);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // all biases at once, on their way while the logits go through LDS: fetched where they are added, each was a
  // memory latency of its own (8192 tokens, 128 experts 46.4 -> 45.4 us; 1600 tokens, 64 experts 13.3 -> 12.9)
  float bias_r[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) bias_r[r] = biased ? bias[16 * r + j < E ? 16 * r + j : E - 1] : 0.0f;
  __syncthreads();   // the chunks' LDS becomes the logits'

  // accumulator register v of lane l: token 4*(l/16) + v, expert (block)*16 + l%16
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int e = (wave * NB + nb) * 16 + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) smem[(4 * (lane >> 4) + v) * ES + e] = acc[nb][v];
  }
  __syncthreads();

  // Softmax, top-k and gates
  float P[NR];
  float mx = -INFINITY;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const float z = smem[tok * ES + 16 * r + j];   // (past E the last block's logits again)
    const float v = biased ? z + bias_r[r] : z;
    P[r] = 16 * r + j < E ? v : -INFINITY;
    mx = larger(mx, P[r]);
  }
  mx = row_max(mx);
#pragma unroll
  for (int r = 0; r < NR; ++r) P[r] = exp_fixed(P[r] - mx);   // 0 past E, without a branch
  // the sum's order: experts e, e+64, .. one after the other, then the xor butterfly 32, 16, 8, 4, 2, 1
  float part[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    part[r] = 0.0f;
#pragma unroll
    for (int i = 0; i < NB; ++i) part[r] = part[r] + P[r + 4 * i];
  }
  const float sum = row_sum_butterfly((part[0] + part[2]) + (part[1] + part[3]));
  // Inside the fused layer (the launch that also carries the ordinal blocks) the probabilities only feed
  // the window scores, which read visual tokens: text rows are not written.
  const bool store_row = probs != nullptr && tv && (ord.cu == nullptr || visual);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int e = 16 * r + j;
    P[r] = (e < E) ? P[r] / sum : -1.0f;   // -1 ranks below every probability
    if (store_row && e < E) probs[(size_t)t * E + e] = P[r];
  }

  // Top-k as k rounds of "take the largest remaining probability" (ties: lowest expert index), which
  // yields the list in the order (probability desc, index asc) directly; lane j keeps entry j of it.
  const int k = visual ? k_visual : k_text;
  // with a selection strategy a token with k < k_base first lists its k_base candidates
  const int kc = (SEL && k < selp.k_base) ? selp.k_base : k;
  const int rounds = (SEL && selp.k_base > Kmax) ? selp.k_base : Kmax;
  float den = 0.0f;
  int my_e = -1;
  float my_p = 0.0f;
  for (int round = 0; round < rounds; ++round) {
    float v = P[0];
#pragma unroll
    for (int r = 1; r < NR; ++r) v = larger(v, P[r]);
    const float m = row_max(v);
    int e = 0x7fff;
#pragma unroll
    for (int r = NR - 1; r >= 0; --r) e = (P[r] == m) ? 16 * r + j : e;
    e = row_min(e);
    const bool active = round < kc;
    if (active && j == round) {
      my_e = e < E ? e : -1;   // -1: a row of NaN has no largest entry
      my_p = m;
    }
    den = den + (active ? m : 0.0f);   // list order, sequential (Eq.5)
#pragma unroll
    for (int r = 0; r < NR; ++r) P[r] = (16 * r + j == e) ? -2.0f : P[r];
  }
  int pos = j < kc ? j : -1;   // place of this lane's entry in the token's list, -1: not in it
  if constexpr (SEL) {
    unsigned int mask = 0u;   // kept candidate positions
    if (selp.strategy == 1) {
      // random strategy: lane j holds the key of candidate position j; a position is kept when fewer
      // than k keys of its token are smaller (ties: lower position)
      const unsigned long long key = splitmix64_nth(selp.seed, (unsigned long long)t * 16ull + (unsigned long long)j + 1ull);
      int rank = 0;
      for (int o = 0; o < 16; ++o) {
        const int src = (lane & 48) + o;
        const unsigned int lo = (unsigned int)__shfl((int)(unsigned int)key, src, 64);
        const unsigned int hi = (unsigned int)__shfl((int)(unsigned int)(key >> 32), src, 64);
        const unsigned long long ok = ((unsigned long long)hi << 32) | lo;
        rank += (o < selp.k_base && (ok < key || (ok == key && o < j))) ? 1 : 0;
      }
      const unsigned long long all = __ballot(j < selp.k_base && rank < k);
      mask = (unsigned int)(all >> (lane & 48)) & 0xffffu;
    } else if (k < selp.k_base) {
      mask = ((1u << k) - 1u) << (selp.strategy == 2 ? selp.k_base - k : 0);
    }
    float d2 = 0.0f;   // Eq.5 over the kept experts, in list order
    for (int p = 0; p < selp.k_base; ++p) {
      const float v = __shfl(my_p, (lane & 48) + p, 64);
      if ((mask >> p) & 1u) d2 = d2 + v;
    }
    if (k < selp.k_base) {   // otherwise not reduced: the list stands
      pos = (pos >= 0 && ((mask >> pos) & 1u)) ? __popc(mask & ((1u << pos) - 1u)) : -1;
      den = d2;
    }
  }
  if (tv) {
    int32_t* oi = topk_idx + (size_t)t * Kmax;
    float* og = topk_gate + (size_t)t * Kmax;
    if (pos >= 0) {
      oi[pos] = my_e;
      og[pos] = renorm ? my_p / den : my_p;
    }
    if (j < Kmax && j >= k) {   // unused tail of the list
      oi[j] = -1;
      og[j] = 0.0f;
    }
  }

  if constexpr (DISPATCH) {
    static_assert(FMOE_ROUTE_DISPATCH_TOKENS <= TOKB, "one block has all tokens");
    static_assert(TOKB <= 31, "the token masks are ints");
    int* s_mask = reinterpret_cast<int*>(smem);          // [FMOE_MAX_EXPERTS] tokens of the expert
    int* s_off = s_mask + FMOE_MAX_EXPERTS;              // [FMOE_MAX_EXPERTS + 1] exclusive scan of their numbers
    int* scratch = s_off + FMOE_MAX_EXPERTS + 2;         // 8-byte aligned
    static_assert((2 * FMOE_MAX_EXPERTS + 2 + FMOE_TILES_SCRATCH) * 4 <= sizeof(smem), "fits where x and the logits were");
    static_assert(FMOE_MAX_EXPERTS == 256, "a mask per thread");
    __syncthreads();   // the logits have been read
    s_mask[tid] = 0;
    __syncthreads();
    const bool listed = tv && pos >= 0 && my_e >= 0;
    if (listed) atomicOr(&s_mask[my_e], 1 << tok);
    __syncthreads();
    if (wave == 0) {   // four experts per lane
      int c[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c[q] = __popc(s_mask[4 * lane + q]);
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
    if (tv) {
      if (listed) {
        const int row = s_off[my_e] + __popc(s_mask[my_e] & ((1 << tok) - 1));
        if (row < job.row_cap) job.perm_src[row] = tok;
        job.inv_perm[tok * Kmax + pos] = row;
      } else if (j < Kmax) {
        job.inv_perm[tok * Kmax + j] = -1;
      }
      if (j == 0) {
        job.kept_idx[tok] = tok;
        if (job.is_visual_out != nullptr) job.is_visual_out[tok] = is_visual[tok];
      }
    }
    if (tid <= E) job.expert_offsets[tid] = s_off[tid];
    if (tid == 0 && E == FMOE_MAX_EXPERTS) job.expert_offsets[E] = s_off[E];
    for (int b = tid; b <= job.B; b += 256) job.new_cu[b] = clampi(job.cu[b], 0, T);
    fmoe_build_tiles<false>(s_off, E, job.row_cap, T, job.n_shared, job.geom.bm, job.geom.run, job.geom.tile_cap,
                            job.geom.cols1, job.geom.scols1, job.tiles1, job.tiles2, job.tile_count, scratch);
  }
}

template <typename XT, int NB, int R>
int launch_route_t(const fmoe_ctx* ctx, const void* x, const uint8_t* is_visual, int T, float* probs,
                   int32_t* topk_idx, float* topk_gate, const fmoe_ordinals_job& ord, hipStream_t stream,
                   const int32_t* T_dev, const fmoe_dispatch_job* dispatch) {
  const int d = ctx->cfg.d_model, E = ctx->cfg.n_experts;
  const int Eb = (E + 15) / 16;
  const int grid = (T + TOKB - 1) / TOKB;
  fmoe_prof_scope prof(ctx, SLOT_ROUTE, stream);
  const int riders = ord.cu != nullptr ? ord.B : 0;
  const fmoe_selection selp{ctx->sel_strategy, ctx->sel_k_base, ctx->sel_seed};
#define FMOE_ROUTE_LAUNCH(SEL, DISPATCH, JOB)                                                                   \
  hipLaunchKernelGGL((route_kernel<XT, NB, R, SEL, DISPATCH>), dim3(grid + riders), dim3(256), 0, stream,       \
                     static_cast<const XT*>(x), static_cast<const float*>(ctx->router_wp),                      \
                     ctx->router_bias, is_visual, T, d, E, Eb, ctx->cfg.k_text, ctx->cfg.k_visual, ctx->kmax,   \
                     ctx->cfg.renormalize, probs, topk_idx, topk_gate, grid, ord, T_dev, selp, JOB)
  if (dispatch != nullptr) {
    if (T > FMOE_ROUTE_DISPATCH_TOKENS || ctx->sel_strategy != 0 || T_dev != nullptr || riders != 0)
      return fmoe_fail(FMOE_ERR_INVALID_ARG, "router: %d tokens cannot be dispatched in its launch", T);
    FMOE_ROUTE_LAUNCH(false, true, *dispatch);
  } else if (ctx->sel_strategy != 0) {
    FMOE_ROUTE_LAUNCH(true, false, fmoe_no_job{});
  } else {
    FMOE_ROUTE_LAUNCH(false, false, fmoe_no_job{});
  }
#undef FMOE_ROUTE_LAUNCH
  FMOE_HIP_CHECK(hipGetLastError());
  return FMOE_OK;
}

template <typename XT>
int launch_route_x(const fmoe_ctx* ctx, const void* x, const uint8_t* is_visual, int T, float* probs,
                   int32_t* topk_idx, float* topk_gate, const fmoe_ordinals_job& ord, hipStream_t stream,
                   const int32_t* T_dev, const fmoe_dispatch_job* dispatch) {
  const int E = ctx->cfg.n_experts;
  // enough weight groups in flight to cover some 2000 cycles at 128 cycles per group and expert block
  if (E <= 64) return launch_route_t<XT, 1, 16>(ctx, x, is_visual, T, probs, topk_idx, topk_gate, ord, stream, T_dev, dispatch);
  if (E <= 128) return launch_route_t<XT, 2, 8>(ctx, x, is_visual, T, probs, topk_idx, topk_gate, ord, stream, T_dev, dispatch);
  return launch_route_t<XT, 4, 4>(ctx, x, is_visual, T, probs, topk_idx, topk_gate, ord, stream, T_dev, dispatch);
}

}  // namespace

size_t router_pack_floats(const fmoe_ctx* ctx) {
  const int Eb = (ctx->cfg.n_experts + 15) / 16, G = NG * router_chunks(ctx->cfg.d_model);
  return (size_t)Eb * G * 256;
}

int launch_pack_router(const fmoe_ctx* ctx, const void* router_w, float* wp, hipStream_t stream) {
  const int E = ctx->cfg.n_experts, d = ctx->cfg.d_model;
  const int Eb = (E + 15) / 16, G = NG * router_chunks(d);
  const size_t n = router_pack_floats(ctx);
  const int grid = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  if (ctx->cfg.dtype == FMOE_BF16)
    hipLaunchKernelGGL(pack_router_kernel<bf16_t>, dim3(grid), dim3(256), 0, stream,
                       static_cast<const bf16_t*>(router_w), wp, E, d, Eb, G);
  else
    hipLaunchKernelGGL(pack_router_kernel<float>, dim3(grid), dim3(256), 0, stream,
                       static_cast<const float*>(router_w), wp, E, d, Eb, G);
  FMOE_HIP_CHECK(hipGetLastError());
  return FMOE_OK;
}

int launch_route(const fmoe_ctx* ctx, const void* x, const uint8_t* is_visual, int T, float* probs,
                 int32_t* topk_idx, float* topk_gate, const fmoe_ordinals_job& ord, hipStream_t stream,
                 const int32_t* T_dev, const fmoe_dispatch_job* dispatch) {
  if (T == 0) return FMOE_OK;
  if (ctx->cfg.dtype == FMOE_BF16)
    return launch_route_x<bf16_t>(ctx, x, is_visual, T, probs, topk_idx, topk_gate, ord, stream, T_dev, dispatch);
  return launch_route_x<float>(ctx, x, is_visual, T, probs, topk_idx, topk_gate, ord, stream, T_dev, dispatch);
}
