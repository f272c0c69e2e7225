// Gate-weighted un-permute / combine (Eq.4):
//   out[p] = (residual[t]) + sum_i y_shared[i][p] + sum_s gate[t,s] * y[inv_perm[p,s]],   t = kept_idx[p]
// A pure bandwidth kernel: one block per kept token, 16-byte loads of every contributing row,
// fp32 accumulation in the fixed order residual, shared, slot 0, 1, ... and a single rounding to
// the storage type, so the result does not depend on scheduling.

#include "common.h"

namespace {

template <typename T> struct Vec;
template <> struct Vec<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void load(const bf16_t* p, float* f) { widen(*reinterpret_cast<const uint4*>(p), f); }
  static __device__ __forceinline__ void widen(uint4 v, float* f) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float* f) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = (uint32_t)f32_to_bf16(f[2 * i]) | ((uint32_t)f32_to_bf16(f[2 * i + 1]) << 16);
    *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
  }
};
template <> struct Vec<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void load(const float* p, float* f) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  }
  static __device__ __forceinline__ void widen(uint4 v, float* f) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
  }
  static __device__ __forceinline__ void store(float* p, const float* f) {
    *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
  }
};

// A small batch is a chain of memory latencies, so the block's indices are fetched in two steps, by scalar
// loads that depend on nothing but the step before: the count, the token and the rows of its slots, then the
// gates (with the first of the data).  KM is the number of slots itself, so that a step is one or two wide
// scalar loads; with arrays of eight or sixteen and a load per entry the scalar cache was the bound of narrow
// rows (22016 tokens of d 128, two slots: 24.9 us, now 11.0; 13.1 through LDS, one thread a slot, behind a
// barrier).  Wavefronts without columns leave at once.  Eight blocks a CU (what the scalar registers of sixteen
// slots would not allow): 1600 tokens of d 2048 in fp32, sixteen slots, 43.8 -> 38.1 us.  8 tokens, d 2048, eight
// slots, through LDS and now: 4.4 -> 4.0 us; 22016 tokens, d 2048, six slots, two shared experts: 165 us both,
// 5.5 TB/s, which is what a large copy reaches.
// TOGETHER: all rows of a token on their way before the first is added (a row that does not count is not asked for:
// reading something else in its place took 10 to 20 % where half of the slots are empty).  Otherwise a wavefront
// waits for each row before it asks for the next (the test for a row that counts stands between), and only the other
// wavefronts of the CU keep the memory busy: with eight to a SIMD and tens of megabytes they do as well.
// The line is drawn at the size of one row set (tokens x d; where the device holds their number, n_expected: what the
// retention leaves, or half of the capacity for a caller who gives none).  Inside a layer, bf16, separate / together,
// us: six slots and two shared experts, d 1280, half of the slots empty 2457 tokens (6 MB) 13.0 / 11.4, 4915 22.1 / 18.6,
// 8192 31.0 / 28.1, 12288 (30 MB) 44.0 / 42.0, none empty 17.8 / 14.8, 29.2 / 25.5, 41.4 / 40.4, 61.3 / 57.9; d 2048,
// half of them empty 2304 (9 MB) 18.8 / 15.8, 3840 24.4 / 23.6, 7680 (30 MB) 43.4 / 44.0, 11520 62.2 / 62.6; a quarter of
// 8000 tokens kept, 128 experts, eight slots 16.6 / 14.0.  One or two fp32 rows a token are nothing to gather: 8192 of d 128
// (4 MB) 5.1 / 5.5, one token 2.8 / 3.0.
constexpr size_t COMBINE_TOGETHER_BYTES = 32u << 20;
template <typename T, int KM, bool TOGETHER>
__global__ __launch_bounds__(256, TOGETHER ? 4 : 8) void combine_kernel(
    const T* __restrict__ y, const T* __restrict__ y_shared, const int32_t* __restrict__ inv_perm,
    const float* __restrict__ topk_gate, const int32_t* __restrict__ kept_idx, int n_cap,
    const int32_t* __restrict__ n_dev, int row_cap, int d, int n_shared, const T* __restrict__ residual,
    T* __restrict__ out) {
  constexpr int N = Vec<T>::N;
  if ((int)(threadIdx.x & ~63u) * N >= d) return;   // uniform over the wavefront
  const int p = blockIdx.x;
  int rows[KM > 0 ? KM : 1];
#pragma unroll
  for (int s = 0; s < KM; ++s) rows[s] = inv_perm[(size_t)p * KM + s];
  const int t = kept_idx ? kept_idx[p] : p;
  if (p >= resolve_count(n_cap, n_dev)) return;
  float gates[KM > 0 ? KM : 1];
#pragma unroll
  for (int s = 0; s < KM; ++s) gates[s] = topk_gate[(size_t)t * KM + s];
  for (int c = threadIdx.x * N; c < d; c += 256 * N) {
    float acc[N], v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.0f;
    if constexpr (TOGETHER) {
      uint4 vr = make_uint4(0u, 0u, 0u, 0u), vs[2] = {vr, vr}, vk[KM > 0 ? KM : 1];
      if (residual) vr = *reinterpret_cast<const uint4*>(residual + (size_t)t * d + c);
      if (y_shared) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
          vs[s] = *reinterpret_cast<const uint4*>(y_shared + ((size_t)(s < n_shared ? s : 0) * n_cap + p) * d + c);
      }
#pragma unroll
      for (int s = 0; s < KM; ++s)
        if (rows[s] >= 0 && rows[s] < row_cap)   // uniform
          vk[s] = *reinterpret_cast<const uint4*>(y + (size_t)rows[s] * d + c);
      if (residual) Vec<T>::widen(vr, acc);
      if (y_shared) {
        for (int s = 0; s < n_shared; ++s) {
          if (s < 2) Vec<T>::widen(vs[s & 1], v);
          else Vec<T>::load(y_shared + ((size_t)s * n_cap + p) * d + c, v);
#pragma unroll
          for (int i = 0; i < N; ++i) acc[i] += v[i];
        }
      }
#pragma unroll
      for (int s = 0; s < KM; ++s) {
        if (rows[s] < 0 || rows[s] >= row_cap) continue;   // uniform
        Vec<T>::widen(vk[s], v);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = fmaf(gates[s], v[i], acc[i]);
      }
      Vec<T>::store(out + (size_t)p * d + c, acc);
      continue;
    }
    if (residual) {
      Vec<T>::load(residual + (size_t)t * d + c, v);
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] = v[i];
    }
    if (y_shared) {
      for (int s = 0; s < n_shared; ++s) {   // first sum of Eq.4, in expert order
        Vec<T>::load(y_shared + ((size_t)s * n_cap + p) * d + c, v);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] += v[i];
      }
    }
#pragma unroll
    for (int s = 0; s < KM; ++s) {
      const int r = rows[s];
      if (r < 0 || r >= row_cap) continue;   // uniform
      Vec<T>::load(y + (size_t)r * d + c, v);
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] = fmaf(gates[s], v[i], acc[i]);
    }
    Vec<T>::store(out + (size_t)p * d + c, acc);
  }
}

template <typename T, int KM>
void launch_combine_t(const fmoe_ctx* ctx, const void* y, const void* y_shared, const int32_t* inv_perm,
                      const float* topk_gate, const int32_t* kept_idx, int n_cap, const int32_t* n_dev,
                      int n_expected, const void* residual, void* out, hipStream_t stream) {
  if constexpr (KM < FMOE_MAX_TOPK) {
    if (ctx->kmax > KM)
      return launch_combine_t<T, KM + 1>(ctx, y, y_shared, inv_perm, topk_gate, kept_idx, n_cap, n_dev, n_expected, residual,
                                         out, stream);
  }
#define FMOE_COMBINE_LAUNCH(TOGETHER)                                                                            \
  hipLaunchKernelGGL((combine_kernel<T, KM, TOGETHER>), dim3(n_cap), dim3(256), 0, stream, static_cast<const T*>(y), \
                     static_cast<const T*>(y_shared), inv_perm, topk_gate, kept_idx, n_cap, n_dev, n_cap * KM,       \
                     ctx->cfg.d_model, ctx->cfg.n_shared, static_cast<const T*>(residual), static_cast<T*>(out))
  const size_t bytes = (size_t)n_expected * ctx->cfg.d_model * sizeof(T);
  const bool few = sizeof(T) == 4 && KM <= 2 && y_shared == nullptr;
  if (bytes <= COMBINE_TOGETHER_BYTES && !few) FMOE_COMBINE_LAUNCH(true);
  else FMOE_COMBINE_LAUNCH(false);
#undef FMOE_COMBINE_LAUNCH
}

}  // namespace

int launch_combine(const fmoe_ctx* ctx, const void* y, const void* y_shared, const int32_t* inv_perm,
                   const float* topk_gate, const int32_t* kept_idx, int n_cap, const int32_t* n_dev,
                   int n_expected, const void* residual, void* out, hipStream_t stream) {
  if (n_cap == 0) return FMOE_OK;
  fmoe_prof_scope prof(ctx, SLOT_COMBINE, stream);
  if (ctx->cfg.dtype == FMOE_BF16)
    launch_combine_t<bf16_t, 0>(ctx, y, y_shared, inv_perm, topk_gate, kept_idx, n_cap, n_dev, n_expected, residual, out, stream);
  else
    launch_combine_t<float, 0>(ctx, y, y_shared, inv_perm, topk_gate, kept_idx, n_cap, n_dev, n_expected, residual, out, stream);
  FMOE_HIP_CHECK(hipGetLastError());
  return FMOE_OK;
}
