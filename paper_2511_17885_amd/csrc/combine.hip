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
  static __device__ __forceinline__ void load(const bf16_t* p, float* f) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
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
template <typename T, int KM>
__global__ __launch_bounds__(256, 8) void combine_kernel(
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
                      const void* residual, void* out, hipStream_t stream) {
  if constexpr (KM < FMOE_MAX_TOPK) {
    if (ctx->kmax > KM)
      return launch_combine_t<T, KM + 1>(ctx, y, y_shared, inv_perm, topk_gate, kept_idx, n_cap, n_dev, residual, out, stream);
  }
  hipLaunchKernelGGL((combine_kernel<T, KM>), dim3(n_cap), dim3(256), 0, stream, static_cast<const T*>(y),
                     static_cast<const T*>(y_shared), inv_perm, topk_gate, kept_idx, n_cap, n_dev, n_cap * KM,
                     ctx->cfg.d_model, ctx->cfg.n_shared, static_cast<const T*>(residual), static_cast<T*>(out));
}

}  // namespace

int launch_combine(const fmoe_ctx* ctx, const void* y, const void* y_shared, const int32_t* inv_perm,
                   const float* topk_gate, const int32_t* kept_idx, int n_cap, const int32_t* n_dev,
                   const void* residual, void* out, hipStream_t stream) {
  if (n_cap == 0) return FMOE_OK;
  fmoe_prof_scope prof(ctx, SLOT_COMBINE, stream);
  if (ctx->cfg.dtype == FMOE_BF16)
    launch_combine_t<bf16_t, 0>(ctx, y, y_shared, inv_perm, topk_gate, kept_idx, n_cap, n_dev, residual, out, stream);
  else
    launch_combine_t<float, 0>(ctx, y, y_shared, inv_perm, topk_gate, kept_idx, n_cap, n_dev, residual, out, stream);
  FMOE_HIP_CHECK(hipGetLastError());
  return FMOE_OK;
}
