// hmoe_combine: the gate-weighted sum of Eq. (1) in gather form,
//   y[t] = sum_{j<K} w[t,j] * o_perm[inv_perm[t*K+j]] (+ o_shared[t]),
// j ascending then the shared term, fp32 accumulation, one rounding.  No atomics: every output
// element is produced by one lane, so results do not depend on scheduling.
// Also: hmoe_router_logits (x . W_g), the small GEMM in front of the router.
#include "router_body.h"

namespace hmoe {

// One 16-byte piece of one token per lane.  All rows of a token are requested before the first is used (K at a time, the
// number of experts per token where that is at most 8): a loop that waits for each row is as many trips to memory as the
// token has experts, which is most of the time of a decode batch.  The row numbers and weights are the same for the whole
// block and come through the scalar cache, without a barrier.  Decode layer of 64 experts, top 6, one token: 40.8 -> 39.8 us;
// 8 experts in 4 bits, top 2: 58.1 -> 57.4.
__device__ __forceinline__ void combine_add(float (&acc)[8], const uint4& v, float w) {
  const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc[2 * i] += w * __uint_as_float(u[i] << 16);
    acc[2 * i + 1] += w * __uint_as_float(u[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void combine_add(float (&acc)[4], const float4& v, float w) {
  acc[0] += w * v.x;
  acc[1] += w * v.y;
  acc[2] += w * v.z;
  acc[3] += w * v.w;
}
__device__ __forceinline__ void combine_store(uint4* y, const float (&acc)[8]) {
  *y = make_uint4((uint32_t)f32_to_bf16(acc[0]) | ((uint32_t)f32_to_bf16(acc[1]) << 16),
                  (uint32_t)f32_to_bf16(acc[2]) | ((uint32_t)f32_to_bf16(acc[3]) << 16),
                  (uint32_t)f32_to_bf16(acc[4]) | ((uint32_t)f32_to_bf16(acc[5]) << 16),
                  (uint32_t)f32_to_bf16(acc[6]) | ((uint32_t)f32_to_bf16(acc[7]) << 16));
}
__device__ __forceinline__ void combine_store(float4* y, const float (&acc)[4]) { *y = make_float4(acc[0], acc[1], acc[2], acc[3]); }

// VEC: 16 bytes, N elements.  K: experts per token (exact up to 8), or 8 at a time of top_k.  STREAM: non-temporal loads.
template <class VEC, int N, int K, bool EXACT, bool SHARED, bool STREAM>
__global__ __launch_bounds__(256) void combine_kernel(const VEC* __restrict__ o_perm, const int32_t* __restrict__ inv_perm,
                                                      const float* __restrict__ topk_w, const VEC* __restrict__ o_shared,
                                                      int top_k, int row_vec, VEC* __restrict__ y) {
  const long t = blockIdx.x;
  const int c = blockIdx.y * blockDim.x + threadIdx.x;
  if (c >= row_vec) return;
  const int32_t* rows = inv_perm + t * (EXACT ? K : top_k);
  const float* w = topk_w + t * (EXACT ? K : top_k);
  VEC shared = {};
  if (SHARED) shared = o_shared[t * row_vec + c];
  float acc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = 0.0f;
  for (int j0 = 0; j0 < (EXACT ? K : top_k); j0 += K) {
    VEC v[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const VEC* row = o_perm + (long)rows[EXACT ? j : min(j0 + j, top_k - 1)] * row_vec + c;
      v[j] = STREAM ? __builtin_bit_cast(VEC, __builtin_nontemporal_load((const u32x4*)row)) : *row;
    }
#pragma unroll
    for (int j = 0; j < K; ++j)
      if (EXACT || j0 + j < top_k) combine_add(acc, v[j], w[EXACT ? j : j0 + j]);
  }
  if (SHARED) combine_add(acc, shared, 1.0f);
  combine_store(&y[t * row_vec + c], acc);
}

template <class VEC, int N>
static void launch_combine(const VEC* o_perm, const int32_t* inv_perm, const float* topk_w, const VEC* o_shared, int T, int top_k,
                           int row_vec, VEC* y, hipStream_t s) {
  // A few tokens: blocks of one wave, spread over the CUs.
  const int threads = T <= 64 ? 64 : 256;
  const dim3 grid((unsigned)T, (unsigned)((row_vec + threads - 1) / threads));
  // Inputs that no L2 holds: non-temporal loads, 5.1 -> 6.0 TB/s (6 rows of 2048 and the shared row, 16384 tokens 106 -> 90 us,
  // 4000 tokens 24.4 -> 22.2; 8 of 3584, 2048 tokens 28.3 -> 25.0).  Smaller ones are still in the caches the down projection
  // wrote them to (1003 tokens of the first 6.1 against 6.5 us).
  const bool stream = (long)T * (top_k + 1) * row_vec * 16 >= 64l << 20;
  auto launch = [&](auto with, auto without, auto with_stream, auto without_stream) {
    const auto kernel = o_shared ? (stream ? with_stream : with) : (stream ? without_stream : without);
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, o_perm, inv_perm, topk_w, o_shared, top_k, row_vec, y);
  };
#define HMOE_COMBINE(K, EXACT)                                                                                    \
  launch(&combine_kernel<VEC, N, K, EXACT, true, false>, &combine_kernel<VEC, N, K, EXACT, false, false>,          \
         &combine_kernel<VEC, N, K, EXACT, true, true>, &combine_kernel<VEC, N, K, EXACT, false, true>)
  switch (top_k) {
    case 1: HMOE_COMBINE(1, true); break;
    case 2: HMOE_COMBINE(2, true); break;
    case 3: HMOE_COMBINE(3, true); break;
    case 4: HMOE_COMBINE(4, true); break;
    case 5: HMOE_COMBINE(5, true); break;
    case 6: HMOE_COMBINE(6, true); break;
    case 7: HMOE_COMBINE(7, true); break;
    case 8: HMOE_COMBINE(8, true); break;
    default: HMOE_COMBINE(8, false); break;
  }
#undef HMOE_COMBINE
}

// fp32 rows that are no multiple of 16 bytes
__global__ __launch_bounds__(256) void combine_f32_kernel(const float* __restrict__ o_perm,
                                                          const int32_t* __restrict__ inv_perm,
                                                          const float* __restrict__ topk_w,
                                                          const float* __restrict__ o_shared, int top_k, int hidden,
                                                          float* __restrict__ y) {
  const long t = blockIdx.x;
  for (int c = threadIdx.x; c < hidden; c += blockDim.x) {
    float acc = 0.0f;
    for (int j = 0; j < top_k; ++j)
      acc += topk_w[t * top_k + j] * o_perm[(long)inv_perm[t * top_k + j] * hidden + c];
    if (o_shared) acc += o_shared[t * hidden + c];
    y[t * hidden + c] = acc;
  }
}

// logits[t, e] = sum_h x[t,h] * w_g[e,h], fp32 accumulate.
// fp32 layers: one wavefront per (token, expert) dot product.
__global__ __launch_bounds__(256) void router_logits_f32_kernel(const float* __restrict__ x, const float* __restrict__ w_g,
                                                                int n_tokens, int n_experts, int hidden,
                                                                float* __restrict__ logits) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const long pair = (long)blockIdx.x * 4 + wave;
  if (pair >= (long)n_tokens * n_experts) return;
  const long t = pair / n_experts;
  const int e = (int)(pair % n_experts);
  const float* xr = x + t * hidden;
  const float* wr = w_g + (long)e * hidden;
  float acc = 0.0f;
  for (int h = lane; h < hidden; h += 64) acc = fmaf(xr[h], wr[h], acc);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) logits[pair] = acc;
}

// bf16 layers: see router_body.h
template <class SHAPE>
__global__ __launch_bounds__(SHAPE::THREADS, SHAPE::WAVES_PER_SIMD) void router_logits_bf16_kernel(const bf16_t* __restrict__ x,
                                                                            const bf16_t* __restrict__ w_g, int n_tokens,
                                                                            int n_experts, int hidden,
                                                                            float* __restrict__ logits, int tokens_per_block) {
  __shared__ float red[SHAPE::RED];
  router_logits_block<SHAPE>(x, w_g, n_tokens, n_experts, hidden, logits, tokens_per_block, red, nullptr, n_experts);
}

// A decode batch: 16 experts per block, so that a router of many is read through several CUs (one block reads it at about 15
// bytes per clock).  With the routing in the FFN's first launch, against one block that computes, routes and ranks (layer, us):
// 64 experts of 2048 x 1408, top 6, 1 token 44.1 -> 37.9; 90 of 1024 x 512, top 8, 2 tokens 32.3 -> 26.1; 24 of 4096 x 1024, top
// 2, 3 tokens 45.3 -> 41.5; 8 of 4096 x 14336, top 2, 8 tokens 381.9 -> 381.1.
constexpr int ROUTER_SPLIT_EXPERTS = 16;
__global__ __launch_bounds__(1024) void router_logits_bf16_split_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w_g,
                                                                        int n_tokens, int n_experts, int hidden,
                                                                        float* __restrict__ logits) {
  typedef RouterShape<1, 1, 16, 16> SHAPE;
  static_assert(SHAPE::EXPERT_FRAGS * 16 == ROUTER_SPLIT_EXPERTS && SHAPE::THREADS == 1024, "");
  __shared__ float red[SHAPE::RED];
  const int e0 = blockIdx.y * ROUTER_SPLIT_EXPERTS;
  router_logits_block<SHAPE>(x, w_g + (long)e0 * hidden, n_tokens, min(n_experts - e0, ROUTER_SPLIT_EXPERTS), hidden, logits + e0, 16, red,
                             nullptr, n_experts);
}

}  // namespace hmoe

extern "C" int32_t hmoe_combine(const hmoe_layer_desc* desc, const void* o_perm, const int32_t* inv_perm,
                                const float* topk_w, const void* o_shared, int32_t T, void* y, void* stream) {
  using namespace hmoe;
  int rc = check_desc(desc);
  if (rc != HMOE_OK) return rc;
  if (T < 0) return HMOE_ERR_INVALID_ARG;
  if (T == 0) return HMOE_OK;
  if (!o_perm || !inv_perm || !topk_w || !y) return HMOE_ERR_INVALID_ARG;
  if (!aligned16(o_perm) || !aligned16(y) || (o_shared && !aligned16(o_shared))) return HMOE_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  if (desc->dtype != HMOE_F32) {
    if (desc->hidden % 8 != 0) return HMOE_ERR_UNSUPPORTED;
    launch_combine<uint4, 8>((const uint4*)o_perm, inv_perm, topk_w, (const uint4*)o_shared, T, desc->top_k, desc->hidden / 8, (uint4*)y, s);
  } else if (desc->hidden % 4 == 0) {
    launch_combine<float4, 4>((const float4*)o_perm, inv_perm, topk_w, (const float4*)o_shared, T, desc->top_k, desc->hidden / 4, (float4*)y, s);
  } else {
    hipLaunchKernelGGL(combine_f32_kernel, dim3((unsigned)T), dim3(256), 0, s, (const float*)o_perm, inv_perm, topk_w,
                       (const float*)o_shared, desc->top_k, desc->hidden, (float*)y);
  }
  HMOE_HIP(hipGetLastError());
  return HMOE_OK;
}

extern "C" int32_t hmoe_router_logits(const hmoe_layer_desc* desc, const void* x, const void* w_g, int32_t T,
                                      float* logits, void* stream) {
  using namespace hmoe;
  int rc = check_desc(desc);
  if (rc != HMOE_OK) return rc;
  if (T < 0) return HMOE_ERR_INVALID_ARG;
  if (T == 0) return HMOE_OK;
  if (!x || !w_g || !logits) return HMOE_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const int E = desc->n_experts, H = desc->hidden;
  if (desc->dtype != HMOE_F32) {
    if (H % 16 != 0) return HMOE_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(w_g)) return HMOE_ERR_INVALID_ARG;
    const int tpb = router_tokens_per_block(T);
    const dim3 grid((unsigned)((T + tpb - 1) / tpb));
#define HMOE_LAUNCH_LOGITS(G, VPL, MA, NF, KS, NW)                                                                 \
  hipLaunchKernelGGL((router_logits_bf16_kernel<RouterShape<MA, NF, KS, NW>>), grid, dim3(64 * NW), 0, s, (const bf16_t*)x, \
                     (const bf16_t*)w_g, T, E, H, logits, tpb)
    if (T <= ROUTER_SMALL_T)
      hipLaunchKernelGGL(router_logits_bf16_split_kernel, dim3(1, (unsigned)((E + ROUTER_SPLIT_EXPERTS - 1) / ROUTER_SPLIT_EXPERTS)),
                         dim3(1024), 0, s, (const bf16_t*)x, (const bf16_t*)w_g, T, E, H, logits);
    else HMOE_ROUTER_SHAPES_MANY(E, tpb, HMOE_LAUNCH_LOGITS);
#undef HMOE_LAUNCH_LOGITS
  } else {
    const long pairs = (long)T * E;
    hipLaunchKernelGGL(router_logits_f32_kernel, dim3((unsigned)((pairs + 3) / 4)), dim3(256), 0, s, (const float*)x,
                       (const float*)w_g, T, E, H, logits);
  }
  HMOE_HIP(hipGetLastError());
  return HMOE_OK;
}
