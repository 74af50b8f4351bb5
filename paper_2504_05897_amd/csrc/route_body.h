// Device-side routing of one token by one lane group; shared by hmoe_route and the fused
// small-batch front end.
#pragma once

#include "common.h"

namespace hmoe {

// A logit as an unsigned integer of the same order (+0 and -0 alike), and back.  0 is below every finite logit.
__device__ __forceinline__ uint32_t logit_key(float v) {
  const uint32_t u = __float_as_uint(v + 0.0f);  // -0 becomes +0
  return u ^ ((uint32_t)((int)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_logit(uint32_t k) {
  return __uint_as_float(k ^ (~(uint32_t)((int)k >> 31) | 0x80000000u));
}

// Largest value of a group of G lanes (aligned, a power of two from 8 to 64), in every lane of the group.
template <int CTRL>
__device__ __forceinline__ uint32_t max_with_dpp(uint32_t v) {
  const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
  return v > o ? v : o;
}
template <int G>
__device__ __forceinline__ uint32_t group_max(uint32_t v) {
  v = max_with_dpp<0xB1>(v);                       // quad_perm [1,0,3,2]
  v = max_with_dpp<0x4E>(v);                       // quad_perm [2,3,0,1]
  v = max_with_dpp<0x141>(v);                      // row_half_mirror: the other quad of eight lanes
  if constexpr (G >= 16) v = max_with_dpp<0x140>(v);  // row_mirror: the other eight lanes of a row
  if constexpr (G >= 32) {                         // the other row of a half, then the other half
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = p[0] > p[1] ? p[0] : p[1];
  }
  if constexpr (G >= 64) {
    const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = p[0] > p[1] ? p[0] : p[1];
  }
  return v;
}

// A group of G lanes (G = 8, 16, 32 or 64, the power of two >= min(E, 64)) holds a token's E logits,
// VPL per lane (expert gl + i * G in register i, gl = lane within the group), as order-preserving integers.
template <int G, int VPL>
__device__ __forceinline__ void load_keys(const float* __restrict__ logits, int n_experts, long token, bool live, int gl,
                                          uint32_t (&key)[VPL]) {
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int e = gl + i * G;
    key[i] = (live && e < n_experts) ? logit_key(logits[token * n_experts + e]) : 0u;
  }
}

// K rounds pick the K experts: the largest key of the group (data-parallel primitives between lanes, no trip through
// the LDS crossbar), then among the lanes that hold it the one of the smallest expert id, from a ballot; its key is
// retired.  Equal logits therefore go to the smaller id.  The softmax needs only the K winners.
// What bounds it: the latency of K dependent rounds.  Moving (value, id) pairs through six butterfly exchanges of the
// LDS crossbar instead took about 0.6 us per round: 21 tokens of 64 experts, K = 8, by one block (with four waves
// then, sixteen now) 36 -> 8.4 us, one token, K = 6 6.3 -> 4.0 us.
// lds_idx (or NULL): a copy of topk_idx in LDS; with OUT = false the only output.
// `live` must be uniform over the group; every lane of the wavefront takes part.
template <int G, int VPL, bool OUT = true>
__device__ __forceinline__ void route_keys(uint32_t (&key)[VPL], int n_experts, int top_k, long token, bool live, int gl,
                                           int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int32_t* lds_idx) {
  float win_v[VPL];  // winner j is kept by lane j % G in register j / G
  int win_i[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i) { win_v[i] = 0.0f; win_i[i] = 0; }
  const int lane = threadIdx.x % 64;

  float v_max = 0.0f, denom = 0.0f;
  for (int j = 0; j < top_k; ++j) {
    uint32_t best = key[0];
#pragma unroll
    for (int i = 1; i < VPL; ++i) best = best > key[i] ? best : key[i];
    best = group_max<G>(best);
    int bi = 0;
#pragma unroll
    for (int i = VPL - 1; i >= 0; --i) {  // descending registers: the smallest id is found last
      const uint64_t holders = __ballot(key[i] == best);
      if constexpr (G == 64) {
        if (holders) bi = i * 64 + __ffsll((long long)holders) - 1;
      } else {
        const uint32_t word = lane < 32 ? (uint32_t)holders : (uint32_t)(holders >> 32);
        const uint32_t mine = (word >> (lane % 32 / G * G)) & (uint32_t)((1ull << G) - 1);
        if (mine) bi = i * G + __ffs((int)mine) - 1;
      }
    }
    const float bv = key_logit(best);
    if (j == 0) v_max = bv;
    denom += expf(bv - v_max);
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      if (bi == gl + i * G) key[i] = 0;  // retire the winner
      if (j == gl + i * G) { win_v[i] = bv; win_i[i] = bi; }
    }
  }
  if (!live) return;
  const float inv = 1.0f / denom;
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int j = gl + i * G;
    if (j < top_k) {
      const int e = win_i[i] < n_experts ? win_i[i] : n_experts - 1;  // only reachable with non-finite input
      if (lds_idx) lds_idx[token * top_k + j] = e;
      if constexpr (OUT) {
        topk_idx[token * top_k + j] = e;
        topk_w[token * top_k + j] = expf(win_v[i] - v_max) * inv;
      }
    }
  }
}

template <int G, int VPL>
__device__ __forceinline__ void route_token(const float* __restrict__ logits, int n_experts, int top_k, long token,
                                            bool live, int gl, int32_t* __restrict__ topk_idx,
                                            float* __restrict__ topk_w, int32_t* lds_idx = nullptr) {
  uint32_t key[VPL];
  load_keys<G, VPL>(logits, n_experts, token, live, gl, key);
  route_keys<G, VPL>(key, n_experts, top_k, token, live, gl, topk_idx, topk_w, lds_idx);
}

__device__ __forceinline__ int clamp_key(int key, int n_experts) {
  return key < 0 ? 0 : (key >= n_experts ? n_experts - 1 : key);
}

// The whole permutation of at most 64 assignments (every decode batch) by one wavefront, without LDS and
// without barriers: lane a holds assignment a, learns every other key through readlane, and counts the
// keys that sort before its own (smaller key, or equal key in a lower lane: the stable order); lane l
// does the same counting for experts l, 64 + l, ... (CH of them) to produce the offsets.  Same integers as the general
// path.  Call with the first wavefront of a block.
template <int CH>
__device__ __forceinline__ void permute_rank_one_wave(const int32_t* topk_idx, int n_assign, int n_experts,
                                                      int32_t* __restrict__ expert_offsets,
                                                      int32_t* __restrict__ counts_out, int32_t* __restrict__ perm,
                                                      int32_t* __restrict__ inv_perm) {
  const int lane = threadIdx.x % 64;
  const bool valid = lane < n_assign;
  const int key = valid ? clamp_key(topk_idx[lane], n_experts) : n_experts;
  int before = 0, below[CH], equal[CH];
#pragma unroll
  for (int j = 0; j < CH; ++j) below[j] = equal[j] = 0;
  for (int i = 0; i < n_assign; ++i) {  // uniform
    const int ki = __builtin_amdgcn_readlane(key, i);
    before += (ki < key) | ((ki == key) & (i < lane));
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      below[j] += ki < j * 64 + lane;
      equal[j] += ki == j * 64 + lane;
    }
  }
  if (valid) {
    perm[before] = lane;
    inv_perm[lane] = before;
  }
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int e = j * 64 + lane;
    if (e < n_experts) {
      expert_offsets[e] = below[j];
      if (counts_out) counts_out[e] = equal[j];
    }
  }
  if (lane == 0) expert_offsets[n_experts] = n_assign;
}

}  // namespace hmoe
