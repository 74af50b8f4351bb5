// Router logits x . W_g (Eq. (1), Section II-A) of the tokens of a block; shared by hmoe_router_logits and the fused
// front ends.
#pragma once

#include "common.h"

namespace hmoe {

constexpr int ROUTER_SMALL_T = 16;      // tokens up to which the fused front end is one block, which computes the logits, routes
                                        // and permutes (hmoe_router_logits: a block per 16 experts, all tokens)

// How a block of NW waves divides its work: MA fragments of 16 tokens; the waves split K KS ways, and NW / KS groups of
// them own NF fragments of 16 experts each.
template <int MA_, int NF_, int KS_, int NW_>
struct RouterShape {
  static constexpr int MA = MA_, NF = NF_, KS = KS_, NW = NW_, THREADS = 64 * NW_;
  static constexpr int EXPERT_FRAGS = NW / KS * NF;            // of the block
  static constexpr int ALL = KS * EXPERT_FRAGS * MA * 4 * 64;  // partial sums
  static constexpr int TURNS = ALL > 16384 ? ALL / 16384 : 1;  // they meet in 64 KB of LDS, NF / TURNS fragments of a wave at a time
  static constexpr int RED = ALL / TURNS;
  static_assert(NF % TURNS == 0, "");
  // steps of 32 k loaded at once: as many as the registers hold next to the sums (one set of them per piece, pair and whole)
  static constexpr int WAVES_PER_SIMD = MA * NF <= 8 ? 4 : 2;
  static constexpr int SUMS = (KS == 16 ? 1 : KS == 8 ? 2 : 3) * MA * NF * 4, LEFT = 512 / WAVES_PER_SIMD - 24 - SUMS;
  static constexpr int STEPS = LEFT >= 32 * (MA + NF) ? 8 : LEFT >= 16 * (MA + NF) ? 4 : LEFT >= 8 * (MA + NF) ? 2 : 1;
};

// bf16 operands, K-contiguous rows: lanes load 16x16x32 MFMA fragments straight from global memory (token or expert
// row = lane % 16, 8 k values at 8 * (lane / 16)).  K is cut into 16 contiguous pieces s0..s15, each summed in
// ascending k, and a logit is ((W0 + W1) + W2) + W3 with Wi = (s4i + s4i+1) + (s4i+2 + s4i+3).  That order is the
// same for every block shape, so a token's logits do not depend on the batch it is part of: with KS = 16 a wave owns
// one piece; with KS = 8 or 4 it works through two or four pieces and adds them up itself.
//
// What bounds it: a decode router is a chain of memory round trips, not bandwidth, so what counts is how few loads a
// wave has to wait for one after the other; and a block reads all of w_g through one CU, at about 15 bytes per clock
// where rows lie 2 KB or more apart, so what counts next is that nothing is loaded twice or in vain.  Four waves with
// contiguous quarters of K took 7.9 us for one token, 8 experts, K = 4096 (eight dependent batches of loads); sixteen
// waves, each with all of its piece in flight at once, take 5.0 us.  No load is issued past a piece's end (a wave-uniform
// branch): with a second register set loaded ahead from clamped addresses, a piece of four steps cost twelve steps of
// loads: 16 experts, K = 2048, 12.1 us for 17 to 2048 tokens, now 5.8 (four waves: 6.7).  Of more than 64 experts every
// wave takes as many as its registers hold, so that x is read once or twice and not by four groups of waves: 128 experts,
// K = 4096, 17 to 2048 tokens 54 -> 34 us (four waves: 35); 16384 tokens 214 -> 79 us (92).  Blocks of up to 32 tokens
// halve the reads of w_g of large batches.
//
// tokens_per_block <= 16 MA.  logits [T, logit_pitch] global out (E columns of it); lds_logits [tokens_per_block * E] the same values in LDS, or
// NULL.  Ends with a block barrier.
template <class SHAPE>
__device__ __forceinline__ void router_logits_block(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w_g,
                                                    int n_tokens, int n_experts, int hidden, float* __restrict__ logits,
                                                    int tokens_per_block, float* red, float* lds_logits, int logit_pitch) {
  constexpr int MA = SHAPE::MA, NF = SHAPE::NF, KS = SHAPE::KS, EF = SHAPE::EXPERT_FRAGS;
  constexpr int U = SHAPE::STEPS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int row = lane % 16, kblk = lane / 16;
  const int part = wave % KS, egroup = wave / KS;
  const long t0 = (long)blockIdx.x * tokens_per_block;
  const int kt = (hidden + 31) / 32, quarter = (kt + 3) / 4, piece = (quarter + 3) / 4;
  // (32-bit lane offsets from wave-uniform bases: half the registers of pointers)
  const u32x4* const x_block = (const u32x4*)(x + t0 * hidden);
  const u32x4* const w_all = (const u32x4*)w_g;
  uint32_t xo[MA], wo[NF];
#pragma unroll
  for (int m = 0; m < MA; ++m) {
    const int t = m * 16 + row;
    xo[m] = (uint32_t)(t0 + t < n_tokens ? t : (int)(n_tokens - 1 - t0)) * (uint32_t)(hidden / 8);
  }
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    const int e = (egroup * NF + j) * 16 + row;
    wo[j] = (uint32_t)(e < n_experts ? e : n_experts - 1) * (uint32_t)(hidden / 8);
  }
  const int last_chunk = hidden / 8 - 1;  // 16-byte pieces of a row; hidden is a multiple of 16, so a step may be half full
  u32x4 xa[U][MA], wb[U][NF];
  auto load = [&](int kb, int kb1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kb + u < kb1) {  // uniform over the wave
        const int c = (kb + u) * 4 + kblk, cc = c < last_chunk ? c : last_chunk;
#pragma unroll
        for (int m = 0; m < MA; ++m) xa[u][m] = x_block[xo[m] + cc];
#pragma unroll
        for (int j = 0; j < NF; ++j) wb[u][j] = w_all[wo[j] + cc];
      }
    }
  };
  f32x4_t acc[MA][NF], pair[MA][NF], sum[MA][NF];
  auto multiply = [&](int kb, int kb1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kb + u < kb1) {
        if ((kb + u) * 32 + 32 > hidden) {  // the half step at the end of K: its upper half counts nothing
#pragma unroll
          for (int m = 0; m < MA; ++m) xa[u][m] = kblk < 2 ? xa[u][m] : u32x4{0, 0, 0, 0};
#pragma unroll
          for (int j = 0; j < NF; ++j) wb[u][j] = kblk < 2 ? wb[u][j] : u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
          for (int j = 0; j < NF; ++j) acc[m][j] = mfma_16x16x32_bf16(xa[u][m], wb[u][j], acc[m][j]);
      }
    }
  };
#pragma unroll 1
  for (int q = 0; q < 16 / KS; ++q) {
    const int s = part * (16 / KS) + q;  // piece
    const int end = min((s / 4 + 1) * quarter, kt);
    const int kb0 = min((s / 4) * quarter + (s % 4) * piece, end), kb1 = min(kb0 + piece, end);
#pragma unroll
    for (int m = 0; m < MA; ++m)
#pragma unroll
      for (int j = 0; j < NF; ++j) acc[m][j] = f32x4_t{0, 0, 0, 0};
    for (int kb = kb0; kb < kb1; kb += U) {
      load(kb, kb1);
      multiply(kb, kb1);
    }
#pragma unroll
    for (int m = 0; m < MA; ++m)
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        pair[m][j] = q % 2 == 0 ? acc[m][j] : pair[m][j] + acc[m][j];
        if (q <= 1) sum[m][j] = pair[m][j];
        else if (q == 3) sum[m][j] = sum[m][j] + pair[m][j];
      }
  }
  constexpr int TURNS = SHAPE::TURNS, NT = NF / TURNS, EG = EF / NF;  // expert fragments per wave and turn; expert groups
#pragma unroll
  for (int turn = 0; turn < TURNS; ++turn) {
    // partial sums [part][expert group][expert fragment of the turn][token fragment][register][lane]
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int m = 0; m < MA; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(((part * EG + egroup) * NT + j) * MA + m) * 256 + r * 64 + lane] = sum[m][turn * NT + j][r];
    __syncthreads();
    for (int i = threadIdx.x; i < EG * NT * MA * 256; i += SHAPE::THREADS) {
      // register r of lane l is token 4 (l / 16) + r, expert l % 16 of the fragment
      const int l = i % 64, r = i / 64 % 4, m = i / 256 % MA, j = i / (256 * MA) % NT, g = i / (256 * MA * NT);
      const int tok = m * 16 + 4 * (l / 16) + r, e = (g * NF + turn * NT + j) * 16 + l % 16;
      float v = 0.0f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        float q[KS / 4];
#pragma unroll
        for (int p = 0; p < KS / 4; ++p) q[p] = red[(w * (KS / 4) + p) * (EG * NT * MA * 256) + i];
        const float quarter_sum = KS == 16 ? (q[0] + q[1 % (KS / 4)]) + (q[2 % (KS / 4)] + q[3 % (KS / 4)]) : KS == 8 ? q[0] + q[1 % (KS / 4)] : q[0];
        v = w == 0 ? quarter_sum : v + quarter_sum;
      }
      if (tok < tokens_per_block && t0 + tok < n_tokens && e < n_experts) {
        logits[(t0 + tok) * logit_pitch + e] = v;
        if (lds_logits) lds_logits[tok * n_experts + e] = v;
      }
    }
    __syncthreads();
  }
}

// Tokens per block: 16, or fewer while the grid would leave more than half of the CUs without a block; beyond 2048 tokens
// up to 32, so that the grid stays at half of the CUs until they are full (the other half is left to what runs beside it).
static inline int router_tokens_per_block(int n_tokens) {
  if (n_tokens <= ROUTER_SMALL_T) return 16;
  if (n_tokens > 2048) return n_tokens < 4096 ? (n_tokens + 127) / 128 : 32;
  int tpb = 16;
  while (tpb > 4 && (n_tokens + tpb - 1) / tpb < 128) tpb /= 2;
  return tpb;
}
// CALL(lanes per token when routing, values per lane, the four RouterShape parameters) for a number of experts: batches
// of one block, and larger ones.
// The one block has the GPU to itself and takes sixteen waves.  The blocks of a larger batch run beside the shared
// experts' FFN, whose gate/up launch they would keep off half of the CUs for their whole time: eight waves of up to 116
// registers leave room for a block of it (of up to 128 experts).  Alone both take the same time (64 experts, K = 2048, 2048 tokens 14.2 us); the layer of 64
// experts of 2048 x 1408, top 6, 1024 tokens 295 -> 288 us, 4096 tokens with half as many blocks 585 -> 575 us.
#define HMOE_ROUTER_SHAPES_ONE_BLOCK(E, CALL)            \
  do {                                                   \
    if ((E) <= 8) { CALL(8, 1, 1, 1, 16, 16); }          \
    else if ((E) <= 16) { CALL(16, 1, 1, 1, 16, 16); }   \
    else if ((E) <= 32) { CALL(32, 1, 1, 2, 16, 16); }   \
    else if ((E) <= 64) { CALL(64, 1, 1, 4, 16, 16); }   \
    else if ((E) <= 128) { CALL(64, 2, 1, 8, 16, 16); }  \
    else { CALL(64, 4, 1, 8, 8, 16); }                   \
  } while (0)
#define HMOE_ROUTER_SHAPES_MANY(E, TPB, CALL)            \
  do {                                                   \
    if ((TPB) <= 16) {                                   \
      if ((E) <= 8) { CALL(8, 1, 1, 1, 8, 8); }          \
      else if ((E) <= 16) { CALL(16, 1, 1, 1, 8, 8); }   \
      else if ((E) <= 32) { CALL(32, 1, 1, 2, 8, 8); }   \
      else if ((E) <= 64) { CALL(64, 1, 1, 4, 8, 8); }   \
      else if ((E) <= 128) { CALL(64, 2, 1, 8, 8, 8); }  \
      else { CALL(64, 4, 1, 8, 8, 16); }                 \
    } else {                                             \
      if ((E) <= 8) { CALL(8, 1, 2, 1, 8, 8); }          \
      else if ((E) <= 16) { CALL(16, 1, 2, 1, 8, 8); }   \
      else if ((E) <= 32) { CALL(32, 1, 2, 2, 8, 8); }   \
      else if ((E) <= 64) { CALL(64, 1, 2, 4, 8, 8); }   \
      else if ((E) <= 128) { CALL(64, 2, 2, 8, 8, 8); }  \
      else { CALL(64, 4, 2, 8, 4, 8); }                  \
    }                                                    \
  } while (0)

}  // namespace hmoe
