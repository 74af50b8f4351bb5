// fp32 FFN on matrix instructions (HMOE_F32 with HMOE_FFN_AUTO, hidden and ffn multiples of 4, more than a few rows; the
// rest takes the general kernels of ffn_reference.hip, see ffn_f32_takes).  Weights are plain row-major.
//
// v_mfma_f64_16x16x4_f64 on operands widened to 64 bits: products are exact, sums are kept in 64 bits and rounded once, so
// the order of the sums needs no care.  Error of a layer (2-norm, against 64 bits throughout), with the fp32 instruction and 64
// partial sums per output / here: 256 x 512 1.06e-7 / 7.3e-8, 1024 x 4096 1.9e-7 / 7.4e-8, 4096 x 4096 2.6e-7 / 6.7e-8.  It runs at
// half the rate of the fp32 instruction, which needed eight waves per tile for those sums, and their 64 KB met in LDS.
//   * A tile is 16 MR rows of one expert x 32 weight rows (gate and up of 16 features, or 32 columns of the down
//     projection); every weight row is read once per tile instead of once per token.  The four waves of the block share K in
//     pairs of pieces of 16, dealt in turn, and their sums meet in LDS.  (Pairs next to each other are the 128 bytes of a cache
//     line; single pieces dealt in turn cost 5 to 12 % from K = 1408 on.  Eight waves are faster in a few launches of long K and
//     few rows, gate/up of 4 experts of 4096 x 4096 at 3 tokens 65 against 73 us, and slower in most.)
//   * Lane (j, kblk) loads four consecutive k of row j; element i of both operands forms the k-step {i, 4 + i, 8 + i,
//     12 + i} of a piece, so no data moves between lanes.  Loads are unconditional (clamped), a set of two pieces ahead,
//     weights first: the rows of gate/up hang on the row map.
//   * What bounds it with many rows is the instruction itself and the vector instructions beside it: 71 % of the time the matrix
//     pipe was busy when every operand was widened and cleared past the end of K, one vector instruction each.  Only
//     the last pieces clear now: one expert of 4096 x 4096, 1000 tokens, gate/up 1235 -> 1078 us (fp32 instruction 1168).
// Layers (us in a graph), fp32 instruction / everything cleared, single pieces / now: 8 experts of 256 x 512, top 2, 16 tokens 20.7 /
// 20.7 / 17.9, 77 24.5 / 25.5 / 22.7, 300 36.2 / 33.5 / 33.4, 1000 83.4 / 68.1 / 66.9; 8 of 1024 x 4096, top 2, 64 tokens 158 / 166 / 137, 1000
// 1106 / 1073 / 949; 64 of 2048 x 1408, top 6, 300 tokens 934 / 871 / 764; 4 of 4096 x 4096, top 1, 3 tokens 132 / 127 / 133, 64 276 / 298 /
// 251, 300 708 / 751 / 645, 1000 1847 / 1964 / 1713; one of 4096 x 4096, 64 tokens 147 / 167 / 139.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "tile_locate.h"

namespace hmoe {

// D = A(16x4) * B(4x16) + C in 64 bits.  Lane l supplies A[l%16][l/16] and B[l/16][l%16]; register r of lane l is
// D[4 r + l/16][l%16].
typedef double f64x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f64x4_t mfma_16x16x4_f64(double a, double b, f64x4_t c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int F32_WAVES = 4;
template <bool GATEUP, int MR>
__global__ __launch_bounds__(64 * F32_WAVES) void ffn_f32_kernel(TiledCtx c, const float* __restrict__ in, float* __restrict__ out) {
  constexpr int NW = F32_WAVES, NU = 2, SET = 2;  // SET: pieces per register set, next to each other; two sets alternate
  __shared__ double red[NW][MR][NU][4][64];
  TileLoc loc;
  if (!locate_tile<16 * MR>(c, loc)) return;  // uniform over the block
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, j = lane % 16, kblk = lane / 16;
  const int K = GATEUP ? c.hidden : c.ffn;
  const int n_out = GATEUP ? c.ffn : c.hidden;
  const int m0 = loc.mt * 16 * MR;
  const float* w = (const float*)(c.slots + (size_t)loc.slot * c.slot_bytes) + (GATEUP ? 0 : 2 * (size_t)c.ffn * c.hidden);
  // weight rows and input rows past the end are read from the last valid row; their products are never stored
  const float* ws[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int n = GATEUP ? min(loc.nt * 16 + j, n_out - 1) + u * n_out : min(loc.nt * 32 + u * 16 + j, n_out - 1);
    ws[u] = w + (size_t)n * K;
  }
  int row[MR];
#pragma unroll
  for (int i = 0; i < MR; ++i) {
    row[i] = loc.row_first + min(m0 + i * 16 + j, loc.m_rows - 1);
    if (GATEUP && c.row_map) row[i] = c.row_map[row[i]];
  }

  const int pieces = (K + 15) / 16;
  f32x4_t a[2][SET][MR], b[2][SET][NU];
  const float* xs[MR];
  auto load_weights = [&](int s, int p0) {
#pragma unroll
    for (int d = 0; d < SET; ++d) {
      const int k = min((p0 + d) * 16 + kblk * 4, K - 4);  // K is a multiple of 4: four k are all inside or all outside
#pragma unroll
      for (int u = 0; u < NU; ++u) b[s][d][u] = *(const f32x4_t*)(ws[u] + k);
    }
  };
  auto load_rows = [&](int s, int p0) {
#pragma unroll
    for (int d = 0; d < SET; ++d) {
      const int k = min((p0 + d) * 16 + kblk * 4, K - 4);
#pragma unroll
      for (int i = 0; i < MR; ++i) a[s][d][i] = *(const f32x4_t*)(xs[i] + k);
    }
  };
  f64x4_t acc[MR][NU];
#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int u = 0; u < NU; ++u) acc[i][u] = f64x4_t{0, 0, 0, 0};
  auto multiply_set = [&](int s, int p0, auto inside) {
#pragma unroll
    for (int d = 0; d < SET; ++d) {
      // (both cleared past the end: what was read instead may not be finite)
      const bool ok = decltype(inside)::value || (p0 + d) * 16 + kblk * 4 < K;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double bd[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) bd[u] = (double)(ok ? b[s][d][u][e] : 0.0f);
#pragma unroll
        for (int i = 0; i < MR; ++i) {
          const double ad = (double)(ok ? a[s][d][i][e] : 0.0f);
#pragma unroll
          for (int u = 0; u < NU; ++u) acc[i][u] = mfma_16x16x4_f64(ad, bd[u], acc[i][u]);
        }
      }
    }
  };
  auto multiply = [&](int s, int p0) {
    if ((p0 + SET) * 16 <= K) multiply_set(s, p0, std::true_type{});  // uniform
    else multiply_set(s, p0, std::false_type{});
  };
  load_weights(0, wave * SET);
#pragma unroll
  for (int i = 0; i < MR; ++i) xs[i] = in + (size_t)(GATEUP && c.row_map ? row[i] / c.map_div : row[i]) * K;
  load_rows(0, wave * SET);
  for (int p = wave * SET; p < pieces; p += 2 * SET * NW) {
    load_weights(1, p + SET * NW);
    load_rows(1, p + SET * NW);
    __builtin_amdgcn_sched_barrier(0);  // (the compiler would move the loads down to their uses)
    multiply(0, p);
    __builtin_amdgcn_sched_barrier(0);
    load_weights(0, p + 2 * SET * NW);
    load_rows(0, p + 2 * SET * NW);
    __builtin_amdgcn_sched_barrier(0);
    if (p + SET * NW < pieces) multiply(1, p + SET * NW);  // uniform
    __builtin_amdgcn_sched_barrier(0);
  }

#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][i][u][r][lane] = acc[i][u][r];
  __syncthreads();
  for (int q = wave; q < 4 * MR; q += NW) {  // register r of row fragment i: output row 4 r + kblk of the fragment
    const int i = q / 4, r = q % 4;
    float v[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      double sum = 0.0;
#pragma unroll
      for (int o = 0; o < NW; ++o) sum += red[o][i][u][r][lane];
      v[u] = (float)sum;
    }
    const int m = m0 + i * 16 + 4 * r + kblk;
    if (m >= loc.m_rows) continue;
    float* orow = out + (size_t)(loc.row_first + m) * n_out;
    if (GATEUP) {
      const int n = loc.nt * 16 + j;
      if (n < n_out) orow[n] = v[0] / (1.0f + expf(-v[0])) * v[1];
    } else {
      const int n = loc.nt * 32 + j;
      if (n < n_out) orow[n] = v[0];
      if (n + 16 < n_out) orow[n + 16] = v[1];
    }
  }
}

template <bool GATEUP, int MR>
static void launch_stage_f32(TiledCtx c, int n_rows, const float* in, float* out, hipStream_t s) {
  c.n_tiles_n = GATEUP ? (c.ffn + 15) / 16 : (c.hidden + 31) / 32;
  c.grid_padded = (int)((tiles_upper_bound(c, n_rows, 16 * MR) + 7) / 8 * 8);
  hipLaunchKernelGGL((ffn_f32_kernel<GATEUP, MR>), dim3((unsigned)c.grid_padded), dim3(64 * F32_WAVES), 0, s, c, in, out);
}

// The general kernels read an expert's weights for every row again, out of the caches (about 6 TB/s); the tiles read them
// once, and their two launches start later (locating a tile, one wave per piece of K, sums in LDS).  So the general kernels
// have it until the rows that find their expert's weights already read, by uniform routing, re-read more than 30 MB (100 MB
// where all of the layer's weights stay in an L2) and 15 % of what is read in any case.  The line was drawn where the tiles on
// the fp32 instruction began to win; against the present ones it is late by a few tokens.  Layers, general kernels / tiles,
// us in a graph (* what the rule takes): 8 experts of 256 x 512, top 2: 8 tokens 15.0* / 17.2, 10 tokens 20.3* / 17.2, 16 tokens 24.2 / 17.9*;
// 8 of 1024 x 4096, top 2: 2 tokens 56.0* / 52.5, 3 tokens 67.0 / 57.8*; 64 of 1024 x 512, top 8: 3 tokens 48.2* / 45.2, 6 tokens
// 74.0 / 62.5*; one of 256 x 512: 33 tokens 19.6* / 21.8, 64 tokens 24.0* / 23.6, 90 tokens 29.8 / 22.5*; 4 of 64 x 96, top 2: 64 tokens
// 15.3* / 17.6, 200 tokens 24.2* / 19.0.
bool ffn_f32_takes(const hmoe_layer_desc& d, int n_rows) {
  if (d.dtype != HMOE_F32 || d.hidden % 4 != 0 || d.ffn % 4 != 0) return false;
  const long n_tiles = std::max((d.ffn + 15) / 16, (d.hidden + 31) / 32);  // the grid has to fit its 32-bit dimension
  if (((long)n_rows / 16 + std::min(d.n_experts, n_rows)) * n_tiles >= (1l << 22)) return false;
  const double expert = 12.0 * d.hidden * d.ffn, layer = expert * d.n_experts;
  const double touched = d.n_experts * (1.0 - std::pow(1.0 - (double)d.top_k / d.n_experts, (double)n_rows / d.top_k));
  return (n_rows - touched) * expert > (layer <= 4e6 ? 100e6 : 30e6) + 0.15 * touched * expert;
}

int launch_ffn_f32(const FfnArgs& a) {
  const hmoe_layer_desc& d = *a.desc;
  if (a.n_rows == 0) return HMOE_OK;
  if ((d.ffn + 3) / 4 > 65535 || (d.hidden + 3) / 4 > 65535) return HMOE_ERR_UNSUPPORTED;  // as the general kernels
  TiledCtx c{a.offsets, a.slot_of, a.slots, a.slot_bytes, a.active, d.n_experts, d.hidden, d.ffn, 0, 0, a.row_map, a.map_div};
  // MR: one 16-row fragment per tile while experts have fewer rows than that on average (a second one would be padding),
  // else two, which halve the reads of the weights
  const bool one = a.n_rows < 16 * d.n_experts;
  probe_before(a.stream);
  (one ? launch_stage_f32<true, 1> : launch_stage_f32<true, 2>)(c, a.n_rows, (const float*)a.x_perm, (float*)a.h, a.stream);
  probe_after(a.stream);
  probe_before(a.stream);
  (one ? launch_stage_f32<false, 1> : launch_stage_f32<false, 2>)(c, a.n_rows, (const float*)a.h, (float*)a.o_perm, a.stream);
  probe_after(a.stream);
  HMOE_HIP(hipGetLastError());
  return HMOE_OK;
}

}  // namespace hmoe
