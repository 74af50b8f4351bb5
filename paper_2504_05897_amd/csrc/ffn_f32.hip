// fp32 FFN on matrix instructions (HMOE_F32 with HMOE_FFN_AUTO, hidden and ffn multiples of 4, more than a few rows; the
// rest takes the general kernels of ffn_reference.hip, see ffn_f32_takes).  Weights are plain row-major.
//
// A tile is 16 MR rows of one expert x 32 weight rows (gate and up of 16 features, or 32 columns of the down
// projection); every weight row is read once per tile instead of once per token, in 16-byte loads.  With few rows the
// path is bound by latency, with many by the operands' way through the caches.  K is split over the NW = 4 MR waves of the
// block, so each has a quarter or an eighth of the trips to memory, all of a round issued at once.
// Measured (8 experts of 256 x 512, top 2, whole layer, against one wavefront per output element): 77 tokens 61 -> 35 us,
// 300 tokens 173 -> 38 us, 1024 tokens 527 -> 88 us (gate/up 53 us); with 16 tokens the calls on the host take longer.
//   * v_mfma_f32_16x16x4_f32 is a full fp32 multiply-add.  Lane (j, kblk) loads four consecutive k of row j; element i
//     of both operands forms the k-step {i, 4 + i, 8 + i, 12 + i} of a 16-wide piece of K, so no data moves between
//     lanes.
//   * Every element i and every one of S = 16 / NW consecutive pieces has an accumulator of its own: NW * S * 4 = 64
//     partial sums per output over K / 64 products each (as many as one wavefront per output element would keep), which
//     are added up in 64 bits and rounded once: error of the layer 1.27e-7 against 1.67e-7 (2-norm, 1024 tokens).
#include <algorithm>
#include <cmath>

#include "common.h"
#include "tile_locate.h"

namespace hmoe {

__device__ __forceinline__ f32x4_t mfma_16x16x4_f32(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <bool GATEUP, int MR>
__global__ __launch_bounds__(256 * MR, 2) void ffn_f32_kernel(TiledCtx c, const float* __restrict__ in, float* __restrict__ out) {
  constexpr int NW = 4 * MR, S = 16 / NW, NU = 2;
  __shared__ double red[NW][MR][NU][4][64];
  TileLoc loc;
  if (!locate_tile<16 * MR>(c, loc)) return;  // uniform over the block
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, j = lane % 16, kblk = lane / 16;
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
  const float* xs[MR];
#pragma unroll
  for (int i = 0; i < MR; ++i) {
    const int row = loc.row_first + min(m0 + i * 16 + j, loc.m_rows - 1);
    xs[i] = in + (size_t)(GATEUP ? mapped_row(c.row_map, c.map_div, row) : row) * K;
  }

  f32x4_t acc[S][4][MR][NU];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < MR; ++i)
#pragma unroll
        for (int u = 0; u < NU; ++u) acc[s][e][i][u] = f32x4_t{0, 0, 0, 0};
  for (int k0 = 0; k0 < K; k0 += 256) {  // 256 k per round of the block: S pieces of 16 per wave
    f32x4_t a[S][MR], b[S][NU];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k = k0 + (s * NW + wave) * 16 + kblk * 4;
      const bool ok = k < K;  // K is a multiple of 4: four k are all inside or all outside
#pragma unroll
      for (int i = 0; i < MR; ++i) a[s][i] = ok ? *(const f32x4_t*)(xs[i] + k) : f32x4_t{0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < NU; ++u) b[s][u] = ok ? *(const f32x4_t*)(ws[u] + k) : f32x4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MR; ++i)
#pragma unroll
          for (int u = 0; u < NU; ++u) acc[s][e][i][u] = mfma_16x16x4_f32(a[s][i][e], b[s][u][e], acc[s][e][i][u]);
  }

#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double p[S];
#pragma unroll
        for (int s = 0; s < S; ++s) p[s] = ((double)acc[s][0][i][u][r] + acc[s][1][i][u][r]) + ((double)acc[s][2][i][u][r] + acc[s][3][i][u][r]);
#pragma unroll
        for (int d = 1; d < S; d *= 2)
#pragma unroll
          for (int s = 0; s + d < S; s += 2 * d) p[s] += p[s + d];
        red[wave][i][u][r][lane] = p[0];
      }
  __syncthreads();
  // NW waves, 4 MR registers of 64 lanes per unit: wave w finishes register w % 4 of row fragment w / 4
  const int i = wave / 4, r = wave % 4;
  const int m = m0 + i * 16 + kblk * 4 + r;
  float v[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    double p[NW];
#pragma unroll
    for (int o = 0; o < NW; ++o) p[o] = red[o][i][u][r][lane];
#pragma unroll
    for (int d = 1; d < NW; d *= 2)
#pragma unroll
      for (int o = 0; o + d < NW; o += 2 * d) p[o] += p[o + d];
    v[u] = (float)p[0];
  }
  if (m >= loc.m_rows) return;
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

template <bool GATEUP, int MR>
static void launch_stage_f32(TiledCtx c, int n_rows, const float* in, float* out, hipStream_t s) {
  c.n_tiles_n = GATEUP ? (c.ffn + 15) / 16 : (c.hidden + 31) / 32;
  c.grid_padded = (int)((tiles_upper_bound(c, n_rows, 16 * MR) + 7) / 8 * 8);
  hipLaunchKernelGGL((ffn_f32_kernel<GATEUP, MR>), dim3((unsigned)c.grid_padded), dim3(256 * MR), 0, s, c, in, out);
}

// The general kernels read an expert's weights for every row again, out of the caches (about 6 TB/s); the tiles read them
// once, but from memory at four fifths of the general kernels' rate, and their two launches start 5 us later (locating a
// tile, one wave per piece of K, sums in LDS).  So the general kernels have it until the rows that find their expert's
// weights already read, by uniform routing, re-read more than 30 MB (100 MB where all of the layer's weights stay in an L2)
// and 15 % of what is read in any case.  Layers, general kernels / tiles, us: 8 experts of 256 x 512, top 2: 8 tokens
// 15.1 / 19.6, 16 tokens 24.6 / 20.5; 8 of 1024 x 4096, top 2: 2 tokens 56.9 / 63.5, 3 tokens 68.5 / 65.6; 64 of 1024 x 512, top 8: 4
// tokens 64.3 / 67.0, 6 tokens 85.2 / 81.0; one of 256 x 512: 33 tokens 19.8 / 23.1, 64 tokens 25.0 / 25.0; 4 of 64 x 96, top 2: 64 tokens
// 15.6 / 19.3.
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
  if (one) launch_stage_f32<true, 1>(c, a.n_rows, (const float*)a.x_perm, (float*)a.h, a.stream);
  else launch_stage_f32<true, 2>(c, a.n_rows, (const float*)a.x_perm, (float*)a.h, a.stream);
  probe_after(a.stream);
  probe_before(a.stream);
  if (one) launch_stage_f32<false, 1>(c, a.n_rows, (const float*)a.h, (float*)a.o_perm, a.stream);
  else launch_stage_f32<false, 2>(c, a.n_rows, (const float*)a.h, (float*)a.o_perm, a.stream);
  probe_after(a.stream);
  HMOE_HIP(hipGetLastError());
  return HMOE_OK;
}

}  // namespace hmoe
