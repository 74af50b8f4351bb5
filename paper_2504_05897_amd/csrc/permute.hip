// hmoe_permute: stable counting sort of the A = T*K assignments by expert id, then row gather.
//
// Per-expert load is the quantity everything downstream consumes (Section IV-B uses it to order
// the queues); here it becomes expert_offsets.  The sort is stable and uses no order-dependent
// atomics, so the result is the same on every run.  A block ranks one assignment per thread: a wave finds the lanes of
// equal key with ballots, and waves are ordered by per-wave LDS counts.  What a block needs besides its own
// assignments is, per expert, how many lie in front of them and how many there are in all:
//   A <= 1024 (every decode shape)  one block of 16 waves, nothing lies elsewhere
//   A <= 4096                       blocks of 8 waves, each counts all A keys itself (16 KB from L2 at most): one launch
//   A <= 262144                     a histogram launch over chunks of 1024 first; every block of 4 waves adds up the counts
//   beyond                          histogram, one-block scan, rank
// The launches are latency, not bandwidth (a few KB each), so what counts is how many follow one another, and that no
// block counts many keys that are alike: lanes of a wave that add to one LDS counter take turns (about 110 cycles for 64
// of them, one wave at a time).  With blocks of 16 waves counting up to 16384 keys themselves, 16384 rows of one expert took
// 20 us, of 8 experts that all rows name the same two of 12 us.  Now (histogram, scan and rank in three launches before
// either): one expert, 4096 rows 4.5 us (8.1), 16384 rows 6.7 (8.9); 64 experts, top 6, 2288 assignments 4.3 (9.0), 4096
// 4.9 (9.2), 16384 7.1 (9.9), 98304 7.9 (17.4).
// The last two have blocks of four waves and 6 KB of LDS: batches of that size run next to prefill FFN blocks (of the
// shared experts) that leave a CU 56 registers per lane and 9 KB of LDS, and what does not fit beside them waits for
// their end (16-wave blocks there: the 16384-token layer 1.3 % slower).
//   then: gather    x_perm[p] = x[perm[p] / K], 16 bytes per lane
#include <mutex>

#include "route_body.h"
#include "router_body.h"

namespace hmoe {

constexpr int PB_THREADS = 256;              // histogram, scan, decode front end's routing
constexpr int PB_CHUNK = 1024;               // assignments per block
constexpr int PR_THREADS = PB_CHUNK;         // one-block permutation: one assignment per thread
constexpr int PR_SELF_COUNT_CHUNKS = 4;      // up to here every rank block counts all keys itself
constexpr int PR_SELF_SCAN_CHUNKS = 256;     // up to here every rank block adds up the histogram's counts itself

// lanes of this wavefront (among `valid` ones) that hold the same key as the caller
__device__ __forceinline__ uint64_t same_key_mask(int key, bool valid, int key_bits) {
  uint64_t m = __ballot(valid);
  for (int b = 0; b < key_bits; ++b) {
    const bool bit = (key >> b) & 1;
    const uint64_t bal = __ballot(bit);
    m &= bit ? bal : ~bal;
  }
  return m;
}

__global__ __launch_bounds__(PB_THREADS) void permute_hist_kernel(const int32_t* __restrict__ topk_idx, int n_assign,
                                                                  int n_experts, int32_t* __restrict__ block_counts) {
  __shared__ int hist[HMOE_MAX_EXPERTS];
  for (int e = threadIdx.x; e < n_experts; e += PB_THREADS) hist[e] = 0;
  __syncthreads();
  const long base = (long)blockIdx.x * PB_CHUNK;
  for (int i = threadIdx.x; i < PB_CHUNK; i += PB_THREADS) {
    const long a = base + i;
    if (a < n_assign) atomicAdd(&hist[clamp_key(topk_idx[a], n_experts)], 1);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n_experts; e += PB_THREADS) block_counts[(long)blockIdx.x * n_experts + e] = hist[e];
}

// one block: block_counts[b][e] -> exclusive base of (b, e) in the sorted order; expert_offsets
__global__ __launch_bounds__(PB_THREADS) void permute_scan_kernel(int32_t* __restrict__ block_counts, int n_blocks,
                                                                  int n_experts, int n_assign,
                                                                  int32_t* __restrict__ expert_offsets,
                                                                  int32_t* __restrict__ counts_out) {
  __shared__ int total[HMOE_MAX_EXPERTS];
  __shared__ int start[HMOE_MAX_EXPERTS];
  // (the counts are read 16 blocks at a time: one after the other, a read could not start before the store in
  // front of it)
  constexpr int AHEAD = 16;
  const int e = threadIdx.x;
  if (e < n_experts) {
    int run = 0;
    for (int b0 = 0; b0 < n_blocks; b0 += AHEAD) {
      int c[AHEAD];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) c[i] = b0 + i < n_blocks ? block_counts[(long)(b0 + i) * n_experts + e] : 0;
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        if (b0 + i < n_blocks) block_counts[(long)(b0 + i) * n_experts + e] = run;
        run += c[i];
      }
    }
    total[e] = run;
    if (counts_out) counts_out[e] = run;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int i = 0; i < n_experts; ++i) { start[i] = run; expert_offsets[i] = run; run += total[i]; }
    expert_offsets[n_experts] = run;
  }
  __syncthreads();
  if (e < n_experts) {
    const int s = start[e];
    for (int b0 = 0; b0 < n_blocks; b0 += AHEAD) {
      int c[AHEAD];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) c[i] = b0 + i < n_blocks ? block_counts[(long)(b0 + i) * n_experts + e] : 0;
#pragma unroll
      for (int i = 0; i < AHEAD; ++i)
        if (b0 + i < n_blocks) block_counts[(long)(b0 + i) * n_experts + e] = c[i] + s;
    }
  }
}

// Where a rank block learns what lies outside its chunk.
enum RankSource {
  RANK_SINGLE,     // nothing does: the chunk is the whole input
  RANK_COUNT_ALL,  // it counts every key of the input
  RANK_ADD_UP,     // counts [chunks][E] of the histogram launch
  RANK_BASES       // exclusive bases [chunks][E] of the scan launch (which also wrote the offsets)
};

// Ranks assignments [64 NW b, 64 NW (b + 1)) in block b of NW waves.  expert_offsets and counts_out are written by block 0.
template <RankSource SRC, int NW>
__device__ __forceinline__ void permute_rank_body(const int32_t* topk_idx, int n_assign, int n_experts, int key_bits,
                                                  const int32_t* __restrict__ from_before,
                                                  int32_t* __restrict__ expert_offsets,
                                                  int32_t* __restrict__ counts_out, int32_t* __restrict__ perm,
                                                  int32_t* __restrict__ inv_perm) {
  constexpr int THREADS = 64 * NW;
  constexpr int PER_CHUNK = PB_CHUNK / THREADS;    // blocks that share one chunk of the histogram
  static_assert(NW >= HMOE_MAX_EXPERTS / 64, "one thread per expert");
  __shared__ int wave_base[NW][HMOE_MAX_EXPERTS];  // first counts, then bases
  __shared__ int outside[2][HMOE_MAX_EXPERTS];     // per expert: in front of the block's assignments, and the rest of the others
  __shared__ int wave_total[4];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  if (SRC == RANK_SINGLE && n_assign <= 64) {  // uniform over the block: nothing below runs, so no barrier is left unmatched
    if (wave == 0) {
      if (n_experts <= 64) permute_rank_one_wave<1>(topk_idx, n_assign, n_experts, expert_offsets, counts_out, perm, inv_perm);
      else permute_rank_one_wave<HMOE_MAX_EXPERTS / 64>(topk_idx, n_assign, n_experts, expert_offsets, counts_out, perm, inv_perm);
    }
    return;
  }
  const int block = SRC == RANK_SINGLE ? 0 : (int)blockIdx.x;
  const int chunk = block / PER_CHUNK;
  const long a = (long)block * THREADS + threadIdx.x;
  const bool valid = a < n_assign;
  const int key = valid ? clamp_key(topk_idx[a], n_experts) : -1;
  for (int i = threadIdx.x; i < NW * HMOE_MAX_EXPERTS; i += THREADS) (&wave_base[0][0])[i] = 0;
  for (int i = threadIdx.x; i < 2 * HMOE_MAX_EXPERTS; i += THREADS) (&outside[0][0])[i] = 0;
  const uint64_t same = same_key_mask(key, valid, key_bits);
  __syncthreads();
  if (valid && (same >> lane) >> 1 == 0) wave_base[wave][key] = __popcll(same);  // highest lane of the group
  if constexpr (SRC == RANK_COUNT_ALL) {
    constexpr int MOST = PR_SELF_COUNT_CHUNKS * PER_CHUNK;  // blocks
    int others[MOST];
#pragma unroll
    for (int b = 0; b < MOST; ++b) {
      const long i = (long)b * THREADS + threadIdx.x;
      others[b] = b != block && i < n_assign ? clamp_key(topk_idx[i], n_experts) : -1;
    }
#pragma unroll
    for (int b = 0; b < MOST; ++b) {
      // the lanes that hold the key of the first one are counted by that one alone: a popular expert, or one of few
      const uint64_t in = __ballot(others[b] >= 0);
      if (!in) continue;  // uniform over the wave
      const int key0 = __builtin_amdgcn_readlane(others[b], __ffsll((long long)in) - 1);
      const uint64_t alike = __ballot(others[b] == key0);
      const bool counts_alike = lane == __ffsll((long long)alike) - 1;
      if (others[b] >= 0 && (others[b] != key0 || counts_alike))
        atomicAdd(&outside[b < block ? 0 : 1][others[b]], counts_alike ? __popcll(alike) : 1);
    }
  }
  if constexpr (SRC == RANK_ADD_UP || SRC == RANK_BASES) {
    // the rest of the block's own chunk
    for (int q = 0; q < PER_CHUNK; ++q) {
      const long i = (long)chunk * PB_CHUNK + q * THREADS + threadIdx.x;
      if (q != block % PER_CHUNK && i < n_assign) atomicAdd(&outside[q < block % PER_CHUNK ? 0 : 1][clamp_key(topk_idx[i], n_experts)], 1);
    }
  }
  if constexpr (SRC == RANK_ADD_UP) {
    // THREADS / slice chunks at a time, one thread per expert of each
    const int slice = n_experts <= 64 ? 64 : n_experts <= 128 ? 128 : 256;
    const int e = threadIdx.x % slice, n_chunks = (n_assign + PB_CHUNK - 1) / PB_CHUNK, step = THREADS / slice;
    int before = 0, after = 0;
    if (e < n_experts) {
#pragma unroll 8
      for (int c = threadIdx.x / slice; c < n_chunks; c += step) {
        const int n = from_before[(long)c * n_experts + e];
        before += c < chunk ? n : 0;
        after += c > chunk ? n : 0;
      }
      if (before) atomicAdd(&outside[0][e], before);
      if (after) atomicAdd(&outside[1][e], after);
    }
  }
  __syncthreads();

  // counts -> exclusive bases over (expert, wave)
  const int e = threadIdx.x;
  int first = 0, mine = 0;
  if (SRC == RANK_BASES) {
    if (e < n_experts) first = from_before[(long)chunk * n_experts + e] + outside[0][e];
  } else {
    int tot = 0, incl = 0;
    if (e < HMOE_MAX_EXPERTS) {  // the first four waves
      if (e < n_experts) {
#pragma unroll
        for (int w = 0; w < NW; ++w) mine += wave_base[w][e];
        tot = mine + outside[0][e] + outside[1][e];
      }
      incl = tot;
#pragma unroll
      for (int d = 1; d < 64; d *= 2) {
        const int below = __shfl_up(incl, d);
        if (lane >= d) incl += below;
      }
      if (lane == 63) wave_total[wave] = incl;
    }
    __syncthreads();
    if (e < n_experts) {
      for (int w = 0; w < wave; ++w) incl += wave_total[w];
      const int start = incl - tot;
      first = start + outside[0][e];
      if (block == 0) {
        expert_offsets[e] = start;
        if (counts_out) counts_out[e] = tot;
        if (e == n_experts - 1) expert_offsets[n_experts] = incl;
      }
    }
  }
  if (e < n_experts) {
    int run = first;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int n = wave_base[w][e];
      wave_base[w][e] = run;
      run += n;
    }
  }
  __syncthreads();
  if (valid) {
    const int pos = wave_base[wave][key] + __popcll(same & ((1ull << lane) - 1ull));
    perm[pos] = (int)a;
    inv_perm[a] = pos;
  }
}

template <RankSource SRC, int NW>
__global__ __launch_bounds__(64 * NW) void permute_rank_kernel(const int32_t* __restrict__ topk_idx, int n_assign,
                                                                  int n_experts, int key_bits,
                                                                  const int32_t* __restrict__ from_before,
                                                                  int32_t* __restrict__ expert_offsets,
                                                                  int32_t* __restrict__ counts_out,
                                                                  int32_t* __restrict__ perm,
                                                                  int32_t* __restrict__ inv_perm) {
  permute_rank_body<SRC, NW>(topk_idx, n_assign, n_experts, key_bits, from_before, expert_offsets, counts_out, perm, inv_perm);
}

// One block routes its tokens a few at a time, so beyond a few dozen tokens the many-block
// route kernel plus the one-block rank kernel are faster than the single launch (measured at 512
// tokens: 10 us against 25 us).
constexpr int ROUTE_PERMUTE_SMALL_T = 64;
constexpr int ROUTE_APART_T = 2048;  // hmoe_router_route_permute: larger batches were routed by hmoe_route, with its checks

// Small batches (T <= 64 and A <= 1024, every decode shape): routing and permutation in ONE block and one launch.
// The block first routes all tokens (lane groups as in hmoe_route; the next group's logits are on their way while one
// is routed), then ranks the assignments it has just made (kept in LDS).  Sixteen waves: 21 tokens of 64 experts, K = 8 were
// routed in six rounds by four waves.
template <int G, int VPL>
__global__ __launch_bounds__(PR_THREADS) void route_permute_small_kernel(const float* __restrict__ logits, int n_tokens,
                                                                         int n_experts, int top_k, int key_bits,
                                                                         int32_t* topk_idx, float* __restrict__ topk_w,
                                                                         int32_t* __restrict__ expert_offsets,
                                                                         int32_t* __restrict__ counts_out,
                                                                         int32_t* __restrict__ perm,
                                                                         int32_t* __restrict__ inv_perm) {
  constexpr int TOKENS_PER_PASS = PR_THREADS / G;
  __shared__ int32_t chosen[PB_CHUNK];  // the ids once more, for the ranking below
  const int gl = threadIdx.x % G;
  uint32_t next[VPL];
  load_keys<G, VPL>(logits, n_experts, threadIdx.x / G, (int)threadIdx.x / G < n_tokens, gl, next);
  for (int t0 = 0; t0 < n_tokens; t0 += TOKENS_PER_PASS) {
    const long token = t0 + threadIdx.x / G;
    uint32_t key[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) key[i] = next[i];
    load_keys<G, VPL>(logits, n_experts, token + TOKENS_PER_PASS, token + TOKENS_PER_PASS < n_tokens, gl, next);
    route_keys<G, VPL>(key, n_experts, top_k, token, token < n_tokens, gl, topk_idx, topk_w, chosen);
  }
  __syncthreads();
  permute_rank_body<RANK_SINGLE, PR_THREADS / 64>(chosen, n_tokens * top_k, n_experts, key_bits, nullptr, expert_offsets, counts_out, perm,
                                 inv_perm);
}

// bf16 batches: router logits and routing in one launch.  A block computes the logits of its tokens (global memory,
// they are an output, and LDS) and routes them from LDS, lane groups as in hmoe_route.
template <int G, int VPL, class SHAPE>
__device__ __forceinline__ void front_tokens_body(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w_g, int hidden,
                                                  float* __restrict__ logits, int n_tokens, int n_experts, int top_k,
                                                  int tokens_per_block, int32_t* __restrict__ topk_idx,
                                                  float* __restrict__ topk_w, int32_t* lds_idx) {
  constexpr int MAX_EXPERTS = SHAPE::EXPERT_FRAGS * 16;
  __shared__ float red[SHAPE::RED];
  __shared__ float lds_logits[SHAPE::MA * 16 * MAX_EXPERTS];
  router_logits_block<SHAPE>(x, w_g, n_tokens, n_experts, hidden, logits, tokens_per_block, red, lds_logits, n_experts);  // ends with a barrier
  constexpr int TOKENS_PER_PASS = SHAPE::THREADS / G;
  const long t0 = (long)blockIdx.x * tokens_per_block;
  for (int l0 = 0; l0 < tokens_per_block; l0 += TOKENS_PER_PASS) {
    const int local = l0 + threadIdx.x / G;
    const bool valid = local < tokens_per_block && t0 + local < n_tokens;
    route_token<G, VPL>(lds_logits, n_experts, top_k, local, valid, threadIdx.x % G, topk_idx + t0 * top_k,
                        topk_w + t0 * top_k, lds_idx);
  }
}

// ... of up to ROUTER_SMALL_T tokens: one block, which permutes as well.
template <int G, int VPL, class SHAPE>
__global__ __launch_bounds__(PR_THREADS) void front_small_kernel(const bf16_t* __restrict__ x,
                                                                 const bf16_t* __restrict__ w_g, int hidden,
                                                                 float* __restrict__ logits, int n_tokens, int n_experts,
                                                                 int top_k, int key_bits, int32_t* topk_idx,
                                                                 float* __restrict__ topk_w,
                                                                 int32_t* __restrict__ expert_offsets,
                                                                 int32_t* __restrict__ counts_out,
                                                                 int32_t* __restrict__ perm,
                                                                 int32_t* __restrict__ inv_perm) {
  static_assert(PR_THREADS == SHAPE::THREADS, "");
  __shared__ int32_t chosen[PB_CHUNK];
  front_tokens_body<G, VPL, SHAPE>(x, w_g, hidden, logits, n_tokens, n_experts, top_k, 16, topk_idx, topk_w, chosen);
  __syncthreads();
  permute_rank_body<RANK_SINGLE, PR_THREADS / 64>(chosen, n_tokens * top_k, n_experts, key_bits, nullptr, expert_offsets, counts_out, perm,
                                 inv_perm);
}

// ... of more: the permutation, which needs every token's choice, stays a launch of its own.
template <int G, int VPL, class SHAPE>
__global__ __launch_bounds__(SHAPE::THREADS, SHAPE::WAVES_PER_SIMD) void front_tokens_kernel(const bf16_t* __restrict__ x,
                                                                      const bf16_t* __restrict__ w_g, int hidden,
                                                                      float* __restrict__ logits, int n_tokens, int n_experts,
                                                                      int top_k, int tokens_per_block, int32_t* topk_idx,
                                                                      float* __restrict__ topk_w) {
  front_tokens_body<G, VPL, SHAPE>(x, w_g, hidden, logits, n_tokens, n_experts, top_k, tokens_per_block, topk_idx, topk_w, nullptr);
}

// x_perm[p, :] = x[perm[p] / K, :], rows of row_bytes (multiple of 16)
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4* __restrict__ x, const int32_t* __restrict__ perm,
                                                          int top_k, int row_vec, int n_assign,
                                                          uint4* __restrict__ x_perm) {
  const int p = blockIdx.x;
  if (p >= n_assign) return;
  const long src = (long)(perm[p] / top_k) * row_vec, dst = (long)p * row_vec;
  for (int i = threadIdx.x; i < row_vec; i += blockDim.x) x_perm[dst + i] = x[src + i];
}

static inline int n_chunks(long n_assign) { return (int)((n_assign + PB_CHUNK - 1) / PB_CHUNK); }

}  // namespace hmoe

extern "C" size_t hmoe_permute_workspace_bytes(const hmoe_layer_desc* desc, int32_t T) {
  if (hmoe::check_desc(desc) != HMOE_OK || T < 0) return 0;
  const long A = (long)T * desc->top_k;
  // per-block counts + one row of counts for the pinned-host copy
  return ((size_t)hmoe::n_chunks(A) + 1) * desc->n_experts * sizeof(int32_t) + 256;
}

// hmoe_permute and hmoe_permute_static share this body; they differ in where the scratch memory comes from.
static int32_t permute_with_workspace(const hmoe_layer_desc* desc, const int32_t* topk_idx, int32_t T, const void* x,
                                      void* x_perm, int32_t* expert_offsets, int32_t* perm, int32_t* inv_perm,
                                      int32_t* h_counts_pinned, void* workspace, size_t workspace_bytes, void* stream) {
  using namespace hmoe;
  int rc = check_desc(desc);
  if (rc != HMOE_OK) return rc;
  if (T < 0 || !expert_offsets) return HMOE_ERR_INVALID_ARG;
  const long A = (long)T * desc->top_k;
  if (A > 0x7fffffffL - PB_CHUNK) return HMOE_ERR_UNSUPPORTED;
  if (A > 0 && (!topk_idx || !perm || !inv_perm)) return HMOE_ERR_INVALID_ARG;
  if ((x == nullptr) != (x_perm == nullptr)) return HMOE_ERR_INVALID_ARG;
  const size_t elem = desc->dtype == HMOE_F32 ? 4 : 2;
  const size_t row_bytes = (size_t)desc->hidden * elem;
  if (x && (row_bytes % 16 != 0)) return HMOE_ERR_UNSUPPORTED;
  if (x && (!aligned16(x) || !aligned16(x_perm))) return HMOE_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < hmoe_permute_workspace_bytes(desc, T)) return HMOE_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & 3u) return HMOE_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const int E = desc->n_experts;
  int key_bits = 0;
  while ((1 << key_bits) < E) ++key_bits;
  const int nblk = n_chunks(A);
  int32_t* block_counts = (int32_t*)workspace;
  int32_t* const counts_host = (int32_t*)device_view_of_pinned(h_counts_pinned);
  int32_t* const counts_dev = counts_host ? counts_host : block_counts + (size_t)(nblk > 0 ? nblk : 0) * E;

#define HMOE_LAUNCH_RANK(SRC, NW, FROM, OFFSETS, COUNTS)                                                              \
  hipLaunchKernelGGL((permute_rank_kernel<SRC, NW>), dim3(A > 0 ? (unsigned)((A + 64 * NW - 1) / (64 * NW)) : 1), dim3(64 * NW), 0, s, \
                     topk_idx, (int)A, E, key_bits, (const int32_t*)(FROM), OFFSETS, COUNTS, perm, inv_perm)
  if (nblk <= 1) {
    HMOE_LAUNCH_RANK(RANK_SINGLE, 16, nullptr, expert_offsets, counts_dev);
  } else if (nblk <= PR_SELF_COUNT_CHUNKS) {
    HMOE_LAUNCH_RANK(RANK_COUNT_ALL, 8, nullptr, expert_offsets, counts_dev);
  } else {
    hipLaunchKernelGGL(permute_hist_kernel, dim3(nblk), dim3(PB_THREADS), 0, s, topk_idx, (int)A, E, block_counts);
    if (nblk <= PR_SELF_SCAN_CHUNKS) {
      HMOE_LAUNCH_RANK(RANK_ADD_UP, 4, block_counts, expert_offsets, counts_dev);
    } else {
      hipLaunchKernelGGL(permute_scan_kernel, dim3(1), dim3(PB_THREADS), 0, s, block_counts, nblk, E, (int)A,
                         expert_offsets, counts_dev);
      HMOE_LAUNCH_RANK(RANK_BASES, 4, block_counts, (int32_t*)nullptr, (int32_t*)nullptr);
    }
  }
#undef HMOE_LAUNCH_RANK
  HMOE_HIP(hipGetLastError());
  if (h_counts_pinned && !counts_host)  // (where kernels cannot write the host memory themselves)
    HMOE_HIP(hipMemcpyAsync(h_counts_pinned, counts_dev, (size_t)E * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  if (x && A > 0) {
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)A), dim3(256), 0, s, (const uint4*)x, perm, desc->top_k,
                       (int)(row_bytes / 16), (int)A, (uint4*)x_perm);
    HMOE_HIP(hipGetLastError());
  }
  return HMOE_OK;
}

extern "C" int32_t hmoe_permute(const hmoe_layer_desc* desc, const int32_t* topk_idx, int32_t T, const void* x,
                                void* x_perm, int32_t* expert_offsets, int32_t* perm, int32_t* inv_perm,
                                int32_t* h_counts_pinned, void* workspace, size_t workspace_bytes, void* stream) {
  return permute_with_workspace(desc, topk_idx, T, x, x_perm, expert_offsets, perm, inv_perm, h_counts_pinned, workspace,
                                workspace_bytes, stream);
}

// ---- hmoe_permute without a workspace from the caller ------------------------------------------------------
// The per-block counts live in a file-scope device array instead.  In host code the array's name is only a
// stand-in: the address the kernels can use comes from hipGetSymbolAddress, once per device (each GPU holds its
// own copy of the array at its own address), and that pointer is what every launch and copy below is given.
static __device__ __align__(256) unsigned char scratch[HMOE_PERMUTE_STATIC_BYTES];

namespace hmoe {
constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` per device, nullptr = not looked up yet
static std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device (looked up on the first call on that device).
static int32_t static_scratch(void** out) {
  int dev = -1;
  HMOE_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return set_error_text(HMOE_ERR_UNSUPPORTED, "hmoe_permute_static: device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    HMOE_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return set_error_text(HMOE_ERR_HIP, "hmoe_permute_static: hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return HMOE_OK;
}
}  // namespace hmoe

extern "C" int32_t hmoe_permute_static(const hmoe_layer_desc* desc, const int32_t* topk_idx, int32_t T, const void* x,
                                       void* x_perm, int32_t* expert_offsets, int32_t* perm, int32_t* inv_perm,
                                       int32_t* h_counts_pinned, void* stream) {
  using namespace hmoe;
  int rc = check_desc(desc);
  if (rc != HMOE_OK) return rc;
  if (T < 0) return HMOE_ERR_INVALID_ARG;
  const size_t need = hmoe_permute_workspace_bytes(desc, T);
  if (need == 0 || need > (size_t)HMOE_PERMUTE_STATIC_BYTES)
    return set_error_text(HMOE_ERR_WORKSPACE, "hmoe_permute_static: T * top_k assignments over n_experts experts need more than the "
                                              "library's static scratch array (HMOE_PERMUTE_STATIC_BYTES); use hmoe_permute");
  void* ws = nullptr;
  rc = static_scratch(&ws);
  if (rc != HMOE_OK) return rc;
  // Nothing in the scratch memory has to start at zero: the histogram kernel writes every per-block count before
  // anything reads it, and the row of per-expert totals is written in full by the scan or by the first rank block.
  return permute_with_workspace(desc, topk_idx, T, x, x_perm, expert_offsets, perm, inv_perm, h_counts_pinned, ws,
                                (size_t)HMOE_PERMUTE_STATIC_BYTES, stream);
}

extern "C" int32_t hmoe_route_permute(const hmoe_layer_desc* desc, const float* logits, int32_t T, int32_t* topk_idx,
                                      float* topk_w, int32_t* expert_offsets, int32_t* perm, int32_t* inv_perm,
                                      int32_t* h_counts_pinned, void* workspace, size_t workspace_bytes, void* stream) {
  using namespace hmoe;
  int rc = check_desc(desc);
  if (rc != HMOE_OK) return rc;
  if (T < 0 || !expert_offsets) return HMOE_ERR_INVALID_ARG;
  const long A = (long)T * desc->top_k;
  if (A > PB_CHUNK || T > ROUTE_PERMUTE_SMALL_T || T == 0) {  // larger batches: the two separate calls
    rc = hmoe_route(desc, logits, T, topk_idx, topk_w, stream);
    if (rc != HMOE_OK) return rc;
    return hmoe_permute(desc, topk_idx, T, nullptr, nullptr, expert_offsets, perm, inv_perm, h_counts_pinned, workspace,
                        workspace_bytes, stream);
  }
  if (!logits || !topk_idx || !topk_w || !perm || !inv_perm) return HMOE_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < hmoe_permute_workspace_bytes(desc, T)) return HMOE_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & 3u) return HMOE_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const int E = desc->n_experts, K = desc->top_k;
  int key_bits = 0;
  while ((1 << key_bits) < E) ++key_bits;
  int32_t* const counts_host = (int32_t*)device_view_of_pinned(h_counts_pinned);
  int32_t* const counts_dev = counts_host ? counts_host : (int32_t*)workspace + (size_t)n_chunks(A) * E;
#define HMOE_LAUNCH_SMALL(G, VPL)                                                                                   \
  hipLaunchKernelGGL((route_permute_small_kernel<G, VPL>), dim3(1), dim3(PR_THREADS), 0, s, logits, (int)T, E, K, key_bits, \
                     topk_idx, topk_w, expert_offsets, counts_dev, perm, inv_perm)
  if (E <= 8) HMOE_LAUNCH_SMALL(8, 1);
  else if (E <= 16) HMOE_LAUNCH_SMALL(16, 1);
  else if (E <= 32) HMOE_LAUNCH_SMALL(32, 1);
  else if (E <= 64) HMOE_LAUNCH_SMALL(64, 1);
  else if (E <= 128) HMOE_LAUNCH_SMALL(64, 2);
  else HMOE_LAUNCH_SMALL(64, 4);
#undef HMOE_LAUNCH_SMALL
  HMOE_HIP(hipGetLastError());
  if (h_counts_pinned && !counts_host)  // (where kernels cannot write the host memory themselves)
    HMOE_HIP(hipMemcpyAsync(h_counts_pinned, counts_dev, (size_t)E * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  return HMOE_OK;
}

extern "C" int32_t hmoe_router_route_permute(const hmoe_layer_desc* desc, const void* x, const void* w_g, int32_t T,
                                             float* logits, int32_t* topk_idx, float* topk_w, int32_t* expert_offsets,
                                             int32_t* perm, int32_t* inv_perm, int32_t* h_counts_pinned, void* workspace,
                                             size_t workspace_bytes, void* stream) {
  using namespace hmoe;
  int rc = check_desc(desc);
  if (rc != HMOE_OK) return rc;
  if (T < 0 || !expert_offsets) return HMOE_ERR_INVALID_ARG;
  const long A = (long)T * desc->top_k;
  if ((T > ROUTER_SMALL_T || A > PB_CHUNK) && desc->dtype != HMOE_F32 && desc->hidden % 16 == 0 && x && w_g && logits && topk_idx &&
      topk_w && aligned16(x) && aligned16(w_g)) {
    // logits and routing in one launch, then the permutation
    // (pointers that hmoe_route refuses; batches that have always been routed with their logits run with any)
    if (T > ROUTE_APART_T && ((reinterpret_cast<uintptr_t>(logits) | reinterpret_cast<uintptr_t>(topk_idx) |
                               reinterpret_cast<uintptr_t>(topk_w)) & 3u))
      return HMOE_ERR_INVALID_ARG;
    const int E = desc->n_experts, K = desc->top_k;
    const int tpb = router_tokens_per_block(T);
    const dim3 grid((unsigned)((T + tpb - 1) / tpb));
#define HMOE_LAUNCH_FRONT_TOKENS(G, VPL, MA, NF, KS, NW)                                                                    \
  hipLaunchKernelGGL((front_tokens_kernel<G, VPL, RouterShape<MA, NF, KS, NW>>), grid, dim3(64 * NW), 0, (hipStream_t)stream, \
                     (const bf16_t*)x, (const bf16_t*)w_g, desc->hidden, logits, (int)T, E, K, tpb, topk_idx, topk_w)
    HMOE_ROUTER_SHAPES_MANY(E, tpb, HMOE_LAUNCH_FRONT_TOKENS);
#undef HMOE_LAUNCH_FRONT_TOKENS
    HMOE_HIP(hipGetLastError());
    return hmoe_permute(desc, topk_idx, T, nullptr, nullptr, expert_offsets, perm, inv_perm, h_counts_pinned, workspace,
                        workspace_bytes, stream);
  }
  if (T == 0 || T > ROUTER_SMALL_T || A > PB_CHUNK || desc->dtype == HMOE_F32) {  // the separate calls
    rc = hmoe_router_logits(desc, x, w_g, T, logits, stream);
    if (rc != HMOE_OK) return rc;
    return hmoe_route_permute(desc, logits, T, topk_idx, topk_w, expert_offsets, perm, inv_perm, h_counts_pinned,
                              workspace, workspace_bytes, stream);
  }
  if (!x || !w_g || !logits || !topk_idx || !topk_w || !perm || !inv_perm) return HMOE_ERR_INVALID_ARG;
  if (desc->hidden % 16 != 0) return HMOE_ERR_UNSUPPORTED;
  if (!aligned16(x) || !aligned16(w_g)) return HMOE_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < hmoe_permute_workspace_bytes(desc, T)) return HMOE_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & 3u) return HMOE_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const int E = desc->n_experts, K = desc->top_k;
  int key_bits = 0;
  while ((1 << key_bits) < E) ++key_bits;
  int32_t* const counts_host = (int32_t*)device_view_of_pinned(h_counts_pinned);
  int32_t* const counts_dev = counts_host ? counts_host : (int32_t*)workspace + (size_t)n_chunks(A) * E;
#define HMOE_LAUNCH_FRONT(G, VPL, MA, NF, KS, NW)                                                                            \
  hipLaunchKernelGGL((front_small_kernel<G, VPL, RouterShape<MA, NF, KS, NW>>), dim3(1), dim3(PR_THREADS), 0, s, (const bf16_t*)x, \
                     (const bf16_t*)w_g, desc->hidden, logits, (int)T, E, K, key_bits, topk_idx, topk_w, expert_offsets,   \
                     counts_dev, perm, inv_perm)
  HMOE_ROUTER_SHAPES_ONE_BLOCK(E, HMOE_LAUNCH_FRONT);
#undef HMOE_LAUNCH_FRONT
  HMOE_HIP(hipGetLastError());
  if (h_counts_pinned && !counts_host)  // (where kernels cannot write the host memory themselves)
    HMOE_HIP(hipMemcpyAsync(h_counts_pinned, counts_dev, (size_t)E * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  return HMOE_OK;
}
