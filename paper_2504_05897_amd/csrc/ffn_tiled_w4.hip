// Prefill FFN over 4-bit expert weights (HMOE_BF16_W4, HMOE_FFN_TILED): the grouped GEMM of ffn_tiled.hip
// with the arithmetic of the 4-bit decode kernel.
//
// Tile: up to 96 rows of one expert x 128 packed weight rows (gate/up: 64 features as gate/up pairs of 16; down: 128
// output columns), 4 waves, two blocks per CU.  An expert's 16-row fragments are dealt evenly to as few tiles as hold
// them, and a tile multiplies the FM fragments it has: with 75 rows per expert one tile of 5 fragments does what two
// tiles of 64 rows, half of the second one padding, did before.  A wave owns two packed 16-row units of the weight matrix
// and all rows, as FM x 2 accumulator tiles of v_mfma_f32_16x16x32_bf16 (tokens are the A operand, weights the B operand);
// twice the running sums (one set per scale group, one for the result) make more than 6 fragments too many registers.
//   * K advances one scale group (128 k) per step.  The activation tile of a step sits in LDS, three stages; the following
//     ones travel global -> registers -> LDS meanwhile.  A row is 16 chunks of 16 bytes; chunk c of row r is stored at
//     position c ^ (r % 16), so the 16 lanes that read the same k block of 16 consecutive rows hit all banks.
//   * The codes of a unit and group are 1 KiB (16 bytes per lane) in operand order and go from global memory
//     to registers, three groups ahead; one bfloat16 scale per lane (= per weight row) and group with them.
//   * As in the decode kernel a dword of eight codes becomes the four operand registers of bfloat16 values
//     128 + q, and   sum_k x_k (q_k - 8) = sum_k x_k (128 + q_k) - 136 sum_k x_k.   The group's sums start from the second
//     term: the row sums of the activation tile, the same for all waves, are multiplied out by the matrix cores one step
//     ahead, each wave some of the fragments, and left in LDS.  Folding a group into the result is then one multiply-add
//     per accumulator register.
//   * What bounds it: the matrix instructions and the vector ALU instructions of a SIMD hardly overlap, so a step takes
//     about the sum of both (5 fragments: 48 and 120), and with few rows the trip to memory that a step waits for.
//   * A tile costs as much as its expert has rows, so the n-tiles of every expert are dealt to the XCDs in turn
//     (locate_tile_spread).
//   * Rows past the end of the expert and units past the end of the matrix are computed from clamped
//     addresses and never stored.
// Measured (8 experts of 4096 x 14336, top 2; gate/up and down launch, tiles of 64 x 256 -> these): 65 tokens 187 -> 118 and
// 145 -> 66 us, 301 tokens 347 -> 262 and 164 -> 137 us, 1003 tokens 649 -> 633 and 387 -> 323 us (0.74 PFLOP/s).  From 320
// rows per expert on the former are the faster ones (ffn_tiled_w4_wide.hip, chosen in launch_stage_tile_w4).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "tile_locate.h"

namespace hmoe {

constexpr int W4T_WAVES = 4;
constexpr int W4T_NU = 2;                      // packed 16-row units per wave
constexpr int W4T_UNITS = W4T_WAVES * W4T_NU;  // per tile: 128 packed rows
constexpr int W4T_FM_MAX = 6;                  // 16-row fragments per tile, at most
constexpr int W4T_RING = 3;                    // scale groups of codes in flight per wave, and activation stages in LDS

// a wave-uniform pointer, held in scalar registers
template <class T>
__device__ __forceinline__ const T* in_scalars(const T* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const T*)(((uint64_t)hi << 32) | lo);
}

template <class T>
using global_ptr = const __attribute__((address_space(1))) T*;

constexpr int W4T_STAGE = W4T_FM_MAX * 16 * 16;  // 16-byte chunks of an activation stage
constexpr int W4T_SUMS = W4T_FM_MAX * 16;         // row sums of a stage
struct __attribute__((aligned(256))) W4TileLds {
  u32x4 a[W4T_RING][W4T_STAGE];                                   // activation stages, [row][16-byte chunk]
  __attribute__((aligned(16))) float xs[2 * W4T_RING * W4T_SUMS + 4 * 64];  // -136 * row sums per stage; a part nothing reads (see sums_at)
};

// (`in` is not declared __restrict__: loads that nothing can alias are moved past a step's barrier, down to their uses.)
// One tile of FM 16-row fragments: rows m0 .. m0 + 16 FM of the expert `loc` names.  A lane addresses its input by a byte
// offset of 32 bits from a scalar base: with a row map the input itself (smaller than 4 GiB, the launch sees to it),
// without one the tile's first row.
template <bool GATEUP, int FM, int KS>
__device__ __forceinline__ void w4_tile(const TiledCtx& c, const TileLoc& loc, const int m0, const bf16_t* in, bf16_t* out, W4TileLds (&lds_of)[KS]) {
  constexpr int THREADS = 64 * W4T_WAVES;
  static_assert(FM * 256 % THREADS == 0, "");
  constexpr int COPIES = FM * 256 / THREADS;  // 16-byte chunks of a stage per thread
  const int K = GATEUP ? c.hidden : c.ffn;
  const int n_out = GATEUP ? c.ffn : c.hidden;
  const int n_groups = K / W4_GROUP, n_steps = (n_groups + KS - 1) / KS;
  const int units_total = (GATEUP ? 2 * c.ffn : c.hidden) / 16;
  const int part_k = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / THREADS);  // scale groups KS g + part_k
  W4TileLds& lds = lds_of[part_k];
  int tid = threadIdx.x % THREADS;
  asm volatile("" : "+v"(tid));  // (opaque: nothing that the tiles of all heights share is kept in registers ahead of the choice)
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  const int j = lane % 16, kblk = lane / 16;

  const char* slot = c.slots + (size_t)loc.slot * c.slot_bytes;
  const W4Offsets off = w4_offsets((size_t)c.hidden, (size_t)c.ffn);
  const u32x4* units = (const u32x4*)(slot + (GATEUP ? 0 : off.down_units));
  const bf16_t* scales = (const bf16_t*)(slot + (GATEUP ? off.gate_up_scales : off.down_scales));
  const u32x4* wq[W4T_NU];
  const bf16_t* ws[W4T_NU];
  const int unit0 = __builtin_amdgcn_readfirstlane(loc.nt) * W4T_UNITS + wave * W4T_NU;  // gate/up: the gate and up unit of features 8 * unit0 .. + 16
#pragma unroll
  for (int u = 0; u < W4T_NU; ++u) {
    const size_t unit = unit0 + u < units_total ? unit0 + u : 0;  // clamped: never stored
    wq[u] = in_scalars(units + unit * (size_t)n_groups * 64);
    ws[u] = in_scalars(scales + unit * (size_t)n_groups * 16);
  }
  // the chunks of a stage this thread moves: chunk id = i * THREADS + tid -> row id / 16, k chunk id % 16
  uint32_t a_src[COPIES];
  const bool mapped = GATEUP && c.row_map;
  const char* const first = in_scalars((const char*)(in + (mapped ? 0 : (size_t)(loc.row_first + m0) * K)));
  const int a_dst = tid / 16 * 16 + ((tid % 16) ^ (tid / 16));  // + i * THREADS: 16 rows further, the same swizzle
  static_assert(THREADS == 256, "a copy instruction of the block moves 16 rows");
#pragma unroll
  for (int i = 0; i < COPIES; ++i) {
    const int r = i * 16 + tid / 16;
    const int row = m0 + r < loc.m_rows ? r : loc.m_rows - 1 - m0;  // of the tile; clamped: never stored
    const int in_row = mapped ? c.row_map[loc.row_first + m0 + row] / c.map_div : row;
    a_src[i] = (uint32_t)in_row * (uint32_t)(2 * K) + 16 * (tid % 16);
  }

  u32x4 codes[W4T_RING][W4T_NU];
  uint32_t scale_bits[W4T_RING][W4T_NU];  // raw bfloat16, converted at use
  auto load_codes = [&](int ring_slot, int g) {
    const int gc = min(KS * g + part_k, n_groups - 1);  // clamped: a group past the end is not added to the result
    uint32_t lane_at = lane;  // (opaque: the offset is widened where it is used and not held as 64 bits)
    asm volatile("" : "+v"(lane_at));
#pragma unroll
    for (int u = 0; u < W4T_NU; ++u) {
      // (wave-uniform addresses in scalar registers, the lane's part as an offset)
      const u32x4* q = wq[u] + (size_t)gc * 64;
      const bf16_t* sc = ws[u] + (size_t)gc * 16;
      asm volatile("" : "+s"(q), "+s"(sc));
      codes[ring_slot][u] = __builtin_nontemporal_load((global_ptr<u32x4>)q + lane_at);
      scale_bits[ring_slot][u] = (uint32_t)((global_ptr<bf16_t>)sc)[lane_at % 16];
    }
  };

  f32x4_t acc[FM][W4T_NU], part[FM][W4T_NU];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int u = 0; u < W4T_NU; ++u) acc[i][u] = part[i][u] = f32x4_t{0, 0, 0, 0};
  float sc_prev[W4T_NU] = {0.0f, 0.0f};
  u32x4 offsets = {0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u};  // bfloat16 -136
  if (FM < W4T_FM_MAX) asm volatile("" : "+v"(offsets));  // (kept in registers where there is room, not made anew for every use)

  // acc += scale * part for row fragment i of the group whose partial sums `part` holds
  auto fold = [&](int i) {
#pragma unroll
    for (int u = 0; u < W4T_NU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][u][r] = fmaf(sc_prev[u], part[i][u][r], acc[i][u][r]);
  };
  // Row sums: one matrix instruction per k-step against a tile of -136.  Wave w answers for fragment w and, of more than
  // four, w / 4 fragments on; where fragments run out, waves repeat one (the same values are written twice).
  // Accumulator register r is row 4 kblk + r of the fragment, and every column holds the same sums: column 0 writes them,
  // the other columns write to a place that nothing reads (a branch would cut the step into pieces for the scheduler).
  const int sums_at = j == 0 ? 4 * kblk : W4T_RING * W4T_SUMS + 4 * lane;
  constexpr int OWN = FM > W4T_WAVES ? 2 : 1;  // fragments per wave
  const int own[2] = {min(wave, FM - 1), min(W4T_WAVES + wave % 2, FM - 1)};
  // Chunk (t, kblk) of row j of fragment i of stage s lies 64 t bytes flipped into the address of k-step 0 plus a constant.
  // One instruction makes it where it is used (opaque: the compiler would hold one address per k-step and stage).
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u32x4*)&lds.a[0][0];
  const uint32_t chunk0 = lds0 + (j * 16 + (kblk ^ j)) * 16;
  auto chunk_at = [&](uint32_t from, int t) {
    uint32_t at;
    asm volatile("v_xor_b32 %0, %1, %2" : "=v"(at) : "s"(64 * t), "v"(from));
    return at;
  };
  auto chunk = [&](uint32_t at, int stage, int i) {
    return *(const __attribute__((address_space(3))) u32x4*)(at + (uint32_t)(stage * W4T_STAGE * 16 + i * 4096));
  };
  const uint32_t own0[2] = {chunk0 + own[0] * 4096, chunk0 + own[1] * 4096};
  auto read_own = [&](int stage, int n, int t) { return chunk(chunk_at(own0[n], t), stage, 0); };
  auto store_sums = [&](int stage, int n, const f32x4_t& xsum) {
    *(f32x4_t*)&lds.xs[stage * W4T_SUMS + own[n] * 16 + sums_at] = xsum;
  };

  // the four operand registers (bfloat16 values 128 + q) of one k-step from its dword of eight codes
  // (the mask lives in a vector register the compiler cannot see through: an and-or with two literal constants
  // would need two instructions, with one operand in a register it is one)
  uint32_t nibbles;
  asm volatile("v_mov_b32 %0, 0x000f000f" : "=v"(nibbles));
  auto unpack = [nibbles](uint32_t d) {
    return u32x4{(d & nibbles) | 0x43004300u, ((d >> 4) & nibbles) | 0x43004300u, ((d >> 8) & nibbles) | 0x43004300u,
                 ((d >> 12) & nibbles) | 0x43004300u};
  };
  u32x4 w[2][W4T_NU], fa[FM];
  // Activation stages reach LDS two steps before they are multiplied; their loads are issued one step before that, or two
  // where a step is shorter than a trip to memory.
  constexpr int AHEAD = FM <= 4 ? 2 : 1;
  u32x4 ahead[AHEAD == 2 ? W4T_RING : 1][COPIES];
  auto load_stage = [&](int stage, int g) {
    const char* from = first + (size_t)min(KS * g + part_k, n_groups - 1) * (2 * W4_GROUP);  // clamped likewise
#pragma unroll
    for (int i = 0; i < COPIES; ++i) ahead[AHEAD == 2 ? stage : 0][i] = *(global_ptr<u32x4>)(from + a_src[i]);
  };
  auto store_stage = [&](int stage) {
#pragma unroll
    for (int i = 0; i < COPIES; ++i) lds.a[stage][i * THREADS + a_dst] = ahead[AHEAD == 2 ? stage : 0][i];
  };

  // ---- prologue: codes of the first groups, activation stages 0 and 1, row sums of stage 0 ------------
  load_stage(0, 0);
  store_stage(0);
  load_stage(1, 1);
  store_stage(1);
  load_stage(2, 2);
  if (AHEAD == 2) load_stage(0, 3);
#pragma unroll
  for (int s = 0; s < W4T_RING; ++s) {  // (in this order, as the steps issue them: see the loop)
    __builtin_amdgcn_sched_barrier(0);
    load_codes(s, s);
  }
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
#pragma unroll
  for (int n = 0; n < OWN; ++n) {
    f32x4_t xsum = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < 4; ++t) xsum = mfma_16x16x32_bf16(read_own(0, n, t), offsets, xsum);
    store_sums(0, n, xsum);
  }
#pragma unroll
  for (int u = 0; u < W4T_NU; ++u) w[0][u] = unpack(codes[0][u][0]);
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();

  // One step: group g, whose codes are in ring slot RS and whose activations are in stage RS.
  auto step = [&](auto ring_slot, const int g) __attribute__((always_inline)) {
    constexpr int rs = decltype(ring_slot)::value, NEXT = (rs + 1) % 3, AFTER = (rs + 2) % 3;
    f32x4_t xv[2];  // -136 * row sums of this group, what its partial sums start from: two fragments at a time
    auto read_sums = [&](int i) { xv[i & 1] = *(const f32x4_t*)&lds.xs[rs * W4T_SUMS + i * 16 + 4 * kblk]; };
#pragma unroll
    for (int i = 0; i < 2 && i < FM; ++i) read_sums(i);
    uint32_t at = chunk0;
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[i] = chunk(at, rs, i);
    __builtin_amdgcn_sched_barrier(0);
    // The next group's row sums, a part in each k-step: step t multiplies the chunks read in the step before
    u32x4 rf[OWN];
    f32x4_t xsum = {0, 0, 0, 0};
#pragma unroll
    for (int n = 0; n < OWN; ++n) rf[n] = read_own(NEXT, 0, n);
    __builtin_amdgcn_sched_barrier(0);
    // This group's partial sums.  The previous group is folded into the running result fragment by fragment right
    // before the first k-step overwrites that fragment's partial sums; the operand registers of k-step t + 1 are
    // unpacked during k-step t, and a fragment is read again for k-step t + 1 right behind the matrix instructions
    // that used it.  The scheduling hints deal the vector ALU instructions out between the matrix instructions.
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (t < 3) at = chunk_at(chunk0, t + 1);
      // operand registers of the next k-step: the next dword of this group, or the first of the next group
#pragma unroll
      for (int u = 0; u < W4T_NU; ++u) w[(t + 1) & 1][u] = unpack(t < 3 ? codes[rs][u][t + 1] : codes[NEXT][u][0]);
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        if (t == 0) fold(i);
#pragma unroll
        for (int u = 0; u < W4T_NU; ++u) part[i][u] = mfma_16x16x32_bf16(fa[i], w[t & 1][u], t == 0 ? xv[i & 1] : part[i][u]);
        if (t == 0 && i + 2 < FM) read_sums(i + 2);
        if (t < 3) fa[i] = chunk(at, rs, i);
      }
#pragma unroll
      for (int n = 0; n < OWN; ++n) xsum = mfma_16x16x32_bf16(rf[n], offsets, xsum);
      if (OWN == 2 && t == 1) {
        store_sums(NEXT, 0, xsum);
        xsum = f32x4_t{0, 0, 0, 0};
      }
      if (t < 3) {
#pragma unroll
        for (int n = 0; n < OWN; ++n)
          rf[n] = OWN == 1 ? read_own(NEXT, 0, t + 1) : read_own(NEXT, (t + 1) / 2, (t + 1) % 2 * 2 + n);
      }
      constexpr int UNPACK = (14 + 2 * FM - 1) / (2 * FM);  // vector ALU instructions per matrix instruction
#pragma unroll
      for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int u = 0; u < W4T_NU; ++u) {
          if (t == 0) __builtin_amdgcn_sched_group_barrier(0x002, 4 + UNPACK, 0);
          else __builtin_amdgcn_sched_group_barrier(0x002, UNPACK, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one matrix instruction
        }
        if (t == 0 && i + 2 < FM) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        else if (t < 3) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one fragment read for the next k-step
      }
      __builtin_amdgcn_sched_group_barrier(0x008, OWN, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    store_sums(NEXT, OWN - 1, xsum);
#pragma unroll
    for (int u = 0; u < W4T_NU; ++u) sc_prev[u] = KS * g + part_k < n_groups ? __uint_as_float(scale_bits[rs][u] << 16) : 0.0f;
    __builtin_amdgcn_sched_barrier(0);
    store_stage(AFTER);  // last read in the previous step, before the barrier that opened this one
    // (the stage's loads ahead of the codes': waiting for them then leaves the codes in flight)
    load_stage(AHEAD == 2 ? NEXT : rs, g + 2 + AHEAD);
    __builtin_amdgcn_sched_barrier(0);
    load_codes(rs, g + W4T_RING);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
  };
  __builtin_amdgcn_s_waitcnt(0x0F70);  // all loads, once per tile: the loop's own counts then hold in its first round too
  // (Whole rounds of the ring, and what is left behind them: with a way out of the middle of the loop, or one past a step,
  // the compiler cannot count the loads in flight and waits for all of them in every step.)
  int g = 0;
  do {  // (steps past the end have scale 0)
    step(std::integral_constant<int, 0>{}, g);
    step(std::integral_constant<int, 1>{}, g + 1);
    step(std::integral_constant<int, 2>{}, g + 2);
    g += 3;
  } while (KS == 1 ? g + 3 <= n_steps : g < n_steps);
  if (KS == 1) {  // (two sets of waves would need registers that they do not have)
    if (g < n_steps) step(std::integral_constant<int, 0>{}, g);
    if (g + 1 < n_steps) step(std::integral_constant<int, 1>{}, g + 1);
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) fold(i);

  // ---- epilogue: accumulator register r of lane (j, kblk) is row 16 i + 4 kblk + r, weight row j of the unit ----
  // A wave's results are 16 (gate/up) or 32 (down) columns wide, a fraction of a 128-byte line.  The tile's results
  // are collected as bf16 in the idle activation stages, [rows][OUTC columns], and stored as whole lines, 16 bytes per
  // thread.  Units past the end (gate/up and down both hold an even number: a wave's pair is all or nothing) are
  // neither collected nor stored.  (The main loop ends with a barrier: every wave has read its last fragments.)
  constexpr int OUTC = GATEUP ? W4T_WAVES * 16 : W4T_WAVES * 32;
  static_assert(FM * 16 * OUTC * 2 <= (int)sizeof(lds.a), "the tile's results must fit the activation stages");
  // (through a copy the compiler cannot see through, so that no address of the epilogue is held over the main loop)
  int tid_out = threadIdx.x;
  asm volatile("" : "+v"(tid_out));
  const int j_out = tid_out % 16, rows_out = 4 * (tid_out % 64 / 16);
  if constexpr (KS == 2) {  // the second half of the block hands its sums to the first
    static_assert(FM * W4T_NU * THREADS <= W4T_RING * W4T_STAGE, "the sums must fit the activation stages");
    f32x4_t* sums = (f32x4_t*)&lds_of[1].a[0][0] + tid_out % THREADS;
    if (part_k == 1) {
#pragma unroll
      for (int i = 0; i < FM * W4T_NU; ++i) sums[i * THREADS] = acc[i / W4T_NU][i % W4T_NU];
    }
    __syncthreads();
    if (part_k == 0) {
#pragma unroll
      for (int i = 0; i < FM * W4T_NU; ++i) acc[i / W4T_NU][i % W4T_NU] += sums[i * THREADS];
    }
  }
  bf16_t* staged = (bf16_t*)&lds_of[0].a[0][0];
  if (part_k == 0 && unit0 < units_total) {
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        bf16_t* srow = staged + (i * 16 + rows_out + r) * OUTC;
        if (GATEUP) {
          srow[wave * 16 + j_out] = f32_to_bf16(silu_f32(acc[i][0][r]) * acc[i][1][r]);
        } else {
          srow[wave * 32 + j_out] = f32_to_bf16(acc[i][0][r]);
          srow[wave * 32 + 16 + j_out] = f32_to_bf16(acc[i][1][r]);
        }
      }
    }
  }
  __syncthreads();
  const int col0 = loc.nt * OUTC;
  for (int id = tid_out; id < FM * 16 * OUTC / 8; id += KS * THREADS) {
    const int row = id / (OUTC / 8), cc = (id % (OUTC / 8)) * 8;
    const int m = m0 + row;
    if (m < loc.m_rows && col0 + cc < n_out)
      *(u32x4*)(out + (size_t)(loc.row_first + m) * n_out + col0 + cc) = *(const u32x4*)(staged + row * OUTC + cc);
  }
}

// KS = 2: two sets of waves take the scale groups in turn, each with its own stages, and add their sums at the end.
// MOST: the most fragments a tile may have.
template <bool GATEUP, int KS, int MOST>
__global__ __launch_bounds__(64 * W4T_WAVES * KS, 2) void ffn_tile_w4_kernel(TiledCtx c, const bf16_t* in, bf16_t* out) {
  static_assert(MOST <= W4T_FM_MAX, "");
  __shared__ W4TileLds lds[KS];
  TileLoc loc;
  if (!(c.spread ? locate_tile_spread<16 * MOST>(c, loc) : locate_tile<16 * MOST>(c, loc))) return;  // uniform over the block
  // the expert's fragments dealt evenly to its m-tiles
  const int mts = (loc.m_rows + 16 * MOST - 1) / (16 * MOST);
  const int frags = (loc.m_rows + 15) / 16, base = frags / mts, rem = frags % mts;
  const int fm = __builtin_amdgcn_readfirstlane(base + (loc.mt < rem ? 1 : 0));
  const int m0 = __builtin_amdgcn_readfirstlane(16 * (loc.mt * base + (loc.mt < rem ? loc.mt : rem)));
#define HMOE_W4_TILE(FM)                                                                              \
  if constexpr (FM <= MOST) {                                                                         \
    if (fm == FM) return w4_tile<GATEUP, FM, KS>(c, loc, m0, in, out, lds);                           \
  }
  HMOE_W4_TILE(1) HMOE_W4_TILE(2) HMOE_W4_TILE(3) HMOE_W4_TILE(4) HMOE_W4_TILE(5) HMOE_W4_TILE(6)
#undef HMOE_W4_TILE
}

template <bool GATEUP, int KS, int MOST>
static void launch_tiles_w4(TiledCtx c, int n_rows, const bf16_t* in, bf16_t* out, hipStream_t s) {
  // (one expert's tiles are as high as each other, and few columns would be too few to divide)
  c.spread = c.n_experts > 1 && (long)std::min(c.n_experts, n_rows) * c.n_tiles_n >= 64;
  c.grid_padded = (int)(c.spread ? blocks_spread(c, n_rows, 16 * MOST) : (tiles_upper_bound(c, n_rows, 16 * MOST) + 7) / 8 * 8);
  hipLaunchKernelGGL((ffn_tile_w4_kernel<GATEUP, KS, MOST>), dim3((unsigned)c.grid_padded), dim3(64 * KS * W4T_WAVES), 0, s, c, in, out);
}

template <bool GATEUP>
static void launch_stage_tile_w4(TiledCtx c, int n_rows, const bf16_t* in, bf16_t* out, hipStream_t s) {
  const int units_total = (GATEUP ? 2 * c.ffn : c.hidden) / 16;
  c.n_tiles_n = (units_total + W4T_UNITS - 1) / W4T_UNITS;
  const long busy = std::min(c.n_experts, n_rows), per_expert = (n_rows + c.n_experts - 1) / c.n_experts;
  auto per = [](long rows, int most) { return (rows + 16 * most - 1) / (16 * most); };  // m-tiles of at most `most` fragments
  // tiles when every expert has as many rows, or the few more that random routing gives some, and when some have twice as
  // many (but no more than all rows can make)
  auto even = [&](int most) { return busy * per(per_expert, most) * (long)c.n_tiles_n; };
  const long likely = busy == 1 ? n_rows : per_expert + (long)(2.0 * std::sqrt((double)per_expert));
  const long likely6 = busy * per(likely, 6) * (long)c.n_tiles_n;
  auto uneven = [&](int most) {
    const long all = busy == 1 ? per(n_rows, most) : std::min(busy * per(2 * per_expert, most), n_rows / (16 * most) + busy);
    return all * (long)c.n_tiles_n;
  };
  // At most one tile per CU (down projections, few experts): a CU then holds one wave per SIMD, and two sets of waves per
  // tile fill it (down projection above: 301 tokens 158 -> 137 us, 150 tokens 101 -> 82 us, 77 tokens 76 -> 66 us).  With
  // more tiles two blocks share a CU anyway.
  // The most fragments a tile may have: six, which read and unpack a weight for 96 rows -- unless lower tiles make no more
  // rounds either (a step of 6, 4 and 2 fragments takes about 1.4, 1 and 0.6), also if some experts have more rows than
  // average.  Layers, six at most -> now: one expert of 1024 x 512, 64 tokens 36.9 -> 26.9 us; one of 2048 x 2816, 301 tokens
  // 57.9 -> 42.7 us (tiles of 64 rows and 256 columns before either: 46.5 and 63 us); one of 3584 x 20480, 1003 tokens,
  // down launch 287 -> 211 us (200).
  // (Two sets with six fragments need a K range to share: below 16 scale groups two blocks of four are faster, one expert
  // of 1024 x 512, 3000 tokens 50 -> 44 us.)
  const bool two6 = likely6 <= 256 && ((GATEUP ? c.hidden : c.ffn) >= 16 * W4_GROUP || uneven(4) > 512);
  const int most = uneven(2) <= 256 ? 2 : uneven(4) <= 256 || (!two6 && uneven(4) <= 512) ? 4 : 6;
  const bool two_sets = most == 6 ? two6 : uneven(most) <= 256;
  // Tiles of 64 x 256 (one block per CU) for experts of 320 rows or more, where the activations are read often enough to
  // count, unless they make more rounds: a round of them takes about 0.92 of one of two blocks of 4 fragments.  Launches,
  // these tiles / the others: 8 experts of 4096 x 14336, 375 rows each, gate/up 853 / 879 us and down 502 / 493, 512 rows
  // 1156 / 1251 and 630 / 617, 1024 rows 2329 / 2467 and 1168 / 1263, but 250 rows 649 / 633 and 387 / 323; one expert of
  // 3584 x 20480, 2048 rows 755 / 790 and 380 / 461; one of 2048 x 2816, 1000 rows (layer) 85 / 67.  They also take tokens of
  // 4 GiB or more, which the others cannot address through a row map.
  const bool far = GATEUP && c.row_map && (size_t)(n_rows / c.map_div) * (size_t)c.hidden * 2 > 0xffffffffu;
  const long wide = busy * ((per_expert + W4_WIDE_ROWS - 1) / W4_WIDE_ROWS) * ((16l * units_total + W4_WIDE_COLUMNS - 1) / W4_WIDE_COLUMNS);
  const double rounds_wide = 0.92 * (double)((wide + 255) / 256);
  const double rounds = (most == 4 ? 1.0 : 1.41) * (double)((even(most) + 511) / 512);
  if (far || (per_expert >= 320 && !two_sets && rounds_wide < rounds)) return launch_stage_w4_wide(GATEUP, c, n_rows, in, out, s);
  if (two_sets) {
    if (most == 2) launch_tiles_w4<GATEUP, 2, 2>(c, n_rows, in, out, s);
    else if (most == 4) launch_tiles_w4<GATEUP, 2, 4>(c, n_rows, in, out, s);
    else launch_tiles_w4<GATEUP, 2, 6>(c, n_rows, in, out, s);
  } else if (most == 4) {
    launch_tiles_w4<GATEUP, 1, 4>(c, n_rows, in, out, s);
  } else {
    launch_tiles_w4<GATEUP, 1, 6>(c, n_rows, in, out, s);
  }
}

int launch_ffn_tiled_w4(const FfnArgs& a) {
  const hmoe_layer_desc& d = *a.desc;
  if (d.dtype != HMOE_BF16_W4) return HMOE_ERR_UNSUPPORTED;
  if (a.n_rows == 0) return HMOE_OK;
  TiledCtx c{a.offsets, a.slot_of, a.slots, a.slot_bytes, a.active, d.n_experts, d.hidden, d.ffn, 0, 0, a.row_map, a.map_div};
  probe_before(a.stream);
  launch_stage_tile_w4<true>(c, a.n_rows, (const bf16_t*)a.x_perm, (bf16_t*)a.h, a.stream);
  probe_after(a.stream);
  probe_before(a.stream);
  launch_stage_tile_w4<false>(c, a.n_rows, (const bf16_t*)a.h, (bf16_t*)a.o_perm, a.stream);
  probe_after(a.stream);
  HMOE_HIP(hipGetLastError());
  return HMOE_OK;
}

}  // namespace hmoe
