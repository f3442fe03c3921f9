// Chunked-prefill attention for gfx950 on bf16 MFMA (the paper, Section 5:
// prefill is compute bound and a chunk attends to all earlier context, so
// chunking splits the same work; Section 1: max_num_batched_tokens bounds
// the chunk).
//
// Work tile = (kv head g, 32 * 8 / G consecutive new rows of one sequence),
// G = 1, 2, 4 or 8 query heads per kv head.
// A workgroup of 8 wavefronts (two per SIMD) owns one tile: wave w serves
// query head g * G + w % G over 32 rows. K/V steps of 64 keys (4 blocks) are
// gathered through the block table straight into LDS (global_load_lds) once
// per workgroup and shared by the G query heads of the group; three LDS
// buffers each let K be gathered three steps and V one step ahead of their
// use, with one barrier per step.
//
// Per wave and step, with v_mfma_f32_32x32x16_bf16:
//   S^T[key][row] = K[key][:] . Q[row][:]   A = K rows read from the
//       chunk-major K tile, B = Q^T held in registers for the whole kernel.
//       The A rows of a 32-key tile are loaded in a permuted key order so
//       that the accumulator of each lane ends up holding 8 consecutive keys
//       of each of the two blocks for one query row;
//   softmax over keys in the log2 domain against a per-row reference (a
//       past row max): a row's 64 scores live in two lanes (l and l + 32)
//       and the row state is lane-local. The reference is only moved, and
//       O^T and the row sum rescaled, when the row's max grows past it by
//       more than 2^8, so every exponential stays below 256, which bf16 P
//       and fp32 accumulation hold. A lane's exponentials are at most its
//       partial row sum, so a step whose partial sums all stay within 2^8
//       (nearly every step after the first) needs no row max at all; the
//       others take the exact max (one exchange between the row's two
//       lanes) and recompute the step's exponentials;
//   O^T[d][row] += V^T[d][key] P^T[key][row]   A = 16-byte runs of the
//       dim-major V tile, B = the bf16 P values of 8 consecutive keys of one
//       block, already in the lane that produced them.
// Software pipeline: while a wave computes the softmax of step i on the
// vector ALU, its matrix work is p.v of step i - 1 and q.k of step i + 1, so
// both units stay busy; the second wave of the SIMD covers the LDS latency.
// V rows are stored in LDS with their two 16-byte halves swapped on every
// other group of 8 rows, so the A reads of 16 rows hit 16 distinct bank
// groups. The causal mask (bottom-right: row i at position L - n + i sees
// keys 0 .. L - n + i) is applied only on steps that reach the diagonal or
// the end of the sequence.

#include <type_traits>

#include "common.hpp"
#include "decode_walk.hpp"
#include "launch.hpp"

namespace kvattn {

namespace {

constexpr int kD = 128;
constexpr int kBS = 16;
constexpr int kKeys = 64;                  // keys per step
constexpr int kStepBlocks = 4;             // blocks per step
constexpr int kTileBytes = kBS * kD * 2;   // one (block, K/V, head) tile: 4 KiB
constexpr float kLazyRescale = 8.f;        // log2 headroom before the max moves
constexpr float kPsumBound = 256.f;         // 2^kLazyRescale
constexpr int kKBufs = 3;                  // LDS K steps (gathered three steps ahead)
constexpr int kVBufs = 3;                  // LDS V steps (gathered one step ahead)
constexpr int kWaves = 8;                  // wavefronts per workgroup
constexpr int kThreads = kWaves * kWave;
constexpr int kNumCUs = 256;               // gfx950

typedef float f32x16_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16_t mfma32(bf16x8_t a, bf16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// max(a, b, c) in one instruction. The scores here are never NaN (masked
// keys are set to -inf by a select), so the IEEE NaN handling that fmaxf
// adds around every operand is not needed.
__device__ __forceinline__ float max3f(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Two loads of 16 bytes per lane from global memory straight into LDS
// (global_load_lds_dwordx4): load j has lane l read base_j + off_j and its
// bytes land at LDS byte address lds_j + 16 l (base_j and lds_j wave-uniform,
// in SGPRs). A wave-uniform base plus a 32-bit lane offset takes the address
// unit fewer cycles per instruction than 64 lanes of 64-bit addresses. M0
// carries each load's LDS address: the block saves the compiler's M0 first
// and restores it last, so no code outside the block sees M0 change. Issued
// as inline assembly so that the compiler does not treat the loads as LDS
// stores that every later LDS read must wait for: the callers wait for them
// themselves (s_waitcnt vmcnt) before the barrier that publishes the data.
__device__ __forceinline__ void dma16x2(const void* base0, uint32_t off0, uint32_t lds0,
                                        const void* base1, uint32_t off1, uint32_t lds1) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %3\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2\n\t"
      "s_mov_b32 m0, %6\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %4, %5\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(off0), "s"(base0), "s"(lds0), "v"(off1), "s"(base1), "s"(lds1)
      : "memory");
}

// Entry i of a block-table row, read by a scalar memory load: the row pointer
// is wave-uniform and the index is made so, and a load through the constant
// address space from a uniform address is a scalar load. It is therefore
// counted by lgkmcnt, never by the vmcnt that the gathers are waited with.
__device__ __forceinline__ int scalar_entry(const int* row, int i) {
  const __attribute__((address_space(4))) int* p =
      (const __attribute__((address_space(4))) int*)row;
  return p[(unsigned)__builtin_amdgcn_readfirstlane(i)];
}

typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef i32x4_t i32x4_a4_t __attribute__((aligned(4)));

// Entries i .. i + 3 of a block-table row in one 16-byte scalar load (scalar
// loads need only 4-byte alignment).
__device__ __forceinline__ i32x4_t scalar_entries4(const int* row, int i) {
  const __attribute__((address_space(4))) i32x4_a4_t* p =
      (const __attribute__((address_space(4))) i32x4_a4_t*)(
          row + (unsigned)__builtin_amdgcn_readfirstlane(i));
  return *p;
}

// LDS byte address of a pointer into a __shared__ array.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// The lane's index in its wavefront, computed afresh at each call (volatile,
// so it is not merged with an earlier copy that would have to stay live).
__device__ __forceinline__ int lane_id_fresh() {
  int r;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(r));
  return r;
}

}  // namespace

// Rows [lo, hi) of sequence s's chunk, with the offsets clamped into
// [0, total_q] and hi >= lo, so that offsets that break the documented
// contract (decreasing, or past the end of q) can neither read nor write
// outside q and out.
__device__ __forceinline__ int2 chunk_rows(const int* __restrict__ cu, int s, int total_q) {
  const int lo = min(max(cu[s], 0), total_q);
  const int hi = min(max(cu[s + 1], lo), total_q);
  return make_int2(lo, hi);
}

// Lists the work tiles (sequence, first row) of a batch of chunks, the rows
// of a sequence's chunk in descending order so the longest rows start first.
__global__ __launch_bounds__(256) void prefill_tile_map_kernel(const int* __restrict__ cu,
                                                               int num_seqs, int total_q,
                                                               int rows_per_tile,
                                                               int2* __restrict__ tiles,
                                                               int* __restrict__ count,
                                                               int max_tiles) {
  __shared__ int scan[256];
  const int tid = threadIdx.x;
  const int per = (num_seqs + 255) / 256;
  const int s0 = min(num_seqs, tid * per);
  const int s1 = min(num_seqs, s0 + per);
  int mine = 0;
  for (int s = s0; s < s1; ++s) {
    const int2 r = chunk_rows(cu, s, total_q);
    mine += (r.y - r.x + rows_per_tile - 1) / rows_per_tile;
  }
  scan[tid] = mine;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {
    const int v = tid >= o ? scan[tid - o] : 0;
    __syncthreads();
    scan[tid] += v;
    __syncthreads();
  }
  int off = scan[tid] - mine;
  for (int s = s0; s < s1; ++s) {
    const int2 r = chunk_rows(cu, s, total_q);
    const int nt = (r.y - r.x + rows_per_tile - 1) / rows_per_tile;
    for (int k = 0; k < nt; ++k) {
      if (off < max_tiles) tiles[off] = make_int2(s, (nt - 1 - k) * rows_per_tile);
      ++off;
    }
  }
  if (tid == 255) *count = min(scan[255], max_tiles);
}

// ---- planned steps ----
//
// With the workspace kvattn_prefill_workspace_bytes asks for, a step's work is
// laid out by a plan kernel. An item is a run of key steps of one work tile
// (for all kv heads); a tile whose keys are shared by several items leaves a
// partial state per item in a slot, and prefill_combine_kernel merges them.
// A tile is a serial walk of about 1.7 us per key step, one workgroup per CU,
// so a step with few tiles leaves CUs idle, and one whose tiles do not divide
// by the CUs idles them in its last round. A call at 32 query heads over 8,
// whole tiles in sequence order against planned items:
//   201 rows over 6150 cached tokens (32 workgroups of 100 steps)  162 -> 44 us
//   512 rows over 8192                                             215 -> 88 us
//   1024 rows over 1024                                             62 -> 53 us
//   9 chunks of 100 to 900 rows over 1000 to 8000 tokens           443 -> 367 us
//   8192 rows over 24576 (four even rounds, not shared)           3274, 3278 us
// Items go by length over all sequences. Of 15 steps of 3 to 20 chunks that share
// nothing, 13 gain up to 11% by it against sequence by sequence or stay, and two of
// sequences alike lose 5%: 9 chunks of 300 to 600 rows over 1500 to 3000 tokens, 64
// query heads over 8, 306 -> 323 us, 9 of 113 to 679 over 1722 to 3445 275 -> 289.
// Coarser lengths (8 or 32 classes instead of 256) give 2% back on the first and
// lose up to 3% on others.
//
// A sequence that adds one row (a decode sequence in a unified step) is no tile:
// its tile would put one row of each head through 32-row products and stage its
// whole context through LDS for them. It takes decode's walk instead, a
// workgroup's eight wavefronts sharing an item's tokens. Such items are bound by
// HBM and tiles by the matrix units, so the plan lets them run side by side. A
// call at 32 query heads over 8, one-row sequences as tiles against this:
//   2048 rows over 6144 cached tokens, 128 one-row of 1024 to 8192   645 -> 435 us
//   8192 rows over 24576, the same 128                             3667 -> 3477 us
//   two chunks of 5 and 9 rows, 100 one-row of 1024 to 8192          371 -> 306 us
//   64 query heads: 512 rows over 1000, 40 one-row of 1024 to 8192   268 -> 142 us

struct PrefillItem {
  int s, q0;        // sequence, first row of the tile in the chunk (-1: one-row item)
  int i0, i1;       // key steps, i0 even (one-row item: tokens, i0 a multiple of 64)
  int slot;         // partial slot, -1: written to out
  int cu0, n, L;    // the sequence's chunk and clamped length
};

struct PrefillSplit {   // a tile shared by several items
  int row0, rows;       // its rows in q and out
  int slot0, pieces;
};

struct RowSplit {       // a one-row sequence shared by several items
  int row, slot0, pieces, pad;
};

struct PrefillPlan {
  int items, splits, row_splits, pad;
};

// A slot holds, for each of the 8 wavefronts of a tile and its 32 rows, O
// unnormalised in fp32 as [dim pair][row] and (reference max, row sum).
constexpr int kSlotFloats = kWaves * 32 * kD;
constexpr size_t kSlotBytes = kSlotFloats * sizeof(float) + kWaves * 32 * sizeof(float2);

// A one-row slot: O [G][kD] and (max, row sum) [G], whole 16 bytes.
constexpr size_t row_slot_bytes(int group) {
  return ((size_t)group * (kD * sizeof(float) + sizeof(float2)) + 15) & ~size_t(15);
}

constexpr int kPlanThreads = 512;
constexpr int kPlanCandidates = 16;
// Estimated cost, in key steps, of an item's prologue and epilogue, and of
// writing and merging a partial.
constexpr int kItemSteps = 3, kPartialSteps = 6;
// A one-row item's time per 64 tokens and kv head, in key steps: on its CU
// (eight wavefronts, a step of about 2 us each), and of the whole chip's HBM
// time (32 KiB at 4.6 TB/s: the tiles beside it read too). 2048 rows over 6144
// cached tokens with 128 one-row sequences of 1024 to 8192: 502 / 443 / 435 /
// 502 us at 0.15 / 0.3 / 0.5 / 0.8 with the HBM term at 0.0031, and 441 / 439 /
// 430 / 438 us at 0.0015 / 0.0031 / 0.0045 / 0.006; 512 rows over 1000 with 40
// of them 141 / 141 / 149 / 150 us and 141 / 141 / 143 / 143.
constexpr float kRowStep = 0.3f, kRowHbmStep = 0.0042f;
constexpr int kRowTokens = 1024;   // fewest tokens of a shared sequence's item
constexpr int kCombineParts = 4;   // workgroups over the dims of a merge
constexpr int kCombineGrid = 1024;

struct PlanArgs {
  const int* cu;
  const int* seq_lens;
  int num_seqs, total_q, rows_per_tile, num_kv_heads, max_seq_tokens;
  int max_items, max_slots;   // max_slots 0: no tile is shared
  int rows, max_row_slots;    // rows 0: one-row sequences are tiles
  PrefillItem* items;
  PrefillSplit* splits;
  RowSplit* row_splits;
  PrefillPlan* head;
};

// Whether sharing tiles can gain more than it costs, for a call whose longest
// tile walks this many key steps and whose tiles are this many workgroups: below
// eight steps an item's own cost outweighs what it saves, four or more rounds of
// tiles gain nothing, and up to 64 steps the longest walk, over the part of the
// last round that is idle, has to be min_steps. The host asks with its bounds
// whether the wider plan and the merge are worth a launch. 32 query heads over 8,
// whole tiles, shared, and not shared by that rule:
//   2 of 770 rows over 50                         36 / 38 / 33 us
//   9 of 176 over 692, with 2 one-row             38 / 46 / 35 us
//   440 rows over 227                             29 / 31 / 27 us
// and shared by it: 53 -> 41 us (1673 rows with 15 one-row, 8 query heads over 8).
// With a loose bound it launches them, and the plan asks whether to weigh
// candidates, with the lengths. Not shared / shared, under a bound of 131072 (the
// longest walk over the idle part): 512 rows over 256 (9.0) 29.8 / 32.2 us, 200
// over 512 (10.5) 28.5 / 27.1, 1024 over 256 (10.0) 41.9 / 39.5, 1024 over 1024
// (16.0) 59.3 / 53.3.
constexpr int kLaunchSteps = 16, kPlanSteps = 10;
__host__ __device__ __forceinline__ bool sharing_pays(long long steps, long long workgroups,
                                                      int min_steps) {
  const long long chip = workgroups > kNumCUs ? (workgroups + kNumCUs - 1) / kNumCUs * kNumCUs
                                              : kNumCUs;
  return steps > 8 && workgroups < 4 * kNumCUs &&
         (steps > 64 || steps * (chip - workgroups) >= min_steps * chip);
}

// Steps per item and items of a tile of N steps, at most C steps per item.
__device__ __forceinline__ int2 tile_pieces(int N, int C) {
  const int p = (N - 1) / C + 1;
  if (N <= 0 || p <= 1) return make_int2(max(N, 0), 1);
  const int per = (((N + p - 1) / p) + 1) & ~1;   // whole pairs of steps
  return make_int2(per, (N + per - 1) / per);
}

// Tokens per item and items of a one-row sequence of L tokens, at most C
// tokens (a multiple of 64) per item.
__device__ __forceinline__ int2 row_pieces(int L, int C) {
  const int p = (L - 1) / C + 1;
  if (L <= 0 || p <= 1) return make_int2(max(L, 0), 1);
  const int per = ((L - 1) / p / kKeys + 1) * kKeys;
  return make_int2(per, (L - 1) / per + 1);
}

// Exclusive prefix sums of v and of flag over the workgroup, and their totals.
struct PlanScan {
  int before, total, set_before, set_total;
};
__device__ __forceinline__ PlanScan plan_scan(int v, bool flag, int2* lds) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  int x = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int y = __shfl_up(x, o, kWave);
    x += lane >= o ? y : 0;
  }
  const unsigned long long set = __ballot(flag);
  if (lane == kWave - 1) lds[wave] = make_int2(x, (int)__popcll(set));
  __syncthreads();
  PlanScan r = {x - v, 0, (int)__popcll(set & ((1ull << lane) - 1)), 0};
#pragma unroll
  for (int w = 0; w < kPlanThreads / kWave; ++w) {
    const int2 e = lds[w];
    r.before += w < wave ? e.x : 0;
    r.total += e.x;
    r.set_before += w < wave ? e.y : 0;
    r.set_total += e.y;
  }
  __syncthreads();
  r.total = __builtin_amdgcn_readfirstlane(r.total);
  r.set_total = __builtin_amdgcn_readfirstlane(r.set_total);
  return r;
}

// Sums and maxima over the workgroup, in one order whatever the timing: a
// wavefront's by its fixed tree, then the wavefronts' one after another.
struct PlanTotals {
  float steps, tokens;           // sums: they only feed estimates
  float max_steps, max_tokens;
};
__device__ __forceinline__ PlanTotals plan_totals(PlanTotals v, PlanTotals* lds) {
  v = {wave_sum(v.steps), wave_sum(v.tokens), wave_max(v.max_steps), wave_max(v.max_tokens)};
  if (threadIdx.x % kWave == 0) lds[threadIdx.x / kWave] = v;
  __syncthreads();
  PlanTotals r = lds[0];
#pragma unroll
  for (int w = 1; w < kPlanThreads / kWave; ++w) {
    const PlanTotals e = lds[w];
    r = {r.steps + e.steps, r.tokens + e.tokens, fmaxf(r.max_steps, e.max_steps),
         fmaxf(r.max_tokens, e.max_tokens)};
  }
  return r;
}

// Tile t of a chunk of sequences: its sequence's index in the chunk, first row,
// key steps.
struct PlanTile {
  int idx, q0, N;
};

struct PlanChoice {
  int limit, x, y;              // steps per item; CUs / kv heads for tiles, for one-row items
  float tile_time, row_time;    // a tile item's time; a one-row item's on its CU
};

// Latency-bound, one workgroup ahead of the attention kernel. kResident: the
// sequences fit one chunk (512) and their tiles one per thread, the usual case,
// and each thread keeps its tile in registers over all passes. A call that runs in
// one round needs no order and is written at once, also with one-row sequences: 2.5
// us (rocprof), as the tile map. Ordering takes 5.4, candidates to weigh or one-row
// sequences to mix in 7.1, both 10.0. A call of 143 rows with 16 one-row sequences
// under 814 tokens, 8 query heads over 8, took 23.8 us with the ordering passes and
// takes 19.8, 9 of 176 over 692 with 2, 32 over 8, 39.5 and 35.0.
template <bool kResident>
__global__ __launch_bounds__(kPlanThreads) void prefill_plan_kernel(PlanArgs args) {
  __shared__ int seq_cu[kPlanThreads], seq_n[kPlanThreads], seq_L[kPlanThreads];
  __shared__ int first[kPlanThreads + 1];     // first tile of each sequence of the chunk
  __shared__ int2 scan_lds[kPlanThreads / kWave];
  __shared__ int hist[256], row_hist[256], steps[kPlanThreads];
  __shared__ PlanTotals totals_lds[kPlanThreads / kWave];
  __shared__ int extra_row_items, next_slot, next_split, next_row_slot, next_row_split,
      row_slots_needed;
  __shared__ int cand_items[kPlanCandidates], cand_slots[kPlanCandidates];
  __shared__ PlanChoice choice;
  const int tid = threadIdx.x;
  PlanArgs a = args;
  if constexpr (!kResident) {
    // kept in vector registers: the nested loops leave too few scalar ones
    __shared__ PlanArgs lds_args;
    if (tid == 0) lds_args = args;
    __syncthreads();
    a = lds_args;
    a.num_seqs = args.num_seqs;   // the bound of the loops with barriers stays uniform
  }
  const int R = a.rows_per_tile;
  const int seqs = min(a.num_seqs, kPlanThreads);   // sequences of a chunk, at most

  // Loads sequences base .. base + 511 and numbers their tiles.
  auto load_chunk = [&](int base) {
    const int s = base + tid;
    int nt = 0;
    bool row = false;
    if (s < a.num_seqs) {
      const int len = a.seq_lens[s];
      const int2 r = chunk_rows(a.cu, s, a.total_q);
      seq_cu[tid] = r.x;
      seq_n[tid] = r.y - r.x;
      seq_L[tid] = min(max(len, 0), a.max_seq_tokens);
      row = a.rows && r.y - r.x == 1;
      nt = row ? 0 : (r.y - r.x + R - 1) / R;
    }
    const PlanScan at = plan_scan(nt, row, scan_lds);
    first[tid] = at.before;
    if (tid == 0) first[kPlanThreads] = at.total;
    __syncthreads();
    return at;   // of tiles and one-row sequences
  };
  // The rows of a sequence are taken in descending order.
  auto tile_of = [&](int t) {
    int lo = 0, hi = seqs - 1;   // last sequence with first <= t, which has tiles
    while (lo < hi) {
      const int mid = (lo + hi + 1) / 2;
      if (first[mid] <= t) lo = mid; else hi = mid - 1;
    }
    PlanTile r;
    const int nt = (lo + 1 < kPlanThreads ? first[lo + 1] : first[kPlanThreads]) - first[lo];
    const int n = seq_n[lo], L = seq_L[lo];
    r.idx = lo;
    r.q0 = (nt - 1 - (t - first[lo])) * R;
    const int last_pos = min(L - n + r.q0 + min(R, n - r.q0) - 1, L - 1);
    r.N = last_pos >= 0 ? last_pos / kKeys + 1 : 0;
    return r;
  };

  if (tid == 0) {
    extra_row_items = 0;
    next_slot = 0;
    next_split = 0;
    next_row_slot = 0;
    next_row_split = 0;
    row_slots_needed = 0;
  }
  if (tid < 256) {
    hist[tid] = 0;
    row_hist[tid] = 0;
  }
  const PlanScan found = load_chunk(0);   // its barriers also publish the zeros above
  // tiles (of all kv heads) that run at once, one workgroup per CU
  const int lanes = max(1, kNumCUs / a.num_kv_heads);
  int chunk_tiles = kResident ? min(found.total, kPlanThreads) : found.total;
  int all_tiles = chunk_tiles, all_rows = found.set_total;
  PlanTile own = {0, 0, 0};
  // Whole tiles and one-row sequences that all run at once, in any order.
  const bool one_round = kResident && chunk_tiles + all_rows <= min(lanes, a.max_items);
  auto write_whole = [&] {
    if (tid < chunk_tiles)
      a.items[tid] = {own.idx, own.q0, 0, own.N, -1, seq_cu[own.idx], seq_n[own.idx],
                      seq_L[own.idx]};
    if (a.rows && tid < a.num_seqs && seq_n[tid] == 1)
      a.items[chunk_tiles + found.set_before] = {tid, -1, 0, seq_L[tid], -1, seq_cu[tid], 1,
                                                 seq_L[tid]};
    if (tid == 0) *a.head = {chunk_tiles + all_rows, 0, 0, 0};
  };
  if constexpr (kResident) {
    if (tid < chunk_tiles) own = tile_of(tid);
    steps[tid] = own.N;
    if (one_round && a.max_slots == 0 && a.max_row_slots == 0) {
      write_whole();
      return;
    }
  }
  // Runs tile(base, t) over every tile, dealt to the threads in turn, and
  // row(sequence, cu0, L) over every one-row sequence.
  auto each = [&](auto tile, auto row) {
    if constexpr (kResident) {
      if (tid < chunk_tiles) tile(0, own);
      if (a.rows && tid < a.num_seqs && seq_n[tid] == 1) row(tid, seq_cu[tid], seq_L[tid]);
    } else {
      all_tiles = all_rows = 0;
      for (int base = 0; base < a.num_seqs; base += kPlanThreads) {
        const PlanScan chunk = load_chunk(base);
        chunk_tiles = chunk.total;
        all_tiles += chunk_tiles;
        all_rows += chunk.set_total;
        for (int t = tid; t < chunk_tiles; t += kPlanThreads) tile(base, tile_of(t));
        if (a.rows && base + tid < a.num_seqs && seq_n[tid] == 1)
          row(base + tid, seq_cu[tid], seq_L[tid]);
        __syncthreads();
      }
    }
  };

  // ---- totals ----
  PlanTotals sum = {0.f, 0.f, 1.f, 1.f};
  each(
      [&](int, const PlanTile& t) {
        sum.steps += t.N;
        sum.max_steps = fmaxf(sum.max_steps, t.N);
      },
      [&](int, int, int L) {
        sum.tokens += L;
        sum.max_tokens = fmaxf(sum.max_tokens, L);
      });
  sum = plan_totals(sum, totals_lds);
  const int tiles = all_tiles, rows = all_rows;
  const int longest = (int)sum.max_steps, max_tokens = (int)fminf(sum.max_tokens, 1e9f);
  const float steps_sum = sum.steps, tokens_sum = sum.tokens;
  constexpr int kWhole = 0x7fffffff;

  // ---- one-row sequences: at least two items per CU, whole above that ----
  int row_c = kWhole, row_items = rows;
  if (rows > 0 && a.max_row_slots > 0)
    row_c = max(kRowTokens, ((int)fminf(tokens_sum / (2 * lanes), 1e9f) / 512 + 1) * 512);
  const bool share = kResident && a.max_slots > 0 &&
                     sharing_pays(longest, (long long)tiles * a.num_kv_heads, kPlanSteps);
  if constexpr (kResident) {
    if (one_round && !share && max_tokens <= row_c) {
      write_whole();
      return;
    }
  }
  if (max_tokens > row_c) {
    each([](int, const PlanTile&) {},
         [&](int, int, int L) {
           const int p = row_pieces(L, row_c).y;
           if (p > 1) {
             atomicAdd(&row_slots_needed, p);
             atomicAdd(&extra_row_items, p - 1);
           }
         });
    __syncthreads();
    if (row_slots_needed > a.max_row_slots) row_c = kWhole;
    else row_items += extra_row_items;
  }
  const float row_steps = tokens_sum / 64.f;
  const float row_work = kRowStep * row_steps + (float)kItemSteps * row_items;
  const float row_hbm = kRowHbmStep * a.num_kv_heads * row_steps;

  // ---- how many steps an item gets, and how tiles and one-row items mix ----
  // Candidate k limits an item to 1 / (k + 1) of the longest tile. Its time is
  // estimated as r rounds of its items on the fewest CUs that do them in r
  // rounds, while the one-row items run on the others as far as those and HBM
  // allow, and the rest of them after; without one-row items r is as few as
  // fit. The fewest items within 3% of the best win.
  PlanChoice pick = {kWhole, 1, 0, 1.f, 1.f};   // whole tiles, nothing to mix
  if (share || rows) {
    constexpr int kPer = kPlanThreads / kPlanCandidates;   // 32 lanes per candidate
    auto limit = [&](int k) { return k ? max(4, ((longest + k) / (k + 1) + 1) & ~1) : kWhole; };
    if (share) {
      const int cand = tid / kPer, mine = limit(cand);
      int items = 0, slots = 0;
      for (int t = tid % kPer; t < tiles; t += kPer) {
        const int p = tile_pieces(steps[t], mine).y;
        items += p;
        slots += p > 1 ? p : 0;
      }
#pragma unroll
      for (int o = kPer / 2; o > 0; o >>= 1) {
        items += __shfl_xor(items, o, kPer);
        slots += __shfl_xor(slots, o, kPer);
      }
      if (tid % kPer == 0) { cand_items[cand] = items; cand_slots[cand] = slots; }
    } else if (tid < kPlanCandidates) {
      cand_items[tid] = tid ? 0 : tiles;
      cand_slots[tid] = 0;
    }
    __syncthreads();
    if (tid < kPlanCandidates) {
      const int n = cand_items[tid], k = cand_slots[tid];
      PlanChoice mine = {kWhole, 1, 0, 1.f, 1.f};
      float est = INFINITY;
      if (n > 0 && k <= a.max_slots) {
        const float work = steps_sum + (float)kItemSteps * n + (float)kPartialSteps * k;
        const float each = work / n;
        const int r0 = (n + lanes - 1) / lanes;
        for (int r = r0; r < r0 + (rows ? 4 : 1); ++r) {
          const int x = (n + r - 1) / r, y = lanes - x;
          const float span = r * each;
          const float done = rows ? fminf(fminf(1.f, y * span / row_work), span / row_hbm) : 1.f;
          const float e = fmaxf(span, (work + row_work) / lanes) +
                          (1.f - done) * fmaxf(row_hbm, row_work / lanes);
          if (e < est) {
            est = e;
            mine = {limit(tid), x, y, each, rows ? y * span / fmaxf(done * row_items, 1e-3f) : 1.f};
          }
        }
      }
      float best = est;
#pragma unroll
      for (int o = kPlanCandidates / 2; o > 0; o >>= 1)
        best = fminf(best, __shfl_xor(best, o, kPlanCandidates));
      const unsigned long long good = __ballot(est <= 1.03f * best);
      if (tid == __ffsll(good) - 1) choice = mine;
    }
    __syncthreads();
    pick = choice;
    if constexpr (kResident) {
      if (one_round && !rows && pick.limit == kWhole) {
        write_whole();
        return;
      }
    }
  }
  const int C = pick.limit;
  const float per_bucket = 255.f / max(1, min(longest, C));   // C bounds an item's steps
  const float row_per_bucket = 255.f / max(1, min(max_tokens, row_c));

  // ---- items in descending length, so that the last to start are short ----
  auto bucket = [&](int per) { return 255 - min(255, (int)(per * per_bucket)); };
  auto row_bucket = [&](int per) { return 255 - min(255, (int)(per * row_per_bucket)); };
  each(
      [&](int, const PlanTile& t) {
        const int2 p = tile_pieces(t.N, C);
        atomicAdd(&hist[bucket(p.x)], p.y);
      },
      [&](int, int, int L) {
        const int2 p = row_pieces(L, row_c);
        atomicAdd(&row_hist[row_bucket(p.x)], p.y);
      });
  __syncthreads();
  const PlanScan at = plan_scan(tid < 256 ? hist[tid] : 0, false, scan_lds);
  const int total = at.total;
  int row_total = 0;
  if (rows) {
    const PlanScan row_at = plan_scan(tid < 256 ? row_hist[tid] : 0, false, scan_lds);
    row_total = row_at.total;
    if (tid < 256) row_hist[tid] = row_at.before;
  }
  if (tid < 256) hist[tid] = at.before;
  __syncthreads();
  // ---- one list in the order of planned starts ----
  // Tile item j starts at (j / x) dt, one-row item k at (k / y) dd (times in
  // 1/16 steps); on a tie the tile is first. y 0: one-row items after all tiles.
  const int x = max(1, pick.x), y = pick.y;
  const long long dt = max(1, (int)(pick.tile_time * 16.f));
  const long long dd = max(1, (int)fminf(pick.row_time * 16.f, 1e9f));
  auto tile_pos = [&](int j) {
    if (row_total == 0 || y <= 0) return j;
    const long long before = ((j / x) * dt + dd - 1) / dd * y;
    return j + (int)min(before, (long long)row_total);
  };
  auto row_pos = [&](int k) {
    if (y <= 0) return total + k;
    const long long before = ((k / y) * dd / dt + 1) * x;
    return k + (int)min(before, (long long)total);
  };
  each(
      [&](int base, const PlanTile& t) {
        const int2 p = tile_pieces(t.N, C);
        const int j0 = atomicAdd(&hist[bucket(p.x)], p.y);
        const int cu0 = seq_cu[t.idx], n = seq_n[t.idx], L = seq_L[t.idx];
        int slot = -1;
        if (p.y > 1) {
          slot = atomicAdd(&next_slot, p.y);
          const int k = atomicAdd(&next_split, 1);
          a.splits[k] = {cu0 + t.q0, min(R, n - t.q0), slot, p.y};
        }
        for (int k = 0; k < p.y; ++k) {
          const int pos = tile_pos(j0 + k);
          if (pos < a.max_items)
            a.items[pos] = {base + t.idx, t.q0, k * p.x, min(t.N, (k + 1) * p.x),
                            slot < 0 ? -1 : slot + k, cu0, n, L};
        }
      },
      [&](int s, int cu0, int L) {
        const int2 p = row_pieces(L, row_c);
        const int k0 = atomicAdd(&row_hist[row_bucket(p.x)], p.y);
        int slot = -1;
        if (p.y > 1) {
          slot = atomicAdd(&next_row_slot, p.y);
          const int k = atomicAdd(&next_row_split, 1);
          a.row_splits[k] = {cu0, slot, p.y, 0};
        }
        for (int k = 0; k < p.y; ++k) {
          const int pos = row_pos(k0 + k);
          if (pos < a.max_items)
            a.items[pos] = {s, -1, k * p.x, min(L, (k + 1) * p.x), slot < 0 ? -1 : slot + k, cu0,
                            1, L};
        }
      });
  __syncthreads();
  if (tid == 0)
    *a.head = {min(total + row_total, a.max_items), next_split, next_row_split, 0};
}

// Merge the partials of the shared tiles: one workgroup per (tile, kv head,
// wavefront of the tile's 8, quarter of the dims), 32 rows of one query head.
// Bound by the latency of reading the partials, 4 KiB each: every load is a
// row's 8 bytes per lane, contiguous over the rows, and four partials' loads are
// issued together; the merged rows go through LDS to be written in 64-byte
// pieces. 7 us for 28 tiles' heads of 8 partials (26 MB); one workgroup per 32
// rows of all dims, a partial at a time, took 8.5.
template <int G>
__global__ __launch_bounds__(256) void prefill_combine_kernel(
    const PrefillPlan* __restrict__ head, const PrefillSplit* __restrict__ splits,
    const RowSplit* __restrict__ row_splits, const uint8_t* __restrict__ slots,
    const uint8_t* __restrict__ row_slots, uint16_t* __restrict__ out, int num_q_heads,
    int num_kv_heads) {
  constexpr int kPart = kCombineParts;
  __shared__ uint32_t tile[32][kD / 2 / kPart + 1];
  const int row_tasks = head->row_splits * num_kv_heads;
  for (int task = gridDim.x - 1 - blockIdx.x; task < row_tasks; task += gridDim.x) {
    const RowSplit sp = row_splits[task / num_kv_heads];
    const int g = task % num_kv_heads;
    const size_t stride = (size_t)num_kv_heads * row_slot_bytes(G);
    const uint8_t* base = row_slots + ((size_t)sp.slot0 * num_kv_heads + g) * row_slot_bytes(G);
    for (int e = threadIdx.x; e < G * kD; e += 256) {
      merge_states<float>(
          sp.pieces, [&](int j) { return reinterpret_cast<const float*>(base + j * stride)[e]; },
          [&](int j) {
            return reinterpret_cast<const float2*>(base + j * stride +
                                                   G * kD * sizeof(float))[e / kD];
          },
          [&](float, float l, float o) {
            const float inv = l > 0.f ? 1.f / l : 0.f;
            out[((size_t)sp.row * num_q_heads + g * G) * kD + e] = to_bf16(o * inv);
          });
    }
  }
  const int tasks = head->splits * num_kv_heads * kWaves * kPart;   // of shared tiles
  for (int task = blockIdx.x; task < tasks; task += gridDim.x) {
    const int part = task % kPart;
    const int w = (task / kPart) % kWaves;
    const int g = (task / (kPart * kWaves)) % num_kv_heads;
    const PrefillSplit sp = splits[task / (kPart * kWaves * num_kv_heads)];
    const int r0 = (w / G) * 32;
    if (r0 >= sp.rows) continue;
    constexpr int kDimPairs = kD / 2 / kPart;          // of this workgroup
    constexpr int kPer = kDimPairs / 8;                // of a thread: p0 + 8 i
    constexpr int kBatch = 4;
    const int row = threadIdx.x % 32, p0 = threadIdx.x / 32;
    const size_t stride = (size_t)num_kv_heads * kSlotBytes;
    const uint8_t* base = slots + ((size_t)sp.slot0 * num_kv_heads + g) * kSlotBytes;
    const uint8_t* ml_base = base + (size_t)kSlotFloats * sizeof(float) +
                             (w * 32 + row) * sizeof(float2);
    const uint8_t* o_base = base + ((w * (kD / 2) + part * kDimPairs + p0) * 32 + row) *
                                       sizeof(float2);

    float m = -INFINITY, l = 0.f;
    float2 o[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) o[i] = make_float2(0.f, 0.f);
    for (int j0 = 0; j0 < sp.pieces; j0 += kBatch) {
      float2 ml[kBatch], v[kBatch][kPer];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {   // past the end: the last partial, at weight 0
        const size_t at = (size_t)min(j0 + b, sp.pieces - 1) * stride;
        ml[b] = *reinterpret_cast<const float2*>(ml_base + at);
#pragma unroll
        for (int i = 0; i < kPer; ++i)
          v[b][i] = *reinterpret_cast<const float2*>(o_base + at + i * 8 * 32 * sizeof(float2));
      }
      float mn = m;
#pragma unroll
      for (int b = 0; b < kBatch; ++b) mn = fmaxf(mn, ml[b].x);
      const float ref = (mn == -INFINITY) ? 0.f : mn;
      const float alpha = fast_exp2(m - ref);
      m = mn;
      l *= alpha;
#pragma unroll
      for (int i = 0; i < kPer; ++i) { o[i].x *= alpha; o[i].y *= alpha; }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        if (j0 + b >= sp.pieces) break;
        const float wgt = fast_exp2(ml[b].x - ref);
        l = fmaf(wgt, ml[b].y, l);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
          o[i].x = fmaf(wgt, v[b][i].x, o[i].x);
          o[i].y = fmaf(wgt, v[b][i].y, o[i].y);
        }
      }
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      tile[row][p0 + 8 * i] = pack_bf16x2(o[i].x * inv, o[i].y * inv);
    __syncthreads();
    const int nrows = min(32, sp.rows - r0);
    const int h = g * G + w % G;
    for (int e = threadIdx.x; e < nrows * kDimPairs; e += 256) {
      const int r = e / kDimPairs, d2 = e % kDimPairs;
      reinterpret_cast<uint32_t*>(out)[((size_t)(sp.row0 + r0 + r) * num_q_heads + h) * (kD / 2) +
                                       part * kDimPairs + d2] = tile[r][d2];
    }
    __syncthreads();   // the next task writes the tile
  }
}

// One item of a work tile.
template <int G, bool kPow2Blocks>
__device__ __forceinline__ void prefill_tile(
    const PrefillItem& it, int g, const uint16_t* __restrict__ q, const uint8_t* __restrict__ kv,
    int num_blocks, const int* __restrict__ block_table, uint16_t* __restrict__ out,
    uint8_t* __restrict__ slots, int num_q_heads, int num_kv_heads, int max_blocks,
    float scale_log2) {
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // uniform per wavefront
  const int lane = tid % kWave;
  const int h = g * G + wave % G;
  const int s = it.s, q0 = it.q0, cu0 = it.cu0, n = it.n;
  const int L = __builtin_amdgcn_readfirstlane(it.L);
  const int row0 = q0 + (wave / G) * 32;        // first row of this wave
  const int c = L - n;                          // cached context before the chunk
  const int i0 = it.i0, N = it.i1;              // steps of the item
  __builtin_assume(i0 >= 0 && N >= 0);
  const bool idle = row0 >= n;                  // none of the wave's 32 rows is in the chunk

  __shared__ __attribute__((aligned(16))) uint8_t lds_k[kKBufs][kStepBlocks][kTileBytes];
  __shared__ __attribute__((aligned(16))) uint8_t lds_v[kVBufs][kStepBlocks][kTileBytes];

  const size_t block_bytes = 2 * (size_t)num_kv_heads * kTileBytes;
  // log2 of the block size when it is a power of two (a shift replaces the
  // 64-bit multiply in every gather's address)
  const int block_shift = kPow2Blocks ? __builtin_ctzll(block_bytes) : 0;
  const size_t k_off = (size_t)g * kTileBytes;
  const size_t v_off = (size_t)(num_kv_heads + g) * kTileBytes;
  const int* bt = block_table + (size_t)s * max_blocks;
  const int qstride = num_q_heads * kD;

  const int lm = lane % 32;     // MFMA row / column index of this lane
  const int lh = lane / 32;     // which 8-wide half of the 16-wide k slice
  // Key permutation of the S^T rows: A row m = 8a + 4b + e holds key
  // 16 (a / 2) + 8 b + 4 (a % 2) + e of the 32-key tile, so accumulator
  // element i of lane l is key 16 (i / 8) + 8 (l / 32) + i % 8.
  const int ka = lm / 8, kb4 = (lm / 4) % 2, ke = lm % 4;
  const int k_blk = ka / 2;                              // block within the key tile
  const int k_slot = 8 * kb4 + 4 * (ka % 2) + ke;        // slot within the block

  // ---- Q^T operand of the wave's 32 rows, loaded once into registers ----
  // Lane (lm, lh) of k-step ks holds dims ks * 16 + lh * 8 .. + 8 of row
  // row0 + lm; rows past the chunk read the chunk's last row (never written).
  bf16x8_t qr[8];
  if (!idle) {
    const int row = min(row0 + lm, n - 1);
    const uint16_t* qrow = q + (size_t)(cu0 + row) * qstride + (size_t)h * kD + lh * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      qr[ks] = *reinterpret_cast<const bf16x8_t*>(qrow + ks * 16);
  }

  f32x16_t oacc[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
  float m_ref = -INFINITY;   // reference max of the lane's row (log2 domain)
  float l_run = 0.f;         // lane-partial row sum

  // ---- gather of K or V of one 64-key step straight into LDS (global_load_lds) ----
  // The block ids of a step are read from the table first (step_ids), in
  // SGPRs: one 16-byte scalar load when all 4 blocks lie inside the sequence,
  // single entries otherwise; a block past L or with an id outside
  // [0, num_blocks) gets id -1. The bit mask of a step (bit kb: block kb is
  // real) lets the softmax mask its keys and patch_v zero its values.
  const int nblk = (L + kBS - 1) / kBS;   // table entries the sequence uses
  struct StepIds {
    int id[kStepBlocks];
  };
  auto step_ids = [&](int step) __attribute__((always_inline)) {
    StepIds r;
    const int b0 = step * kStepBlocks;
    if (b0 + kStepBlocks <= nblk) {
      const i32x4_t v = scalar_entries4(bt, b0);
#pragma unroll
      for (int kb = 0; kb < kStepBlocks; ++kb) r.id[kb] = v[kb];
    } else {
#pragma unroll
      for (int kb = 0; kb < kStepBlocks; ++kb)
        r.id[kb] = b0 + kb < nblk ? scalar_entry(bt, b0 + kb) : -1;
    }
    return r;
  };
  // Ids are checked against the layer only where they are used, so that
  // nothing waits for the loads where they are issued.
  auto real_id = [&](int id) __attribute__((always_inline)) {
    return (unsigned)id < (unsigned)num_blocks;
  };
  auto id_bits = [&](const StepIds& r) __attribute__((always_inline)) {
    int bits = 0;
#pragma unroll
    for (int kb = 0; kb < kStepBlocks; ++kb) bits |= real_id(r.id[kb]) ? (1 << kb) : 0;
    return bits;
  };
  // The gather itself: a half step is 4 tiles of 4 KiB (blocks 0..3); in
  // round j wavefront w fills quarter (w + 8 j) % 4 of tile (w + 8 j) / 4, a
  // contiguous 1 KiB with 16 bytes per lane. K is copied as stored; for V the
  // lane picks the global 16 bytes that belong at its swizzled LDS position
  // (row pos / 2, half pos % 2 holds global half (pos % 2) ^ ((row >> 3) & 1)).
  // A block that is not real is read from block 0 instead (the host
  // guarantees one exists) and masked afterwards.
  auto gather = [&](auto v_tag, int step, const StepIds& ids) __attribute__((always_inline)) {
    constexpr bool kV = decltype(v_tag)::value;
    // The lane id is recomputed here rather than kept live across the step.
    const int ln = lane_id_fresh();
    const uint8_t* base[2];
    uint32_t off[2], lds[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int kb = (wave + kWaves * j) / 4;     // wave-uniform
      const int quarter = (wave + kWaves * j) % 4;
      // kb is wave / 4 + 2 j: pick the id by a uniform select, not an index
      const int id = wave < 4 ? ids.id[2 * j] : ids.id[2 * j + 1];
      const size_t id0 = real_id(id) ? (size_t)(unsigned)id : 0;
      base[j] = kv + (kPow2Blocks ? id0 << block_shift : id0 * block_bytes) + (kV ? v_off : k_off);
      const unsigned pos = quarter * kWave + (unsigned)ln;   // 16-byte position in the tile
      if constexpr (kV) {
        const unsigned vrow = pos / 2;
        off[j] = vrow * 32 + (((pos % 2) ^ ((vrow >> 3) & 1)) * 16);
        lds[j] = __builtin_amdgcn_readfirstlane(
            lds_addr(&lds_v[step % kVBufs][kb][quarter * 1024]));
      } else {
        off[j] = pos * 16;
        lds[j] = __builtin_amdgcn_readfirstlane(
            lds_addr(&lds_k[step % kKBufs][kb][quarter * 1024]));
      }
    }
    dma16x2(base[0], off[0], lds[0], base[1], off[1], lds[1]);
  };
  auto load_half = [&](auto v_tag, int step) __attribute__((always_inline)) {
    const StepIds ids = step_ids(step);
    gather(v_tag, step, ids);
    return id_bits(ids);
  };
  // Zero the V slots of a landed step that must not contribute: blocks that
  // are not real, and slots at or past L (their bytes may be NaN, and a zero
  // weight times NaN is NaN). Every wavefront patches the whole step right
  // before its own p.v reads it: the writes of different wavefronts are
  // identical and idempotent, so no barrier is needed between them. Called
  // only when such slots exist.
  auto patch_v = [&](int step, int bits) __attribute__((always_inline)) {
    const int kbase = step * kKeys;
    // recomputed here, so no lane constant of this rare path stays live
    // across the pipelined loop
    const int ln = lane_id_fresh();
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int cidx = ln + kWave * j;            // 16-byte chunk of the 4 V tiles
      const int kb = cidx / 256;
      const int pos = cidx % 256;
      const int vrow = pos / 2;
      const int half_g = (pos % 2) ^ ((vrow >> 3) & 1);
      uint4* v = reinterpret_cast<uint4*>(&lds_v[step % kVBufs][kb][pos * 16]);
      if (!((bits >> kb) & 1)) {
        *v = make_uint4(0, 0, 0, 0);
        continue;
      }
      const int key = kbase + kb * kBS + 8 * half_g;
      if (key + 8 <= L) continue;
      uint4 w4 = *v;
      uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t lo = (key + 2 * k < L) ? 0x0000ffffu : 0u;
        const uint32_t hi = (key + 2 * k + 1 < L) ? 0xffff0000u : 0u;
        w[k] &= (lo | hi);
      }
      *v = make_uint4(w[0], w[1], w[2], w[3]);
    }
  };
  auto step_clean = [&](int step, int bits) __attribute__((always_inline)) { return bits == 0xf && (step + 1) * kKeys <= L; };

  const int wave_pos0 = c + row0;   // position of the wave's first row
  const int v_read = lm * 32 + ((lh ^ ((lm >> 3) & 1)) * 16);

  // S^T for one step: 2 key tiles x 8 k-steps of 16 dims.
  auto qk = [&](int step, f32x16_t (&sa)[2]) {
    const int buf = step % kKBufs;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) sa[kt][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const bf16x8_t b = qr[ks];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const int chunk = 2 * ks + lh;
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(
            &lds_k[buf][2 * kt + k_blk][(chunk * kBS + k_slot) * 16]);
        sa[kt] = mfma32(a, b, sa[kt]);
      }
    }
  };
  // O^T += V^T P^T for one step: one k-step per block, 4 accumulator chains.
  // Used once per tile, after the pipelined loop; the fence after each block
  // keeps the compiler from hoisting all 16 operand reads at once, which
  // would need more registers than the kernel has left.
  auto pv = [&](int step, const bf16x8_t (&pr)[4]) {
    const int buf = step % kVBufs;
#pragma unroll
    for (int kb = 0; kb < kStepBlocks; ++kb) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const bf16x8_t a =
            *reinterpret_cast<const bf16x8_t*>(&lds_v[buf][kb][dt * 32 * 32 + v_read]);
        oacc[dt] = mfma32(a, pr[kb], oacc[dt]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Causal / length / real-block mask of one step's scores, in place; run
  // only on the steps that need it.
  auto mask_scores = [&](int step, int bits, f32x16_t (&sr)[2]) {
    const int kbase = step * kKeys;
    const int ln = lane_id_fresh();   // as in patch_v
    const int qpos = wave_pos0 + ln % 32;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int kpos = kbase + kt * 32 + (i / 8) * 16 + (ln / 32) * 8 + (i % 8);
        const int blk_ok = (bits >> (2 * kt + i / 8)) & 1;
        const int keep = (kpos <= qpos) & (kpos < L) & blk_ok;
        sr[kt][i] = keep ? sr[kt][i] : -INFINITY;
      }
  };
  auto needs_mask = [&](int step, int bits) __attribute__((always_inline)) {
    return (step * kKeys + kKeys - 1 > wave_pos0) || !step_clean(step, bits);
  };
  // bitsm1, bits0 .. bits3: real-block masks of steps i - 1, i .. i + 3
  int bitsm1 = 0, bits0 = 0, bits1 = 0, bits2 = 0, bits3 = 0;
  // block ids of the gathers of the coming phase: K of step i + 3 and V of
  // step i + 1, read at the end of the phase before (ahead of its barrier)
  StepIds idsK, idsV;
  f32x16_t sA[2], sB[2];    // scores of even / odd steps
  bf16x8_t pA[4], pB[4];    // P of even / odd steps

  // One pipeline step i: the matrix work (p.v of step i - 1, q.k of step
  // i + 1) next to the softmax of step i, with the gathers of K of step i + 3
  // and V of step i + 1 in between. The step ends by waiting for the gathers
  // of the earlier steps only (those of this step get the whole next step to
  // land) and a barrier;
  // then O takes the rescale of step i's softmax, between the p.v of steps
  // i - 1 and i.
  //
  // The matrix and softmax work is laid out by hand in 32 issue slots: slot
  // k issues matrix instruction k (p.v for k < 16, q.k after), the LDS read
  // of the operand five slots ahead, and one exponential with its share of
  // the row sum and bf16 packing. A wavefront issues in order, so without
  // this the vector work would queue behind runs of matrix instructions
  // instead of running beside them. The gathers' branches split the slots
  // into three blocks, and the compiler gathers most exponentials of a block
  // into one run, so some slots issue their matrix instructions back to back.
  // Holding the exponentials in their slots measured slower, and so did
  // either strict order of the step's two halves (all matrix work first, or
  // all softmax first). The row max, when a step needs it, follows the slots.
  auto phase = [&](auto qk_tag, auto pv_tag, int i, f32x16_t (&s_cur)[2],
                   f32x16_t (&s_nxt)[2], const bf16x8_t (&p_prev)[4], bf16x8_t (&p_cur)[4]) __attribute__((always_inline)) {
    constexpr bool kQK = decltype(qk_tag)::value;
    constexpr bool kPV = decltype(pv_tag)::value;
    // The block ids were read before the barrier that ends the previous
    // phase: wait for them here, while no operand read of this phase is in
    // flight, so that the operand prefetch below is never drained for them
    // (scalar loads share the lgkm counter with LDS reads and return out of
    // order).
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    if (kPV && !step_clean(i - 1, bitsm1)) patch_v(i - 1, bitsm1);
    const bool do_k = i + 3 < N, do_v = i + 1 < N;
    if (needs_mask(i, bits0)) mask_scores(i, bits0, s_cur);

    const int vbuf = (i + kVBufs - 1) % kVBufs;   // V of step i - 1
    const int kbuf = (i + 1) % kKBufs;            // K of step i + 1
    auto has_mfma = [&](int k) __attribute__((always_inline)) { return k < 16 ? kPV : kQK; };
    auto a_frag = [&](int k) __attribute__((always_inline)) {
      if (k < 16)
        return *reinterpret_cast<const bf16x8_t*>(
            &lds_v[vbuf][k / 4][(k % 4) * 32 * 32 + v_read]);
      const int ks = (k - 16) / 2, kt = (k - 16) % 2;
      return *reinterpret_cast<const bf16x8_t*>(
          &lds_k[kbuf][2 * kt + k_blk][((2 * ks + lh) * kBS + k_slot) * 16]);
    };
    constexpr int kAhead = kQK ? 5 : 3;   // the last step keeps fewer reads in flight
    bf16x8_t fr[kAhead + 1];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (has_mfma(k)) fr[k % (kAhead + 1)] = a_frag(k);
    }
    float ref = (m_ref == -INFINITY) ? 0.f : m_ref, alpha = 1.f, psum = 0.f;
    bool rescale = false;
    float pe[32];
    uint32_t pw[16];
    f32x16_t zero;
#pragma unroll
    for (int e = 0; e < 16; ++e) zero[e] = 0.f;
    // Raised issue priority while this wavefront issues its matrix slots, so
    // that the arbiter prefers its MFMAs and operand reads over the vector
    // work of the other wavefront of the SIMD (0.5-0.9% faster, same-box A/B).
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      // operand reads for slot k + kAhead
      const int kn = k + kAhead;
      if (kn < 32 && has_mfma(kn)) fr[kn % (kAhead + 1)] = a_frag(kn);
      // matrix instruction k
      if (k < 16) {
        if (kPV) oacc[k % 4] = mfma32(fr[k % (kAhead + 1)], p_prev[k / 4], oacc[k % 4]);
      } else if (kQK) {
        const int ks = (k - 16) / 2, kt = (k - 16) % 2;
        s_nxt[kt] = mfma32(fr[k % (kAhead + 1)], qr[ks], ks == 0 ? zero : s_nxt[kt]);
      }
      // softmax share of slot k: the exponential of score k against the
      // current reference
      {
        const int e = k;
        pe[e] = fast_exp2(fmaf(s_cur[e / 16][e % 16], scale_log2, -ref));
        if (e % 2 == 1) {
          // the row sum adds the bf16 values that p.v multiplies
          pw[e / 2] = pack_bf16x2(pe[e - 1], pe[e]);
          psum = dot2_bf16(pw[e / 2], kBf16OnePair, psum);
        }
      }
      // the step's gathers, issued inside the schedule (K in slot 10, V in
      // slot 26) so that their LDS writes do not land in one burst
      if (k == 10 && do_k) {
        gather(std::false_type{}, i + 3, idsK);
        bits3 = id_bits(idsK);
      }
      if (k == 26 && do_v) gather(std::true_type{}, i + 1, idsV);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
    // A row without a reference yet, or a lane whose partial row sum (which
    // bounds each of its exponentials) left 2^8: take the exact row max, move
    // the reference of the rows that outgrew theirs by more than 2^8, and
    // redo the step's exponentials against it. Rows that did not outgrow
    // theirs get the same values again.
    if (__builtin_amdgcn_ballot_w64(m_ref == -INFINITY || !(psum <= kPsumBound)) != 0) {
      float mp0 = -INFINITY, mp1 = -INFINITY;
#pragma unroll
      for (int e = 0; e < 32; e += 4) {
        mp0 = max3f(mp0, s_cur[e / 16][e % 16], s_cur[e / 16][e % 16 + 1]);
        mp1 = max3f(mp1, s_cur[e / 16][e % 16 + 2], s_cur[e / 16][e % 16 + 3]);
      }
      float mx = max3f(mp0, mp1, mp1);
      mx = max3f(mx, __shfl_xor(mx, 32, kWave), mx);
      const float tmax = mx * scale_log2;
      const bool grow = tmax > m_ref + kLazyRescale;
      rescale = __builtin_amdgcn_ballot_w64(grow) != 0;
      const float nref = grow ? tmax : m_ref;
      alpha = (m_ref == -INFINITY) ? 0.f : fast_exp2(m_ref - nref);
      m_ref = nref;
      ref = (nref == -INFINITY) ? 0.f : nref;
      psum = 0.f;
#pragma unroll
      for (int e = 0; e < 32; e += 2) {
        pw[e / 2] = pack_bf16x2(fast_exp2(fmaf(s_cur[e / 16][e % 16], scale_log2, -ref)),
                                fast_exp2(fmaf(s_cur[e / 16][e % 16 + 1], scale_log2, -ref)));
        psum = dot2_bf16(pw[e / 2], kBf16OnePair, psum);
      }
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
      p_cur[kb] = __builtin_bit_cast(
          bf16x8_t, make_uint4(pw[4 * kb], pw[4 * kb + 1], pw[4 * kb + 2], pw[4 * kb + 3]));
    l_run = l_run * alpha + psum;
    // keep the softmax in its slots (the compiler would otherwise sink it
    // next to its first use, away from the matrix work it should overlap)
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" ::"v"(p_cur[k]));
    asm volatile("" ::"v"(l_run));
    // the block ids of the next phase's gathers
    if (i + 4 < N) idsK = step_ids(i + 4);
    if (i + 2 < N) idsV = step_ids(i + 2);
    // wait for the gathers of steps before this one (each thread issued two
    // for K when i + 3 < N and two for V when i + 1 < N in this step)
    if (i + 3 < N)
      asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    else if (i + 1 < N)
      asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (rescale) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) oacc[dt] *= alpha;
    }
    bitsm1 = bits0;
    bits0 = bits1;
    bits1 = bits2;
    bits2 = bits3;
  };

  // A wavefront none of whose rows lies in the chunk (a short chunk's last
  // tile, a one-row decode sequence in a unified batch) still takes its share
  // of every gather and meets every barrier, step for step like the others,
  // but does no matrix or softmax work and writes nothing.
  if (idle) {
    if (N > i0) {
      load_half(std::false_type{}, i0);
      if (i0 + 1 < N) load_half(std::false_type{}, i0 + 1);
      if (i0 + 2 < N) load_half(std::false_type{}, i0 + 2);
      load_half(std::true_type{}, i0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      __syncthreads();   // the others' q.k of the first step
      for (int i = i0; i < N; ++i) {
        if (i + 3 < N) load_half(std::false_type{}, i + 3);
        if (i + 1 < N) load_half(std::true_type{}, i + 1);
        if (i + 3 < N)
          asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        else if (i + 1 < N)
          asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
        else
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
      }
    }
    return;
  }

  if (N > i0) {
    bits0 = load_half(std::false_type{}, i0);
    if (i0 + 1 < N) bits1 = load_half(std::false_type{}, i0 + 1);
    if (i0 + 2 < N) bits2 = load_half(std::false_type{}, i0 + 2);
    load_half(std::true_type{}, i0);
    if (i0 + 3 < N) idsK = step_ids(i0 + 3);
    if (i0 + 1 < N) idsV = step_ids(i0 + 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    qk(i0, sA);
    __syncthreads();   // K of the first step is read; its pipeline step gathers into its buffer
    constexpr std::true_type T{};
    constexpr std::false_type F{};
    if (i0 + 1 < N)
      phase(T, F, i0, sA, sB, pB, pA);
    else
      phase(F, F, i0, sA, sB, pB, pA);
    int i = i0 + 1;   // i0 is even: even steps use sA and pA
    for (; i + 1 <= N - 2; i += 2) {
      phase(T, T, i, sB, sA, pA, pB);
      phase(T, T, i + 1, sA, sB, pB, pA);
    }
    if (i <= N - 2) {
      phase(T, T, i, sB, sA, pA, pB);
      ++i;
    }
    // p.v of the last step (its V landed by the last step's full wait)
    if (i0 + 1 < N) {
      if (i & 1)
        phase(F, T, i, sB, sA, pA, pB);
      else
        phase(F, T, i, sA, sB, pB, pA);
    }
    if (!step_clean(N - 1, bitsm1)) patch_v(N - 1, bitsm1);
    pv(N - 1, ((N - 1) & 1) ? pB : pA);
  }

  // ---- write O (this lane: row lm): normalised, or the item's partial ----
  {
    const float lt = l_run + __shfl_xor(l_run, 32, kWave);
    const int r = row0 + lm;
    if (it.slot < 0) {
      // A lane holds 8-byte pieces of its row, two lanes per row: stored like
      // that, an instruction touches 32 rows of 16 bytes. Half the dims at a
      // time go through the wavefront's part of the K buffers, which nobody
      // reads any more, and are stored in runs of 128 bytes. A call, stored directly and
      // like this: 7 fresh prompts of 188 to 2031 rows (64 query heads over 8)
      // 172 -> 159 us, 64 of 100 rows (32 over 8) 59 -> 51 us, 4 of 64 rows 12.8 ->
      // 10.6 us; tiles of hundreds of steps do not notice.
      constexpr int kHalf = kD / 2, kRowBytes = kHalf * 2 + 16;   // padded against conflicts
      static_assert(kWaves * 32 * kRowBytes <= (int)sizeof(lds_k), "fits the K buffers");
      uint8_t* stage = &lds_k[0][0][0] + wave * 32 * kRowBytes;
      const float inv = lt > 0.f ? 1.f / lt : 0.f;
      const int sr = lane / 16, sc = lane % 16;   // row of four, 8-byte piece of its half
#pragma unroll
      for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int dt = 2 * half; dt < 2 * half + 2; ++dt) {
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            const f32x16_t& o = oacc[dt];
            *reinterpret_cast<uint2*>(stage + lm * kRowBytes +
                                      ((dt - 2 * half) * 32 + a * 8 + lh * 4) * 2) =
                make_uint2(pack_bf16x2(o[4 * a + 0] * inv, o[4 * a + 1] * inv),
                           pack_bf16x2(o[4 * a + 2] * inv, o[4 * a + 3] * inv));
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int rr = 4 * j + sr;
          const uint2 w = *reinterpret_cast<const uint2*>(stage + rr * kRowBytes + sc * 8);
          if (row0 + rr < n)
            *reinterpret_cast<uint2*>(out + (size_t)(cu0 + row0 + rr) * qstride +
                                      (size_t)h * kD + half * kHalf + sc * 4) = w;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    } else if (r < n) {
      uint8_t* slot = slots + ((size_t)it.slot * num_kv_heads + g) * kSlotBytes;
      float2* po = reinterpret_cast<float2*>(slot) + wave * 32 * (kD / 2) + lm;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int a = 0; a < 8; ++a)   // dims dt 32 + (a / 2) 8 + lh 4 + (a % 2) 2 .. + 2
          po[(dt * 16 + (a / 2) * 4 + lh * 2 + a % 2) * 32] =
              make_float2(oacc[dt][2 * a], oacc[dt][2 * a + 1]);
      if (lh == 0)
        reinterpret_cast<float2*>(slot + kSlotFloats * sizeof(float))[wave * 32 + lm] =
            make_float2(m_ref, lt);
    }
  }
}

// One item of a one-row sequence: the eight wavefronts share its tokens evenly
// in whole steps of 64 and merge their states through LDS.
template <int G>
__device__ __forceinline__ void prefill_row(
    const PrefillItem& it, int g, const uint16_t* __restrict__ q, const uint8_t* __restrict__ kv,
    int num_blocks, const int* __restrict__ block_table, uint16_t* __restrict__ out,
    uint8_t* __restrict__ row_slots, int num_q_heads, int num_kv_heads, int max_blocks,
    float scale_log2) {
  __shared__ __attribute__((aligned(16))) float o_lds[kWaves][G * kD];
  __shared__ float2 ml_lds[kWaves][G];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int i0 = it.i0, i1 = it.i1;
  const int per = max(1, (i1 - i0 + kWaves * kKeys - 1) / (kWaves * kKeys)) * kKeys;
  const int parts = (i1 - i0 + per - 1) / per;     // wavefronts with tokens
  const size_t head_off = (size_t)g * kTileBytes;
  const DecodeTiles<false> tiles = {kv, nullptr, 0, 2 * (size_t)num_kv_heads * kTileBytes,
                                    head_off, (size_t)num_kv_heads * kTileBytes + head_off};
  const size_t row = ((size_t)it.cu0 * num_q_heads + g * G) * kD;
  if (wave < parts) {
    const int t0 = i0 + wave * per;
    walk_bf16<kD, G, false, false>(tiles, q + row, block_table + (size_t)it.s * max_blocks, num_blocks,
                            t0, min(i1, t0 + per), scale_log2, o_lds[wave], ml_lds[wave]);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < G * kD; e += kThreads) {
    merge_states<float>(
        parts, [&](int j) { return o_lds[j][e]; }, [&](int j) { return ml_lds[j][e / kD]; },
        [&](float m, float l, float o) {
          if (it.slot < 0) {
            const float inv = l > 0.f ? 1.f / l : 0.f;
            out[row + e] = to_bf16(o * inv);
          } else {
            uint8_t* slot = row_slots + ((size_t)it.slot * num_kv_heads + g) * row_slot_bytes(G);
            reinterpret_cast<float*>(slot)[e] = o;
            if (e % kD == 0)
              reinterpret_cast<float2*>(slot + G * kD * sizeof(float))[e / kD] =
                  make_float2(m, l);
          }
        });
  }
}

// Work tiles only: one workgroup per (item or tile, kv head).
template <int G, bool kPow2Blocks>
__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads),
                          amdgpu_waves_per_eu(2, 2)))
void prefill_kernel(const uint16_t* __restrict__ q, const uint8_t* __restrict__ kv,
                    int num_blocks, const int* __restrict__ block_table,
                    const int* __restrict__ seq_lens, const int* __restrict__ cu,
                    uint16_t* __restrict__ out, const int2* __restrict__ tiles,
                    const int* __restrict__ tile_count, const PrefillItem* __restrict__ items,
                    uint8_t* __restrict__ slots, int total_q, int num_q_heads, int num_kv_heads,
                    int max_blocks, int max_seq_len, float scale_log2) {
  constexpr int kRows = 32 * kWaves / G;   // rows per work tile
  const int g = blockIdx.x % num_kv_heads;
  const int ti = blockIdx.x / num_kv_heads;
  PrefillItem it;
  if (items) it = items[ti];   // the list has room for the whole grid: read beside the count
  if (ti >= *tile_count) return;
  if (!items) {   // no plan: the tile map's whole tiles
    const int2 tl = tiles[ti];
    const int2 rows = chunk_rows(cu, tl.x, total_q);
    it.s = tl.x;
    it.q0 = tl.y;
    it.cu0 = rows.x;
    it.n = rows.y - rows.x;
    it.L = min(max(seq_lens[tl.x], 0), min(max_seq_len, max_blocks * kBS));
    const int last_pos = min(it.L - it.n + it.q0 + min(kRows, it.n - it.q0) - 1, it.L - 1);
    it.i0 = 0;
    it.i1 = last_pos >= 0 ? last_pos / kKeys + 1 : 0;
    it.slot = -1;
  }
  prefill_tile<G, kPow2Blocks>(it, g, q, kv, num_blocks, block_table, out, slots, num_q_heads,
                               num_kv_heads, max_blocks, scale_log2);
}

// A planned step that may hold one-row sequences.
template <int G, bool kPow2Blocks>
__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads),
                          amdgpu_waves_per_eu(2, 2)))
void prefill_step_kernel(const uint16_t* __restrict__ q, const uint8_t* __restrict__ kv,
                         int num_blocks, const int* __restrict__ block_table,
                         uint16_t* __restrict__ out, const PrefillPlan* __restrict__ head,
                         const PrefillItem* __restrict__ items, uint8_t* __restrict__ slots,
                         uint8_t* __restrict__ row_slots, int num_q_heads, int num_kv_heads,
                         int max_blocks, float scale_log2) {
  const int g = blockIdx.x % num_kv_heads;
  const int ti = blockIdx.x / num_kv_heads;
  const PrefillItem it = items[ti];   // the list has room for the whole grid
  if (ti >= head->items) return;
  if (it.q0 < 0)
    prefill_row<G>(it, g, q, kv, num_blocks, block_table, out, row_slots, num_q_heads,
                   num_kv_heads, max_blocks, scale_log2);
  else
    prefill_tile<G, kPow2Blocks>(it, g, q, kv, num_blocks, block_table, out, slots, num_q_heads,
                                 num_kv_heads, max_blocks, scale_log2);
}

// Offsets of a planned step's pieces of the workspace.
namespace {
struct PrefillWs {
  int max_items, max_slots, max_row_slots;   // items; slots per kv head
  size_t items, splits, row_splits, slots, row_slots;   // byte offsets; the head is at 0
  size_t total;
};

size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// Workgroups' worth of partial slots: the plan fills the chip once or twice.
constexpr int kSlotWorkgroups = 2 * kNumCUs;

PrefillWs prefill_ws(int num_seqs, int total_q, int group, int num_kv_heads) {
  PrefillWs w;
  const int lanes = num_kv_heads < kNumCUs ? kNumCUs / num_kv_heads : 1;
  w.max_slots = num_kv_heads <= kNumCUs ? kSlotWorkgroups / num_kv_heads : 0;
  // shared one-row sequences of T tokens in all have at most 2 T / (T / (2 lanes)) items
  w.max_row_slots = 4 * lanes + 8;
  w.max_items = total_q / (32 * kWaves / group) + num_seqs + w.max_slots + w.max_row_slots;
  w.items = 256;
  w.splits = w.items + up256((size_t)w.max_items * sizeof(PrefillItem));
  w.row_splits = w.splits + up256((size_t)(w.max_slots / 2 + 1) * sizeof(PrefillSplit));
  w.slots = w.row_splits + up256((size_t)(w.max_row_slots / 2 + 1) * sizeof(RowSplit));
  w.row_slots = w.slots + (size_t)w.max_slots * num_kv_heads * kSlotBytes;
  w.total = w.row_slots + (size_t)w.max_row_slots * num_kv_heads * row_slot_bytes(group);
  return w;
}
}  // namespace

size_t prefill_planned_bytes(int num_seqs, int total_q, int num_q_heads) {
  // the most of every group size's layout
  size_t most = 0;
  for (int group = 1; group <= 8; group *= 2) {
    if (num_q_heads % group) continue;
    const size_t t = prefill_ws(num_seqs, total_q, group, num_q_heads / group).total;
    most = t > most ? t : most;
  }
  return most;
}

template <int G>
static hipError_t launch_prefill_t(const PrefillArgs& a) {
  constexpr int kRowsPerTile = 32 * kWaves / G;
  uint8_t* ws = static_cast<uint8_t*>(a.workspace);
  const PrefillWs w = prefill_ws(a.num_seqs, a.total_q_tokens, G, a.num_kv_heads);
  // Sharing tiles is weighed here by the bounds the host knows, and by the plan,
  // with room for the partials, by the lengths it finds. One sequence whose tiles
  // are not shared needs no plan: the tile map lists its tiles in the same order
  // without the passes that order several. The plan of more than kPlanThreads
  // sequences or tiles shares none.
  const long long bound = (long long)a.total_q_tokens / kRowsPerTile + a.num_seqs;
  const bool resident = a.num_seqs <= kPlanThreads && bound <= kPlanThreads;
  const long long steps = ((long long)a.max_seq_len + kKeys - 1) / kKeys;
  const long long tile_wgs = (long long)(a.total_q_tokens / kRowsPerTile) * a.num_kv_heads;
  const bool share = resident && sharing_pays(steps, tile_wgs, kLaunchSteps);
  // Several sequences may hold one-row ones (only the device knows), one does if
  // it is one row; with one longer sequence the kernel without that branch runs.
  const bool rows = a.num_seqs > 1 || a.total_q_tokens == 1;
  const bool planned = a.workspace_bytes >= w.total && (rows || share);
  const int2* tiles = nullptr;
  const int* count;
  const PrefillItem* items = nullptr;
  int grid_items, max_slots = 0, max_row_slots = 0;
  hipError_t e;
  if (planned) {
    max_slots = share ? w.max_slots : 0;
    PlanArgs p;
    p.cu = a.cu_seqlens_q;
    p.seq_lens = a.seq_lens;
    p.num_seqs = a.num_seqs;
    p.total_q = a.total_q_tokens;
    p.rows_per_tile = kRowsPerTile;
    p.num_kv_heads = a.num_kv_heads;
    p.max_seq_tokens = a.max_seq_len < a.max_blocks * kBS ? a.max_seq_len : a.max_blocks * kBS;
    // One-row sequences are shared from 1024 tokens on (a CU's walk of 4 us), from
    // 2048 where only they would need the merge's launch (about 4 us), or from
    // 8192 beside four or more rounds of tiles, which such a walk can hide in.
    const int shared_from = share ? kRowTokens
                            : tile_wgs < 4 * kNumCUs ? 2 * kRowTokens : 8 * kRowTokens;
    max_row_slots = rows && a.max_seq_len > shared_from ? w.max_row_slots : 0;
    grid_items = (int)(bound + max_slots + max_row_slots);
    p.max_items = grid_items;
    p.max_slots = max_slots;
    p.rows = rows;
    p.max_row_slots = max_row_slots;
    p.items = reinterpret_cast<PrefillItem*>(ws + w.items);
    p.splits = reinterpret_cast<PrefillSplit*>(ws + w.splits);
    p.row_splits = reinterpret_cast<RowSplit*>(ws + w.row_splits);
    p.head = reinterpret_cast<PrefillPlan*>(ws);
    items = p.items;
    count = &p.head->items;
    trace_before(a.stream, "prefill_plan");
    hipLaunchKernelGGL(resident ? prefill_plan_kernel<true> : prefill_plan_kernel<false>, dim3(1),
                       dim3(kPlanThreads), 0, a.stream, p);
  } else {
    // One sequence of whole tiles, or a workspace of the tile list's size alone.
    int* c = reinterpret_cast<int*>(ws);
    int2* t = reinterpret_cast<int2*>(ws + 16);
    const long long max_tiles = (long long)((a.workspace_bytes - 16) / sizeof(int2));
    grid_items = (int)(bound < max_tiles ? bound : max_tiles);
    tiles = t;
    count = c;
    trace_before(a.stream, "prefill_tile_map");
    hipLaunchKernelGGL(prefill_tile_map_kernel, dim3(1), dim3(256), 0, a.stream, a.cu_seqlens_q,
                       a.num_seqs, a.total_q_tokens, kRowsPerTile, t, c, grid_items);
  }
  trace_after(a.stream);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const long long blocks = (long long)grid_items * a.num_kv_heads;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  trace_before(a.stream, "prefill");
  const unsigned kvh = (unsigned)a.num_kv_heads;
  const bool pow2 = (kvh & (kvh - 1)) == 0;
  const uint16_t* q = static_cast<const uint16_t*>(a.q);
  const uint8_t* kv = static_cast<const uint8_t*>(a.kv);
  uint16_t* out = static_cast<uint16_t*>(a.out);
  const PrefillPlan* head = reinterpret_cast<const PrefillPlan*>(ws);
  const float scale_log2 = a.scale * kLog2e;
  if (planned && rows) {
    auto kernel = pow2 ? prefill_step_kernel<G, true> : prefill_step_kernel<G, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, a.stream, q, kv,
                       a.num_blocks, a.block_table, out, head, items, ws + w.slots,
                       ws + w.row_slots, a.num_q_heads, a.num_kv_heads, a.max_blocks,
                       scale_log2);
  } else {
    auto kernel = pow2 ? prefill_kernel<G, true> : prefill_kernel<G, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, a.stream, q, kv,
                       a.num_blocks, a.block_table, a.seq_lens, a.cu_seqlens_q, out, tiles, count,
                       items, ws + w.slots, a.total_q_tokens, a.num_q_heads, a.num_kv_heads,
                       a.max_blocks, a.max_seq_len, scale_log2);
  }
  trace_after(a.stream);
  e = hipGetLastError();
  if (e != hipSuccess || (max_slots == 0 && max_row_slots == 0)) return e;
  trace_before(a.stream, "prefill_combine");
  hipLaunchKernelGGL((prefill_combine_kernel<G>), dim3(kCombineGrid), dim3(256), 0, a.stream, head,
                     reinterpret_cast<const PrefillSplit*>(ws + w.splits),
                     reinterpret_cast<const RowSplit*>(ws + w.row_splits), ws + w.slots,
                     ws + w.row_slots, out, a.num_q_heads, a.num_kv_heads);
  trace_after(a.stream);
  return hipGetLastError();
}

hipError_t launch_prefill(const PrefillArgs& a) {
  if (a.head_dim != kD) return hipErrorNotSupported;
  switch (a.num_q_heads / a.num_kv_heads) {
    case 1: return launch_prefill_t<1>(a);
    case 2: return launch_prefill_t<2>(a);
    case 4: return launch_prefill_t<4>(a);
    case 8: return launch_prefill_t<8>(a);
    default: return hipErrorNotSupported;
  }
}

}  // namespace kvattn
