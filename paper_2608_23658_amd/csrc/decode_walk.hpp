// One wavefront's walk over a run of a sequence's cached tokens for the query
// heads of one kv head: the work that decode and the one-row sequences of a
// chunked-prefill step share.
#pragma once

#include "common.hpp"

namespace kvattn {

template <int D, bool BF16>
struct DecodeShape {
  static constexpr int kEsz = BF16 ? 2 : 4;
  static constexpr int kVec = 16 / kEsz;          // elements per 16-byte chunk
  static constexpr int kBS = 16;                  // tokens per block
  static constexpr int kTile = 64;                // tokens per wavefront step
  static constexpr int kTB = kTile / kBS;         // blocks per step
  static constexpr int kKCh = D / kVec;           // 16-byte chunks per K row
  static constexpr int kR = kBS * kEsz / 16;      // 16-byte chunks per V dim row
  static constexpr int kDPI = kWave / kR;         // V dim rows per load
  static constexpr int kVI = D / kDPI;            // V loads per block
  static constexpr int kTileElems = kBS * D;      // one (block, K/V, head) tile
  static_assert(kVI * 1024 == kTileElems * kEsz, "V tile is kVI loads of 1 KiB");
  static_assert(kKCh == 4 * kVI, "a K load of 1 KiB holds a quarter of each of 16 rows");
};

// The ids of the next 64 blocks from token t (a multiple of 16) of a
// sequence, one per lane: one load instead of one dependent load per step.
// Blocks at or past t1 and ids outside the layer give -1.
__device__ __forceinline__ int walk_ids(const int* __restrict__ bt, int t, int t1,
                                        int num_blocks) {
  const int lane = threadIdx.x % kWave;
  int id = -1;
  if (t + lane * 16 < t1) id = bt[t / 16 + lane];
  return (unsigned)id < (unsigned)num_blocks ? id : -1;
}

__device__ __forceinline__ float fma_each(float w, float x, float o) { return fmaf(w, x, o); }
__device__ __forceinline__ float4 fma_each(float w, float4 x, float4 o) {
  return make_float4(fmaf(w, x.x, o.x), fmaf(w, x.y, o.y), fmaf(w, x.z, o.z), fmaf(w, x.w, o.w));
}

// Merges n softmax states of one output element, or of four of one row, in
// order (log-sum-exp): o_of(j) and ml_of(j) give state j's unnormalised value
// and (max, row sum); done(m, l, o) gets the merged ones.
template <typename T, typename O, typename Ml, typename Done>
__device__ __forceinline__ void merge_states(int n, O o_of, Ml ml_of, Done done) {
  float m = -INFINITY;
  for (int j = 0; j < n; ++j) m = fmaxf(m, ml_of(j).x);
  const float ref = (m == -INFINITY) ? 0.f : m;
  float l = 0.f;
  T o = {};
  for (int j = 0; j < n; ++j) {
    const float2 ml = ml_of(j);
    const float w = fast_exp2(ml.x - ref);
    l = fmaf(w, ml.y, l);
    o = fma_each(w, o_of(j), o);
  }
  done(m, l, o);
}

// Where a workgroup's K and V tiles lie.
// kTwo: the layer is split over two tensors (the design the paper rejects in
// Section 3, "The contiguity constraint"): ids below num_base address kv, the
// others kv2 at id - num_base. Otherwise kv2 and num_base are unused.
template <bool kTwo>
struct DecodeTiles {
  const uint8_t* kv;
  const uint8_t* kv2;
  int num_base;
  size_t block_bytes, k_off, v_off;
  __device__ __forceinline__ const uint8_t* block(int id) const {
    if constexpr (kTwo)
      return id < num_base ? kv + (size_t)id * block_bytes
                           : kv2 + (size_t)(id - num_base) * block_bytes;
    else
      return kv + (size_t)id * block_bytes;
  }
};

// The four blocks of a step: each block's K tile and V tile as they lie in
// memory, 1 KiB per load, the two tiles of a block issued together. Within a
// V load lane l takes 16-byte chunk v_lane of the KiB. A block without a valid
// id (< 0) gives zeros, or with kAlways whatever block 0 holds: the loads then
// sit in no branch, so that a later wait can count them.
template <bool kAlways, int kTB, int kVI, bool kTwo>
__device__ __forceinline__ void load_step(const DecodeTiles<kTwo>& t, const int (&bid)[kTB],
                                          int lane, int v_lane, uint4 (&kreg)[kTB][kVI],
                                          uint4 (&vreg)[kTB][kVI]) {
#pragma unroll
  for (int j = 0; j < kTB; ++j) {
    if (kAlways || bid[j] >= 0) {
      const uint8_t* bp = t.block(kAlways ? max(bid[j], 0) : bid[j]);
      const uint4* kp = reinterpret_cast<const uint4*>(bp + t.k_off) + lane;
      const uint4* vp = reinterpret_cast<const uint4*>(bp + t.v_off) + v_lane;
#pragma unroll
      for (int i = 0; i < kVI; ++i) {
        kreg[j][i] = load_nt(kp + i * kWave);
        vreg[j][i] = load_nt(vp + i * kWave);
      }
    } else {
#pragma unroll
      for (int i = 0; i < kVI; ++i) {
        kreg[j][i] = make_uint4(0, 0, 0, 0);
        vreg[j][i] = make_uint4(0, 0, 0, 0);
      }
    }
  }
}

// One wavefront's walk over tokens [t0, t1) in bf16, on the matrix units: with
// query heads as the 16 columns (G of them real, the rest zero), a step is 16
// products of 16 x 16 x 32 for q.k and 16 for p.v at head_dim 128, whatever G
// is, where bf16 dot2 on the vector unit took 128 G instructions per step.
//   S[token][head]: A = a KiB of the K tile exactly as loaded (lane l: slot
//     l % 16, chunk 4 i + l / 16), B = q in registers. Lane l gets tokens
//     4 (l / 16) .. + 4 of each block for head l % 16, so the softmax state is
//     per lane and one row exchange gives the max.
//   O^T[dim][head] += V^T P^T over 32 tokens, two blocks: the B operand needs 8
//     consecutive tokens per lane, which one swap of the odd lane rows of the
//     first block's P with the even rows of the second's gives; the same swap
//     of the two blocks' V loads gives the matching A operands of 16 dims each.
// kAhead: the next step's loads are issued before a step's products, into a
// second set of registers; at most 64 blocks, whose ids one load gives.
// Leaves the wavefront's state in o_out [G][D] and ml_out [G] (LDS).
template <int D, int G, bool kTwo, bool kAhead>
__device__ __forceinline__ void walk_bf16(const DecodeTiles<kTwo>& tiles,
                                          const uint16_t* __restrict__ q,
                                          const int* __restrict__ bt, int num_blocks, int t0,
                                          int t1, float scale_log2, float* o_out,
                                          float2* ml_out) {
  using S = DecodeShape<D, true>;
  const int lane = threadIdx.x % kWave;
  const int head = lane % 16, row = lane / 16;
  int my_id = walk_ids(bt, t0, t1, num_blocks);
  uint4 qreg[S::kVI];
#pragma unroll
  for (int i = 0; i < S::kVI; ++i) {
    qreg[i] = *reinterpret_cast<const uint4*>(q + min(head, G - 1) * D + i * 32 + row * 8);
    if (head >= G) qreg[i] = make_uint4(0, 0, 0, 0);
  }

  float m_run = -INFINITY, l_run = 0.f;   // head's max; the lane's part of its sum
  f32x4_t acc[2 * S::kVI];
#pragma unroll
  for (int i = 0; i < 2 * S::kVI; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // lane's 16 bytes of a V KiB (32 dims x 2 halves): dim l % 32, half l / 32
  const int v_lane = 2 * (lane % 32) + lane / 32;

  // The products and softmax of one loaded step; tail: it may end inside a
  // block; zero: a block without a valid id still holds what was loaded for it.
  auto compute = [&](int tb, const int (&bid)[S::kTB], bool tail, bool zero,
                     const uint4 (&kreg)[S::kTB][S::kVI],
                     uint4 (&vreg)[S::kTB][S::kVI]) __attribute__((always_inline)) {
    // ---- scores ----
    float x[S::kTB][4];
#pragma unroll
    for (int j = 0; j < S::kTB; ++j) {
      f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < S::kVI; ++i)
        sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kreg[j][i]),
                                                     __builtin_bit_cast(bf16x8_t, qreg[i]), sc, 0,
                                                     0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool keep = bid[j] >= 0 && (!tail || tb + j * S::kBS + row * 4 + r < t1);
        x[j][r] = keep ? sc[r] * scale_log2 : -INFINITY;
      }
    }

    // ---- online softmax over the step (log2 domain) ----
    float mx = m_run;
#pragma unroll
    for (int j = 0; j < S::kTB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, x[j][r]);
    const float mn = cross_row_max(mx);
    const float ref = (mn == -INFINITY) ? 0.f : mn;
    const float alpha = fast_exp2(m_run - ref);
    m_run = mn;
    float psum = 0.f;
    uint2 pw[S::kTB];
#pragma unroll
    for (int j = 0; j < S::kTB; ++j) {
      pw[j].x = pack_bf16x2(fast_exp2(x[j][0] - ref), fast_exp2(x[j][1] - ref));
      pw[j].y = pack_bf16x2(fast_exp2(x[j][2] - ref), fast_exp2(x[j][3] - ref));
      // the row sum adds the bf16 values that p.v multiplies
      psum = dot2_bf16(pw[j].x, kBf16OnePair, psum);
      psum = dot2_bf16(pw[j].y, kBf16OnePair, psum);
    }
    l_run = fmaf(l_run, alpha, psum);
#pragma unroll
    for (int i = 0; i < 2 * S::kVI; ++i) acc[i] *= alpha;

    // ---- p . v, two blocks at a time ----
    if (zero && __builtin_expect((bid[0] | bid[1] | bid[2] | bid[3]) < 0, 0)) {
#pragma unroll
      for (int j = 0; j < S::kTB; ++j) {
        if (bid[j] >= 0) continue;
#pragma unroll
        for (int i = 0; i < S::kVI; ++i) vreg[j][i] = make_uint4(0, 0, 0, 0);
      }
    }
    if (tail) {
#pragma unroll
      for (int j = 0; j < S::kTB; ++j) {
        // slots at or past t1 may hold anything, and zero times NaN is NaN
        const int tok = tb + j * S::kBS + (lane / 32) * 8;
#pragma unroll
        for (int i = 0; i < S::kVI; ++i) {
          uint32_t w[4] = {vreg[j][i].x, vreg[j][i].y, vreg[j][i].z, vreg[j][i].w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t lo = (tok + 2 * k < t1) ? 0x0000ffffu : 0u;
            const uint32_t hi = (tok + 2 * k + 1 < t1) ? 0xffff0000u : 0u;
            w[k] &= (lo | hi);
          }
          vreg[j][i] = make_uint4(w[0], w[1], w[2], w[3]);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < S::kTB; j += 2) {
      uint2 p0 = pw[j], p1 = pw[j + 1];
      swap_rows16(p0.x, p1.x);
      swap_rows16(p0.y, p1.y);
      const bf16x8_t b = __builtin_bit_cast(bf16x8_t, make_uint4(p0.x, p0.y, p1.x, p1.y));
#pragma unroll
      for (int i = 0; i < S::kVI; ++i) {
        uint4 lo = vreg[j][i], hi = vreg[j + 1][i];
        swap_rows16(lo.x, hi.x);   // dims 32 i .. + 16 to lo, 32 i + 16 .. + 16 to hi
        swap_rows16(lo.y, hi.y);
        swap_rows16(lo.z, hi.z);
        swap_rows16(lo.w, hi.w);
        acc[2 * i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8_t, lo), b, acc[2 * i], 0, 0, 0);
        acc[2 * i + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8_t, hi), b, acc[2 * i + 1], 0, 0, 0);
      }
    }
  };
  auto step_ids = [&](int tb, int (&bid)[S::kTB]) __attribute__((always_inline)) {
    const int at = (tb - t0) / S::kBS % kWave;
    if (!kAhead && at == 0 && tb != t0) my_id = walk_ids(bt, tb, t1, num_blocks);
#pragma unroll
    for (int j = 0; j < S::kTB; ++j) bid[j] = __builtin_amdgcn_readlane(my_id, at + j);
  };

  if constexpr (!kAhead) {
    for (int tb = t0; tb < t1; tb += S::kTile) {
      int bid[S::kTB];
      uint4 kreg[S::kTB][S::kVI], vreg[S::kTB][S::kVI];
      step_ids(tb, bid);
      load_step<false>(tiles, bid, lane, v_lane, kreg, vreg);
      compute(tb, bid, tb + S::kTile > t1, false, kreg, vreg);
    }
  } else {
    int id_a[S::kTB], id_b[S::kTB];
    uint4 k_a[S::kTB][S::kVI], v_a[S::kTB][S::kVI], k_b[S::kTB][S::kVI], v_b[S::kTB][S::kVI];
    int tb = t0;
    step_ids(tb, id_a);
    load_step<true>(tiles, id_a, lane, v_lane, k_a, v_a);
    for (;;) {
      if (tb + S::kTile >= t1) {
        compute(tb, id_a, tb + S::kTile > t1, true, k_a, v_a);
        break;
      }
      step_ids(tb + S::kTile, id_b);
      load_step<true>(tiles, id_b, lane, v_lane, k_b, v_b);
      __builtin_amdgcn_sched_barrier(0);   // all of them before the step's products
      compute(tb, id_a, false, true, k_a, v_a);
      tb += S::kTile;
      if (tb + S::kTile >= t1) {
        compute(tb, id_b, tb + S::kTile > t1, true, k_b, v_b);
        break;
      }
      step_ids(tb + S::kTile, id_a);
      load_step<true>(tiles, id_a, lane, v_lane, k_a, v_a);
      __builtin_amdgcn_sched_barrier(0);
      compute(tb, id_b, false, true, k_b, v_b);
      tb += S::kTile;
    }
  }

  const float l_tot = cross_row_sum(l_run);
  if (head < G) {
#pragma unroll
    for (int i = 0; i < 2 * S::kVI; ++i)
      *reinterpret_cast<f32x4_t*>(o_out + head * D + i * 16 + row * 4) = acc[i];
    if (row == 0) ml_out[head] = make_float2(m_run, l_tot);
  }
}

}  // namespace kvattn
