// Split-K paged decode for gfx950: one new query token per sequence attends
// to its whole context, read through the block table (the paper, Section 3
// "The contiguity constraint"; Section 5, decode is one token per sequence).
//
// One workgroup of four wavefronts = one (kv head, sequence, split of the
// context). The 64-token steps of the split are dealt evenly to the wavefronts
// (contiguous runs), each keeps its own softmax state, and the states are
// merged in context order through LDS, so a split costs a quarter of the
// serial walk it cost as one wavefront. What bounds a small batch is that
// walk's latency (one step's loads in flight per wavefront); what bounds a
// large one is HBM. A sequence's arithmetic depends only on its own length. Per
// call, at 2 / 4 / 8 shares a split (32 query heads over 8 kv heads, head_dim
// 128, bf16, graph replay):
//   1 sequence of 1000                13.3 / 9.8 / 8.9 us
//   8 sequences of 200 to 1000        15.0 / 12.0 / 11.4 us
//   64 sequences of 200 to 1000       27.3 / 27.2 / 28.6 us
//   64 sequences of 1000 to 4000       107 / 104 / 107 us
//   256 sequences of 30 to 300        30.8 / 30.7 / 43.1 us
//   256 sequences of 512 to 4096       362 / 361 / 363 us
// Eight gains under 1 us on the smallest batches and loses much on the short
// contexts of a full one. The merge takes four dims per lane, and an fp32 context
// of one share leaves from the registers instead (256 sequences of 1 to 64: 11.4
// -> 9.7 us; the same in fp32 12.1 -> 10.9 us).
//
// Four wavefronts on one CU ask it for 128 KiB a step, about 2 us whatever the
// latency is, while a small batch leaves other CUs idle. So up to kSpreadBlocks
// workgroups (half the CUs) each wavefront's share becomes a workgroup on a CU
// of its own that loads a step ahead (which alone gained 0.5 us), writes its
// state as a partial, and the merge kernel does the split's merge first, with
// the same operations: the results are the same bits. The workgroups of a call
// before, its time before and after (bf16, 32 query heads over 8, head_dim 128,
// or 64 over 8, head_dim 64, graph replay):
//   1 sequence of 3971 (32)         16.3 -> 11.2 us      4 of 3000 to 4000 (128)  18.5 -> 17.3 us
//   1 of 16000 (128)                19.1 -> 19.0 us      1 of 32000 (256)         27.1 -> 30.5 us
//   8 of 500 to 2000 (128)          17.5 -> 14.1 us      16 of 1000 to 2000 (256) 22.7 -> 24.7 us
//   d 64: 1 of 4000 (32)            13.8 -> 10.5 us      4 of 2000 to 4000 (128)  14.9 -> 13.4 us
// A call of one split needs no merge kernel and is not spread; in a spread call
// a context of one share is written by its walk (1 sequence of 37 under a bound
// of 4096: 8.0 -> 6.4 us). At head_dim 64 a step's loads are half the registers,
// so the walk that loads ahead still has two workgroups per CU: it is taken up to
// kAheadBlocks workgroups (256: 15.2 -> 13.2, 512: 25.0 -> 24.0, 1024: 37.5 ->
// 35.4 and 23.0 -> 22.0 us), above which it gains or loses 1%. One split's calls
// lose (2048 workgroups of one step per wavefront 23.4 -> 28.3 us), and so does
// head_dim 128 (8192: 383 -> 390 us, 512: 41.9 -> 43.7 us).
//
// The grid is sized by max_seq_len, and a caller who captures its calls passes
// the longest context it will ever meet, so most workgroups can be without
// tokens. Such a workgroup costs a place on a CU until it has read its length:
// about 1 ns of the call at four wavefronts, half at two, a third at one. So
// above kFullBlocks workgroups two wavefronts take turns with a split's shares,
// above kHalfBlocks one does, and above kMostBlocks a workgroup takes every n-th
// split of its sequence, n at least kMinPieces so that one long context among
// many short ones keeps that many workgroups. The shares and merges are the same,
// and so are the bits. A call at four wavefronts always / by these rules (the
// workgroups of its bound):
//   256 sequences of 512 to 4096, bound 4096 (8192)    387 us (two: 389)
//   6 of 700 to 131071, bound 131071 (6144)            140.5 us (two: 143)
//   64 of 30 to 300, bound 16384 (8192)                16 us (two: 14)
//   256 of 1000 to 16000, bound 16000 (32768)          1280 / 1288 us
//   256 of 30 to 300, bound 8192 (16384)               43 / 34 us (one: 35.5)
//   256 of 30 to 300, bound 16384 (32768)              59 / 38 us (two: 43)
//   64 of 30 to 300, bound 131072 (65536)              67 / 16 us
//   256 of 200 to 1000, bound 131072 (262144)          318 / 106 us
//   255 of 30 to 1000 and one of 131071 (262144)       425 / 274 us
// (kMinPieces 32 / 48 / 64: 315 / 274 / 250 us on the last, but 42 / 50 / 57 us on
// 256 of 30 to 300, bound 131072).
// In fp32 four wavefronts lose on short contexts at any bound: up to kShortSteps
// steps and from kShortBlocks workgroups on two take turns too (32 query heads over 8, head_dim 64: 512 of 30 to
// 200 54 -> 47 us, 256 of 30 to 300 38 -> 35, 256 of 30 to 400 44 -> 45).
//
// The grid is one-dimensional with the kv head varying fastest and the split
// slowest, so consecutive workgroups, which the dispatcher deals round-robin to
// the 8 XCDs, carry equal work: putting the split first would send split k of
// every sequence to XCD k and starve the XCDs that hold the late splits only
// long sequences have. The G query heads sharing the kv head are served by
// every K/V byte read (grouped-query sharing).
//
// A wavefront walks its share in steps of 64 tokens (4 blocks of 16). Each
// block's K tile and V tile are read as they lie in memory, 1 KiB per 16-byte
// load (K and V are read once, so the loads are non-temporal), and the K and V
// loads of a block are issued together. Reading K lane-per-token instead (four
// 256-byte pieces from four blocks per load), or all K loads before all V
// loads, measured 4-6% slower: the memory system serves a block's two tiles
// best when they are asked for at once. The step's products and softmax (log2
// domain) follow once its loads have landed: bf16 on the matrix units
// (walk_bf16), fp32 on the vector unit (walk_f32). The vector form of the bf16
// walk was itself the limit at 8 query heads per kv head and a third of a
// step's latency at 4; against it the matrix form took, per call,
//   64 sequences of 512 to 4096, 64 query heads over 8, head_dim 128: 111 -> 96 us
//   12 sequences of 1 to 4096, 64 over 8, head_dim 64:                 31 -> 18 us
//   1 sequence of 3971, 32 over 8, head_dim 128:                     20.5 -> 16 us
//   256 sequences of 512 to 4096, 32 over 8, head_dim 128 (HBM-bound): 391 -> 387 us
//
// Only the last step of a sequence can hold slots past its length, whose
// contents are arbitrary (possibly NaN); a wavefront's last step masks them.
// Partials (m, l, o) of every split go to the workspace; a second kernel merges
// them (log-sum-exp), in an order that depends only on the sequence's length.

#include <algorithm>

#include "common.hpp"
#include "decode_walk.hpp"
#include "launch.hpp"

namespace kvattn {

constexpr long long kAheadBlocks = 1024;
constexpr long long kFullBlocks = 8192, kHalfBlocks = 16384, kMostBlocks = 32768;
constexpr long long kMinPieces = 48;
constexpr int kShortSteps = 6, kShortBlocks = 1024;   // fp32

// Orders a wavefront's LDS writes before its own later reads by other lanes.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The same in fp32 on the vector unit. Each lane dots its quarter of the rows
// of the four tokens in its slot (one per block) with the same dims of q (read
// from LDS), and the four lanes of a slot add their quarters with two row
// swaps; lane t then takes the score of token t of the step. In the dim-major V
// tile lane l owns dim rows l / R (R = 16-byte chunks per row) and a run of
// consecutive tokens, whose p reach it through LDS. my_id: the ids of the walk's
// blocks (at most 64), one per lane. whole_out, if not null: the walk is the whole
// context, and its result goes there (G rows of D) instead of its state to LDS.
template <int D, int G>
__device__ __forceinline__ void walk_f32(const DecodeTiles<false>& tiles, const uint4* q_lds,
                                         float* p_lds, int my_id, int t0, int t1,
                                         float scale_log2, float* o_out, float2* ml_out,
                                         float* whole_out) {
  using S = DecodeShape<D, false>;
  const int lane = threadIdx.x % kWave;
  float m_run[G], l_run[G], acc[S::kVI][G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m_run[h] = -INFINITY;
    l_run[h] = 0.f;
#pragma unroll
    for (int i = 0; i < S::kVI; ++i) acc[i][h] = 0.f;
  }
  // block of this lane's token within the step, and which quarter of the K
  // rows of its slot the lane holds
  const int kj = lane / S::kBS;
  const int vrc = lane % S::kR;   // this lane's chunk of a V dim row

  for (int tb = t0; tb < t1; tb += S::kTile) {
    const bool tail = tb + S::kTile > t1;   // the step may end inside a block
    int bid[S::kTB];
#pragma unroll
    for (int j = 0; j < S::kTB; ++j)
      bid[j] = __builtin_amdgcn_readlane(my_id, (tb - t0) / S::kBS + j);
    int my_b = bid[0];
#pragma unroll
    for (int j = 1; j < S::kTB; ++j) my_b = (kj == j) ? bid[j] : my_b;
    const bool kvalid = (!tail || tb + lane < t1) && (my_b >= 0);
    uint4 kreg[S::kTB][S::kVI], vreg[S::kTB][S::kVI];
    load_step<false>(tiles, bid, lane, lane, kreg, vreg);

    // ---- scores ----
    float part[S::kTB][G];
#pragma unroll
    for (int j = 0; j < S::kTB; ++j)
#pragma unroll
      for (int h = 0; h < G; ++h) part[j][h] = 0.f;
#pragma unroll
    for (int i = 0; i < S::kVI; ++i) {
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const uint4 qc = q_lds[h * S::kKCh + 4 * i + kj];
#pragma unroll
        for (int j = 0; j < S::kTB; ++j) {
          const uint4 k = kreg[j][i];
          float a = part[j][h];
          a = fmaf(__uint_as_float(k.x), __uint_as_float(qc.x), a);
          a = fmaf(__uint_as_float(k.y), __uint_as_float(qc.y), a);
          a = fmaf(__uint_as_float(k.z), __uint_as_float(qc.z), a);
          a = fmaf(__uint_as_float(k.w), __uint_as_float(qc.w), a);
          part[j][h] = a;
        }
      }
    }
    // this lane's token is slot lane % 16 of block kj
    float sc[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
#pragma unroll
      for (int j = 0; j < S::kTB; ++j) part[j][h] = cross_row_sum(part[j][h]);
      sc[h] = part[0][h];
#pragma unroll
      for (int j = 1; j < S::kTB; ++j) sc[h] = (kj == j) ? part[j][h] : sc[h];
    }

    // ---- online softmax over the step (log2 domain) ----
    float alpha[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float x = kvalid ? sc[h] * scale_log2 : -INFINITY;
      const float mn = fmaxf(m_run[h], wave_max(x));
      const float ref = (mn == -INFINITY) ? 0.f : mn;
      alpha[h] = fast_exp2(m_run[h] - ref);
      const float p = fast_exp2(x - ref);
      p_lds[lane * G + h] = p;
      l_run[h] = l_run[h] * alpha[h] + p;
      m_run[h] = mn;
    }
#pragma unroll
    for (int i = 0; i < S::kVI; ++i)
#pragma unroll
      for (int h = 0; h < G; ++h) acc[i][h] *= alpha[h];
    wave_lds_sync();

    // ---- p . v ----
#pragma unroll
    for (int j = 0; j < S::kTB; ++j) {
      if (bid[j] < 0) continue;
      const int tok0 = tb + j * S::kBS + vrc * S::kVec;   // first token of this lane's chunk
      float pf[4][G];
      const float* pp = p_lds + (j * S::kBS + vrc * 4) * G;
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int h = 0; h < G; ++h) pf[k][h] = pp[k * G + h];
#pragma unroll
      for (int i = 0; i < S::kVI; ++i) {
        const uint4 v = vreg[j][i];
        float vf[4] = {__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                       __uint_as_float(v.w)};
        if (tail) {
#pragma unroll
          for (int k = 0; k < 4; ++k) vf[k] = (tok0 + k < t1) ? vf[k] : 0.f;
        }
#pragma unroll
        for (int h = 0; h < G; ++h) {
          float a = acc[i][h];
#pragma unroll
          for (int k = 0; k < 4; ++k) a = fmaf(pf[k][h], vf[k], a);
          acc[i][h] = a;
        }
      }
    }
    wave_lds_sync();
  }

  // lane sums, merge the chunks of a dim row
  float l_tot[G];
#pragma unroll
  for (int h = 0; h < G; ++h) l_tot[h] = wave_sum(l_run[h]);
#pragma unroll
  for (int i = 0; i < S::kVI; ++i)
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int o = 1; o < S::kR; o <<= 1) acc[i][h] += __shfl_xor(acc[i][h], o, kWave);
  if (whole_out) {
    if (vrc != 0) return;
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float inv = l_tot[h] > 0.f ? 1.f / l_tot[h] : 0.f;
#pragma unroll
      for (int i = 0; i < S::kVI; ++i)
        whole_out[h * D + i * S::kDPI + lane / S::kR] = acc[i][h] * inv;
    }
    return;
  }
  if (vrc == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int i = 0; i < S::kVI; ++i) o_out[h * D + i * S::kDPI + lane / S::kR] = acc[i][h];
  }
  if (lane == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h) ml_out[h] = make_float2(m_run[h], l_tot[h]);
  }
}

// Four elements of a row of out (the at-th four), from the unnormalised o and
// the row sum l.
template <bool BF16>
__device__ __forceinline__ void write_row4(uint8_t* out, size_t at, float l, float4 o) {
  const float inv = l > 0.f ? 1.f / l : 0.f;
  if constexpr (BF16)
    reinterpret_cast<uint2*>(out)[at] =
        make_uint2(pack_bf16x2(o.x * inv, o.y * inv), pack_bf16x2(o.z * inv, o.w * inv));
  else
    reinterpret_cast<float4*>(out)[at] =
        make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
}

// Tokens of a wavefront's share of a split of n tokens: whole steps, spread
// evenly over the wavefronts.
constexpr int kStepTokens = 64;
__device__ __forceinline__ int share_tokens(int n) {
  return (n + kDecodeWaves * kStepTokens - 1) / (kDecodeWaves * kStepTokens) * kStepTokens;
}

// kSpread: one wavefront's share is a workgroup of its own. kAhead: the walk
// loads a step ahead. kTurns: a workgroup of fewer wavefronts than shares, which
// take turns, and with a piece of the context instead of one split. None of
// them changes a result.
template <int D, int G, bool BF16, bool kTwo, bool kAhead, bool kSpread, bool kTurns>
__global__ __attribute__((amdgpu_flat_work_group_size(kWave, kDecodeWaves * kWave),
                          amdgpu_waves_per_eu(kAhead && D == 128 ? 1 : 2)))
void decode_split_kernel(
    const uint8_t* __restrict__ q, const uint8_t* __restrict__ kv,
    const uint8_t* __restrict__ kv2, int num_base, int num_blocks,
    const int* __restrict__ block_table, const int* __restrict__ seq_lens,
    uint8_t* __restrict__ out, float* __restrict__ ws_o, float2* __restrict__ ws_ml,
    int num_seqs, int num_q_heads, int num_kv_heads, int max_blocks, int max_seq_len,
    int split_tokens, int max_splits, float scale_log2) {
  using S = DecodeShape<D, BF16>;
  constexpr int W = kDecodeWaves;
  const int wid = blockIdx.x;
  const int g = wid % num_kv_heads;
  const int s = (wid / num_kv_heads) % num_seqs;
  const int piece = wid / (num_kv_heads * num_seqs);
  const int wave =
      kSpread ? piece % W : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int h0 = g * G;
  const size_t row_bytes = (size_t)D * S::kEsz;

  int L = seq_lens[s];
  L = min(max(L, 0), min(max_seq_len, max_blocks * S::kBS));
  const int nsplit = (L + split_tokens - 1) / split_tokens;

  if (L == 0) {
    if (piece == 0) {
      uint4* o = reinterpret_cast<uint4*>(out + ((size_t)s * num_q_heads + h0) * row_bytes);
      for (int c = threadIdx.x; c < G * D * S::kEsz / 16; c += blockDim.x)
        o[c] = make_uint4(0, 0, 0, 0);
    }
    return;
  }
  const int* bt = block_table + (size_t)s * max_blocks;
  const size_t tile_bytes = (size_t)S::kTileElems * S::kEsz;
  const size_t head_off = (size_t)g * tile_bytes;
  const DecodeTiles<kTwo> tiles = {kv, kv2, num_base, 2 * (size_t)num_kv_heads * tile_bytes,
                                   head_off, (size_t)num_kv_heads * tile_bytes + head_off};
  const uint8_t* q_row = q + ((size_t)s * num_q_heads + h0) * row_bytes;

  constexpr int kStates = kSpread ? 1 : W;
  __shared__ __attribute__((aligned(16))) float o_lds[kStates][G * D];
  __shared__ float2 ml_lds[kStates][G];

  int split = kSpread ? piece / W : piece;
  if (split >= nsplit) return;
  for (;;) {
    const int s0 = split * split_tokens;                       // the split's tokens
    const int s1 = min(L, s0 + split_tokens);
    const int part_tokens = share_tokens(s1 - s0);
    const int parts = (s1 - s0 + part_tokens - 1) / part_tokens;   // shares with tokens
    const bool whole = nsplit == 1 && parts == 1;   // a context of one share: nothing to merge

    if constexpr (kSpread) {   // one share: its state goes out as it is
      if (wave >= parts) return;
      const int t0 = s0 + wave * part_tokens;
      walk_bf16<D, G, kTwo, kAhead>(tiles, reinterpret_cast<const uint16_t*>(q_row), bt,
                                    num_blocks, t0, min(s1, t0 + part_tokens), scale_log2,
                                    o_lds[0], ml_lds[0]);
      wave_lds_sync();
      const size_t row = (size_t)s * num_q_heads + h0;
      for (int e = threadIdx.x; e < G * D / 4; e += kWave) {
        const int h = e / (D / 4), d4 = e % (D / 4);
        const float4 o = reinterpret_cast<const float4*>(o_lds[0])[e];
        if (whole) {
          write_row4<BF16>(out, (row + h) * (D / 4) + d4, ml_lds[0][h].y,
                           fma_each(1.f, o, float4{}));
        } else {
          const size_t idx = ((row + h) * max_splits + split) * W + wave;
          reinterpret_cast<float4*>(ws_o)[idx * (D / 4) + d4] = o;
          if (d4 == 0) ws_ml[idx] = ml_lds[0][h];
        }
      }
      return;
    }
    // A wavefront without a share ends here (a barrier waits for those that are left)
    // and gives its registers back, which the next workgroup's wavefronts take: 160
    // contexts of 8 to 66, one query head per kv head, 8.8 -> 7.2 us; 512 of 30 to 200
    // 43.7 -> 39.8; 256 of 1 to 64 under a bound of 4096, 32 over 8, 23.0 -> 18.6.
    const int step = kTurns ? blockDim.x / kWave : W;
    if (wave >= parts) return;
    const int threads = min(parts, step) * kWave;   // that are left
    if constexpr (BF16) {
      for (int p = wave; p < parts; p += step) {
        const int t0 = s0 + p * part_tokens;
        walk_bf16<D, G, kTwo, kAhead>(tiles, reinterpret_cast<const uint16_t*>(q_row), bt,
                                      num_blocks, t0, min(s1, t0 + part_tokens), scale_log2,
                                      o_lds[p], ml_lds[p]);
        if constexpr (!kTurns) break;
      }
    } else {
      __shared__ float p_lds[W][S::kTile * G];
      __shared__ uint4 q_lds[G * S::kKCh];
      if (!kTurns || split == piece) {
        for (int i = threadIdx.x; i < G * S::kKCh; i += threads)
          q_lds[i] = reinterpret_cast<const uint4*>(q_row)[i];
        __syncthreads();
      }
      float* orow =   // a whole context leaves from the registers
          whole ? reinterpret_cast<float*>(out) + ((size_t)s * num_q_heads + h0) * D : nullptr;
      for (int p = wave; p < parts; p += step) {
        const int t0 = s0 + p * part_tokens, t1 = min(s1, t0 + part_tokens);
        walk_f32<D, G>(tiles, q_lds, p_lds[wave], walk_ids(bt, t0, t1, num_blocks), t0, t1,
                       scale_log2, o_lds[p], ml_lds[p], orow);
        if constexpr (!kTurns) break;
      }
      if (whole) return;
    }
    __syncthreads();

    // ---- merge the shares' states (log-sum-exp, in context order) ----
    for (int e = threadIdx.x; e < G * D / 4; e += threads) {
      const int h = e / (D / 4), d4 = e % (D / 4);
      merge_states<float4>(
          parts, [&](int j) { return reinterpret_cast<const float4*>(o_lds[j])[e]; },
          [&](int j) { return ml_lds[j][h]; },
          [&](float m, float l, float4 o) {
            const size_t row = (size_t)s * num_q_heads + h0 + h;
            if (nsplit == 1) {
              write_row4<BF16>(out, row * (D / 4) + d4, l, o);
            } else {
              const size_t idx = row * max_splits + split;
              reinterpret_cast<float4*>(ws_o)[idx * (D / 4) + d4] = o;
              if (d4 == 0) ws_ml[idx] = make_float2(m, l);
            }
          });
    }
    if constexpr (!kTurns) return;
    split += gridDim.x / (num_kv_heads * num_seqs);
    if (split >= nsplit) return;
    __syncthreads();   // the next split's shares overwrite the states
  }
}

// Merge the split partials of each (sequence, query head): latency-bound, a
// few KiB per pair. A split's D floats are read by D / 4 lanes with 16-byte
// loads, so a wavefront has kSPL splits in flight per load and four loads
// issued together; the weights are computed one split per lane. Up to
// kCombineWaveSplits splits one wavefront does the pair; a longer sequence is
// shared by the four wavefronts of a workgroup (kWide: one pair per workgroup
// instead of four), a contiguous quarter of its splits each, merged in LDS.
// Which of the two is taken depends only on the sequence's own length. kSpread:
// the partials are those of the wavefronts of a split, at most four. At
// 131071 tokens (128 splits) the serial loop this replaces took 23.7 us.
constexpr int kCombineWaves = 4;
constexpr int kCombineWaveSplits = 8;

template <int D, bool BF16, bool kWide, bool kSpread>
__global__ __launch_bounds__(kCombineWaves * kWave) void decode_combine_kernel(
    const float* __restrict__ ws_o, const float2* __restrict__ ws_ml,
    const int* __restrict__ seq_lens, uint8_t* __restrict__ out, int num_seqs,
    int num_q_heads, int max_blocks, int max_seq_len, int split_tokens, int max_splits) {
  constexpr int kLPS = D / 4;            // lanes per split row
  constexpr int kSPL = kWave / kLPS;     // splits per load
  constexpr int kUnroll = kSpread ? 2 : 4;
  constexpr int W = kSpread ? kDecodeWaves : 1;   // states per split
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int w = kWide ? blockIdx.x : blockIdx.x * kCombineWaves + wave;
  if (w >= num_seqs * num_q_heads) return;
  int L = seq_lens[w / num_q_heads];
  L = min(max(L, 0), min(max_seq_len, max_blocks * 16));
  const int ns = (L + split_tokens - 1) / split_tokens;
  if (ns <= 1 && (!kSpread || L <= kStepTokens)) return;   // written by the split kernel
  const bool shared = kWide && ns > kCombineWaveSplits;   // uniform over the workgroup
  if (kWide && !shared && wave != 0) return;
  const int per = shared ? (ns + kCombineWaves - 1) / kCombineWaves : ns;
  const int j0 = shared ? min(ns, wave * per) : 0;
  const int j1 = min(ns, j0 + per);
  const float2* ml = ws_ml + (size_t)w * max_splits * W;
  const float4* po = reinterpret_cast<const float4*>(ws_o + (size_t)w * max_splits * W * D);
  // Split j's states, in its workgroup's order and with its operations.
  auto split_parts = [&](int j) {
    const int n = min(L, (j + 1) * split_tokens) - j * split_tokens;
    const int per_part = share_tokens(n);
    return (n + per_part - 1) / per_part;
  };
  auto split_ml = [&](int j) {
    if constexpr (!kSpread) return ml[j];
    const int n = split_parts(j);
    float2 x[W];
#pragma unroll
    for (int p = 0; p < W; ++p) x[p] = ml[j * W + min(p, n - 1)];
    float mj = -INFINITY, lj = 0.f;
#pragma unroll
    for (int p = 0; p < W; ++p) mj = fmaxf(mj, x[p].x);
    const float rj = (mj == -INFINITY) ? 0.f : mj;
#pragma unroll
    for (int p = 0; p < W; ++p)
      if (p < n) lj = fmaf(fast_exp2(x[p].x - rj), x[p].y, lj);
    return make_float2(mj, lj);
  };

  float m = -INFINITY;
  for (int j = j0 + lane; j < j1; j += kWave) m = fmaxf(m, split_ml(j).x);
  m = wave_max(m);
  const float ref = (m == -INFINITY) ? 0.f : m;
  float l = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
  const int sub = lane / kLPS, col = lane % kLPS;
  for (int c = j0; c < j1; c += kWave) {
    float wgt = 0.f;                     // of split c + lane
    if (c + lane < j1) {
      const float2 x = split_ml(c + lane);
      wgt = fast_exp2(x.x - ref);
      l = fmaf(wgt, x.y, l);
    }
    const int cnt = min(kWave, j1 - c);
    for (int j = 0; j < cnt; j += kSPL * kUnroll) {
      float4 v[kUnroll];
      if constexpr (kSpread) {
        float4 x[kUnroll][W];
        float2 y[kUnroll][W];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
          const int jj = c + min(j + k * kSPL + sub, cnt - 1);
#pragma unroll
          for (int p = 0; p < W; ++p) {
            const int at = jj * W + min(p, split_parts(jj) - 1);
            x[k][p] = po[(size_t)at * kLPS + col];
            y[k][p] = ml[at];
          }
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
          const int n = split_parts(c + min(j + k * kSPL + sub, cnt - 1));
          float mj = -INFINITY;
#pragma unroll
          for (int p = 0; p < W; ++p) mj = fmaxf(mj, y[k][p].x);
          const float rj = (mj == -INFINITY) ? 0.f : mj;
          v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int p = 0; p < W; ++p) {
            if (p >= n) break;
            const float wp = fast_exp2(y[k][p].x - rj);
            v[k].x = fmaf(wp, x[k][p].x, v[k].x);
            v[k].y = fmaf(wp, x[k][p].y, v[k].y);
            v[k].z = fmaf(wp, x[k][p].z, v[k].z);
            v[k].w = fmaf(wp, x[k][p].w, v[k].w);
          }
        }
      } else {
#pragma unroll
        for (int k = 0; k < kUnroll; ++k)   // past the end: the last split, at weight 0
          v[k] = po[(size_t)(c + min(j + k * kSPL + sub, cnt - 1)) * kLPS + col];
      }
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        const int i = j + k * kSPL + sub;
        const float wk = __shfl(wgt, min(i, kWave - 1), kWave);
        if (i < cnt) {
          o[0] = fmaf(wk, v[k].x, o[0]);
          o[1] = fmaf(wk, v[k].y, o[1]);
          o[2] = fmaf(wk, v[k].z, o[2]);
          o[3] = fmaf(wk, v[k].w, o[3]);
        }
      }
    }
  }
  l = wave_sum(l);
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int x = kLPS; x < kWave; x <<= 1) o[k] += __shfl_xor(o[k], x, kWave);

  if constexpr (kWide) {
    __shared__ float4 o_lds[kCombineWaves][kLPS];
    __shared__ float2 ml_lds[kCombineWaves];
    if (shared) {
      if (sub == 0) o_lds[wave][col] = make_float4(o[0], o[1], o[2], o[3]);
      if (lane == 0) ml_lds[wave] = make_float2(m, l);
      __syncthreads();
      if (wave != 0) return;
      float mm = -INFINITY;
#pragma unroll
      for (int k = 0; k < kCombineWaves; ++k) mm = fmaxf(mm, ml_lds[k].x);
      const float r = (mm == -INFINITY) ? 0.f : mm;
      l = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = 0.f;
#pragma unroll
      for (int k = 0; k < kCombineWaves; ++k) {
        const float wk = fast_exp2(ml_lds[k].x - r);
        const float4 v = o_lds[k][col];
        l = fmaf(wk, ml_lds[k].y, l);
        o[0] = fmaf(wk, v.x, o[0]);
        o[1] = fmaf(wk, v.y, o[1]);
        o[2] = fmaf(wk, v.z, o[2]);
        o[3] = fmaf(wk, v.w, o[3]);
      }
    }
  }
  if (sub != 0) return;
  write_row4<BF16>(out, (size_t)w * kLPS + col, l, make_float4(o[0], o[1], o[2], o[3]));
}

template <int D, int G, bool BF16, bool kTwo = false>
static hipError_t launch_decode_t(const DecodeArgs& a) {
  const int max_splits = (a.max_seq_len + a.split_tokens - 1) / a.split_tokens;
  const int splits = max_splits > 0 ? max_splits : 1;
  long long blocks = (long long)splits * a.num_kv_heads * a.num_seqs;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  float* ws_o = reinterpret_cast<float*>(a.workspace);
  constexpr bool kCanSpread = BF16 && !kTwo;
  const bool spread =
      kCanSpread && max_splits > 1 && blocks <= kSpreadBlocks && a.spread_ml_offset != 0;
  float2* ws_ml = reinterpret_cast<float2*>(static_cast<uint8_t*>(a.workspace) +
                                            (spread ? a.spread_ml_offset : a.ws_ml_offset));
  // A context of at most 1, 2 or 3 steps has that many shares of one step each,
  // so further wavefronts would only wait.
  const int steps = (a.max_seq_len + kStepTokens - 1) / kStepTokens;
  int waves = spread || steps < 1 ? 1 : steps < kDecodeWaves ? steps : kDecodeWaves;
  const bool turns = waves == kDecodeWaves &&
                     (blocks > kFullBlocks ||
                      (!BF16 && steps <= kShortSteps && blocks >= kShortBlocks));
  if (turns) {
    waves = blocks <= kHalfBlocks ? 2 : 1;
    const long long per_piece = (long long)a.num_kv_heads * a.num_seqs;
    const long long pieces = std::max(kMinPieces, kMostBlocks / per_piece);
    blocks = per_piece * std::min<long long>(splits, pieces);
  }
  auto split = decode_split_kernel<D, G, BF16, kTwo, false, false, false>;
  if (turns) split = decode_split_kernel<D, G, BF16, kTwo, false, false, true>;
  if constexpr (kCanSpread) {
    if (spread)
      split = decode_split_kernel<D, G, BF16, kTwo, true, true, false>;
    else if constexpr (D == 64)
      if (max_splits > 1 && !turns && blocks <= kAheadBlocks)
        split = decode_split_kernel<D, G, BF16, kTwo, true, false, false>;
  }
  trace_before(a.stream, kTwo ? "decode_split_two_tensor" : "decode_split");
  hipLaunchKernelGGL(split, dim3((unsigned)(spread ? blocks * kDecodeWaves : blocks)),
                     dim3(waves * kWave), 0, a.stream, static_cast<const uint8_t*>(a.q),
                     static_cast<const uint8_t*>(a.kv), static_cast<const uint8_t*>(a.kv2),
                     a.num_base, a.num_blocks, a.block_table, a.seq_lens,
                     static_cast<uint8_t*>(a.out), ws_o, ws_ml, a.num_seqs, a.num_q_heads,
                     a.num_kv_heads, a.max_blocks, a.max_seq_len, a.split_tokens, splits,
                     a.scale * kLog2e);
  trace_after(a.stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || max_splits <= 1) return e;
  // A workgroup holds four pairs while a wavefront can do a pair alone, else one.
  const int pairs = a.num_seqs * a.num_q_heads;
  const bool wide = max_splits > kCombineWaveSplits;
  auto combine = wide ? decode_combine_kernel<D, BF16, true, false>
                      : decode_combine_kernel<D, BF16, false, false>;
  if constexpr (kCanSpread) {
    if (spread)
      combine = wide ? decode_combine_kernel<D, BF16, true, true>
                     : decode_combine_kernel<D, BF16, false, true>;
  }
  trace_before(a.stream, "decode_combine");
  hipLaunchKernelGGL(combine, dim3(wide ? pairs : (pairs + kCombineWaves - 1) / kCombineWaves),
                     dim3(kCombineWaves * kWave), 0, a.stream, ws_o, ws_ml, a.seq_lens,
                     static_cast<uint8_t*>(a.out), a.num_seqs, a.num_q_heads, a.max_blocks,
                     a.max_seq_len, a.split_tokens, splits);
  trace_after(a.stream);
  return hipGetLastError();
}

template <int D, bool BF16>
static hipError_t dispatch_g(const DecodeArgs& a, int G) {
  switch (G) {
    case 1: return launch_decode_t<D, 1, BF16>(a);
    case 2: return launch_decode_t<D, 2, BF16>(a);
    case 4: return launch_decode_t<D, 4, BF16>(a);
    case 8: return launch_decode_t<D, 8, BF16>(a);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_decode(const DecodeArgs& a) {
  const int G = a.num_q_heads / a.num_kv_heads;
  if (a.kv2) {   // two-tensor layer: built for bf16, head_dim 128
    if (!a.bf16 || a.head_dim != 128) return hipErrorNotSupported;
    switch (G) {
      case 1: return launch_decode_t<128, 1, true, true>(a);
      case 2: return launch_decode_t<128, 2, true, true>(a);
      case 4: return launch_decode_t<128, 4, true, true>(a);
      case 8: return launch_decode_t<128, 8, true, true>(a);
      default: return hipErrorInvalidValue;
    }
  }
  if (a.bf16) {
    if (a.head_dim == 128) return dispatch_g<128, true>(a, G);
    if (a.head_dim == 64) return dispatch_g<64, true>(a, G);
  } else {
    if (a.head_dim == 64) return dispatch_g<64, false>(a, G);
  }
  return hipErrorInvalidValue;
}

}  // namespace kvattn
