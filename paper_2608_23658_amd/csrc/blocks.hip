// Copying whole KV blocks from one block id to another in every layer: how a
// caller drains the elastic block-id range before decommitting it (the
// paper, Section 3 "Controller": decommitting first drains the elastic blocks,
// syncs, then unmaps). One workgroup per (pair, layer), bound by HBM: 1024
// threads with four 16-byte non-temporal loads each in flight take 64 KiB in one
// go (every byte is read and written once), and what is left of a block, or a
// smaller block, in one go too, with the chunks past its end left out. 190 blocks
// in 32 layers, other blocks each time, against 256 threads with one cached load
// at a time:
//   64 KiB (797 MB)   159 -> 140 us, 5.7 TB/s     16 KiB   40.6 -> 36.1 us
//   32 KiB           79.4 -> 73.4 us              96 KiB    121 -> 108 us
// (with the rest of a block one cached load at a time 79.7, 42.1 and 119 us on the
// last three). Workgroups per 16 or 32 KiB of a block gain up to 6% at 32 and 96
// KiB and lose 4% at 64; 512 threads with eight loads 140 against 138, 256 with
// eight 148 (64 KiB, the same blocks over and over).

#include "common.hpp"
#include "launch.hpp"

namespace kvattn {

constexpr int kCopyThreads = 1024;
constexpr int kCopyUnroll = 4;

__global__ __launch_bounds__(kCopyThreads) void copy_blocks_kernel(
    CopyLayers layers, const int* __restrict__ src, const int* __restrict__ dst, int num_blocks,
    size_t block_bytes) {
  const int pair = blockIdx.x;
  const int s = src[pair], d = dst[pair];
  if (s < 0 || s >= num_blocks || d < 0 || d >= num_blocks || s == d) return;
  uint8_t* base = static_cast<uint8_t*>(layers.p[blockIdx.y]);
  const uint4* from = reinterpret_cast<const uint4*>(base + (size_t)s * block_bytes);
  uint4* to = reinterpret_cast<uint4*>(base + (size_t)d * block_bytes);
  const size_t n16 = block_bytes / 16;
  size_t i = threadIdx.x;
  for (; i + (kCopyUnroll - 1) * kCopyThreads < n16; i += kCopyUnroll * kCopyThreads) {
    uint4 v[kCopyUnroll];
#pragma unroll
    for (int k = 0; k < kCopyUnroll; ++k) v[k] = load_nt(from + i + k * kCopyThreads);
#pragma unroll
    for (int k = 0; k < kCopyUnroll; ++k) store_nt(to + i + k * kCopyThreads, v[k]);
  }
  if (i >= n16) return;
  uint4 v[kCopyUnroll];
#pragma unroll
  for (int k = 0; k < kCopyUnroll; ++k)
    if (i + k * kCopyThreads < n16) v[k] = load_nt(from + i + k * kCopyThreads);
#pragma unroll
  for (int k = 0; k < kCopyUnroll; ++k)
    if (i + k * kCopyThreads < n16) store_nt(to + i + k * kCopyThreads, v[k]);
}

hipError_t launch_copy_blocks(const CopyArgs& a) {
  if (a.n == 0 || a.num_layers == 0) return hipSuccess;
  for (int l0 = 0; l0 < a.num_layers; l0 += kMaxCopyLayers) {
    CopyLayers layers = {};
    const int nl = a.num_layers - l0 < kMaxCopyLayers ? a.num_layers - l0 : kMaxCopyLayers;
    for (int l = 0; l < nl; ++l) layers.p[l] = a.layers[l0 + l];
    trace_before(a.stream, "copy_blocks");
    hipLaunchKernelGGL(copy_blocks_kernel, dim3(a.n, nl), dim3(kCopyThreads), 0, a.stream, layers,
                       a.src, a.dst, a.num_blocks, a.block_bytes);
    trace_after(a.stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace kvattn
