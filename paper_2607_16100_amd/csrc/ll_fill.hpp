// Fill kernels used by the host entry points (region and output set-up).
#pragma once

#include "ll_device.hpp"

namespace llc {

// Set `bytes` bytes at `dst` (16-byte aligned) to 0xFF: the sentinel of
// every element type.
__global__ __launch_bounds__(256) void k_fill_ones(char *dst, uint64_t bytes) {
  const uint64_t full = bytes / 16;
  const u32x4 ones = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (uint64_t i = t; i < full; i += (uint64_t)gridDim.x * blockDim.x) *(u32x4 *)(dst + i * 16) = ones;
  if (t < bytes % 16) dst[full * 16 + t] = (char)0xFF;
}

// Reset the packet areas of every slice in one launch: zero bytes [lo, mid)
// and set bytes [mid, hi) to the sentinel.  Workgroup (x, y) serves slice y, so
// no lane divides by the slice's length.  A region's reset precedes every
// replay of a captured graph, and one launch costs less than the two it took:
// with the 4 MB region of 16 KiB calls at 8 ranks 4.2 us -> 2.3, with
// the 249 MB region of 1 MiB calls 37 us -> 31 (bound by the write
// rate of the memory-side cache, about 7 TB/s).
__global__ __launch_bounds__(256) void k_reset_areas(char *sym, uint64_t stride, uint64_t lo, uint64_t mid, uint64_t hi) {
  char *const slice = sym + (uint64_t)blockIdx.y * stride;
  const uint64_t step = (uint64_t)gridDim.x * 256 * 16;
  for (uint64_t at = lo + ((uint64_t)blockIdx.x * 256 + threadIdx.x) * 16; at < hi; at += step) {
    const uint32_t v = at < mid ? 0u : ProtoSent::kSentinel;
    *(u32x4 *)(slice + at) = u32x4{v, v, v, v};
  }
}

}  // namespace llc
