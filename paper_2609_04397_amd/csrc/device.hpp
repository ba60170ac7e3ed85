// Device helpers shared by the real and the complex kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace vbcsr {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;

// Index of the calling wave in its workgroup.  The shift is the same for all
// lanes of a wave, but the compiler cannot see that; reading it from the
// first lane puts it (and every row descriptor, address and buffer resource
// derived from it) in scalar registers.
__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  Give every XCD one contiguous range of logical workgroups so that
// panels that share input rows (spatial neighbours) share an L2.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
  constexpr int nx = 8;
  const int x = bid % nx, r = bid / nx;
  const int q = nblocks / nx, rem = nblocks % nx;
  return x * q + min(x, rem) + r;
}

// Raw buffer access to one panel: the descriptor (base, size in bytes) is
// wave-uniform and lives in scalar registers, each lane supplies a 32-bit
// byte offset, and offsets at or beyond the size read as zero.  Panel value
// streams use the non-temporal hint.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t panel_rsrc(const void *base, uint32_t bytes) {
  // 0x00020000: raw 32-bit buffer format of the gfx9 family
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                           0x00020000);
}

// One buffer descriptor serves X when its rows span less than kXSpan bytes.
// Byte offsets are then the sum of a row part (kOutRow for a padding column)
// and a column part (kOutCol for a lane past nrhs): a sum with either or both
// lies beyond every such span and below 2^32, so the load returns zero.
constexpr int64_t kXSpan = (int64_t(1) << 31) - 4096;
constexpr uint32_t kOutRow = 0x80000000u, kOutCol = 0x7FFFF000u;

}  // namespace
}  // namespace vbcsr
