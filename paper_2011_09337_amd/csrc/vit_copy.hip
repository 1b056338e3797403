// vit_copy.hip -- copies of a list of byte ranges, used by the serving loop
// to move its work list and the LLRs of newly admitted frames from pinned
// host memory into the device in one launch per iteration, however many
// frames it holds (the decode kernels write the decoded bytes back into the
// host region themselves).  The range list itself may sit in device memory or
// in mapped pinned host memory.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vit_internal.h"

namespace vit {
namespace {

constexpr int kThreads = 256, kAhead = 4;

// Bytes sh .. sh + 15 of the 32 in a, b (sh uniform, 1..15).
__device__ __forceinline__ uint4 shifted(uint4 a, uint4 b, int sh) {
  if (sh & 8) {
    a = {a.z, a.w, b.x, b.y};
    b.x = b.z;
    b.y = b.w;
  }
  if (sh & 4) {
    a = {a.y, a.z, a.w, b.x};
    b.x = b.y;
  }
  const int r = sh & 3;
  return {__builtin_amdgcn_alignbyte(a.y, a.x, r), __builtin_amdgcn_alignbyte(a.z, a.y, r),
          __builtin_amdgcn_alignbyte(a.w, a.z, r), __builtin_amdgcn_alignbyte(b.x, a.w, r)};
}

// The lane above's word (the last lane's own).
__device__ __forceinline__ uint4 from_above(uint4 v) {
  return {(uint32_t)__shfl_down((int)v.x, 1), (uint32_t)__shfl_down((int)v.y, 1), (uint32_t)__shfl_down((int)v.z, 1),
          (uint32_t)__shfl_down((int)v.w, 1)};
}

// One workgroup per range (grid-strided), in 16-byte words of the destination
// whatever the source's alignment: a read across PCIe takes microseconds, and
// packed int8 frames begin at any byte.  A wave reads 64 aligned words (only
// such as hold a byte of the range) and stores the 63 that lie between them,
// each from its own word and the next lane's; where the source is aligned, all
// 64.  Each thread has kAhead words in flight before it stores.  Byte loads for
// such ranges: 8.0 MB in 2048 frames took 336 us; 175 now (46 GB/s).
__global__ __launch_bounds__(kThreads) void copy_list_kernel(const CopyRange *__restrict__ r, int32_t count) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int32_t i = blockIdx.x; i < count; i += gridDim.x) {
    const uint8_t *src = r[i].src;
    uint8_t *dst = r[i].dst;
    int64_t bytes = r[i].bytes;
    int64_t head = (int64_t)(-(uintptr_t)dst & 15u);  // up to the first whole word of the destination
    if (head > bytes) head = bytes;
    if ((int64_t)threadIdx.x < head) dst[threadIdx.x] = src[threadIdx.x];
    src += head;
    dst += head;
    bytes -= head;
    const int64_t words = bytes >> 4;
    const int sh = __builtin_amdgcn_readfirstlane((int)((uintptr_t)src & 15u));
    const uint4 *s4 = (const uint4 *)((uintptr_t)src & ~(uintptr_t)15);
    uint4 *d4 = (uint4 *)dst;
    const int64_t last = words - (sh ? 0 : 1);  // last word of the source that is needed
    const int per_wave = sh ? 63 : 64;
    const int64_t stride = (int64_t)per_wave * (kThreads / 64);
    for (int64_t base = (int64_t)per_wave * wave; base < words; base += kAhead * stride) {
      uint4 w[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int64_t at = base + u * stride + lane;
        w[u] = s4[at < last ? at : last];
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int64_t at = base + u * stride + lane;
        const uint4 v = sh ? shifted(w[u], from_above(w[u]), sh) : w[u];
        if (at < words && lane < per_wave) d4[at] = v;
      }
    }
    const int64_t tail = words << 4;
    if (tail + (int64_t)threadIdx.x < bytes) dst[tail + threadIdx.x] = src[tail + threadIdx.x];
  }
}

}  // namespace

hipError_t launch_copy_list(const CopyRange *ranges, int32_t count, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  const int grid = count < 2048 ? count : 2048;
  hipLaunchKernelGGL(copy_list_kernel, dim3(grid), dim3(kThreads), 0, stream, ranges, count);
  return hipGetLastError();
}

}  // namespace vit
