// vit_expand.hip -- a batch's work list (one item per block, Sec. III per
// frame) written on the device from one record per frame.
//
// The host used to write the items (40 bytes per block) and a graph's copy
// nodes to upload them: 2.4 MB for 8192 frames in 60 k blocks, about half a
// millisecond before the first kernel could start.  A record is 48 bytes per
// frame (0.4 MB), read in place from pinned host memory; eight lanes take a
// record, so that a wave has eight reads across PCIe in flight.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vit_internal.h"

namespace vit {
namespace {

__global__ __launch_bounds__(256) void expand_kernel(ExpandArgs a) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < 3 * kMaxCodes) {
    const int c = (int)t % kMaxCodes;
    a.header[t] = t < kMaxCodes ? 0 : t < 2 * kMaxCodes ? a.count[c] : a.first[c];
  }
  const int64_t i = t >> 3;
  if (i >= a.nrecords) return;
  const FrameRecord r = a.records[i];
  const int c = r.code;
  const int64_t L = a.L[c], v1 = a.v1[c], v2 = a.v2[c];
  const int64_t n = r.n, N = n + (r.terminated ? a.tail[c] : 0);
  for (int32_t b = r.b0 + (int32_t)(t & 7); b < r.b1; b += 8) {
    const int64_t cs = b * L;
    const int64_t ce = cs + L < n ? cs + L : n;
    const int64_t s = cs - v1 > 0 ? cs - v1 : 0;
    const int64_t e = ce + v2 < N ? ce + v2 : N;
    WorkItem it;
    it.llr_off = r.llr_off;
    it.out_off = r.out_off;
    it.s = (int32_t)s;
    it.e = (int32_t)e;
    it.cs = (int32_t)cs;
    it.ce = (int32_t)ce;
    it.flags = (s == 0 ? 1 : 0) | ((r.terminated && e == N) ? 2 : 0);
    it.cost = (int32_t)(e - s);
    a.items[b == r.nblocks - 1 ? r.last : b == 0 ? r.front : r.middle + b - 1] = it;
  }
}

}  // namespace

hipError_t launch_expand(const ExpandArgs &a, hipStream_t stream) {
  const int64_t threads = a.nrecords * 8 > 3 * kMaxCodes ? a.nrecords * 8 : 3 * kMaxCodes;
  hipLaunchKernelGGL(expand_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace vit
