// vit_kernels_mx_k8.hip -- matrix-core integer kernel instances (stream and batch) for constraint length k = 8.
#include "vit_decoder_mx.h"

namespace vit {
void *pick_kernel_mx_k8(int beta, int in, bool batch, bool quad) { return pick_kernel_mx_k<8>(beta, in, batch, quad); }
}  // namespace vit
