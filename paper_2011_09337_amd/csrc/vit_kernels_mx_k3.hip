// vit_kernels_mx_k3.hip -- matrix-core integer kernel instances (stream and batch) for constraint length k = 3.
#include "vit_decoder_mx.h"

namespace vit {
void *pick_kernel_mx_k3(int beta, int in, bool batch, bool quad) { return pick_kernel_mx_k<3>(beta, in, batch, quad); }
}  // namespace vit
