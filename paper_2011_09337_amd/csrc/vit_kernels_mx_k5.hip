// vit_kernels_mx_k5.hip -- matrix-core integer kernel instances (stream and batch) for constraint length k = 5.
#include "vit_decoder_mx.h"

namespace vit {
void *pick_kernel_mx_k5(int beta, int in, bool batch, bool quad) { return pick_kernel_mx_k<5>(beta, in, batch, quad); }
}  // namespace vit
