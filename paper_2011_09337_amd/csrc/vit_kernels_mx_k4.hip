// vit_kernels_mx_k4.hip -- matrix-core integer kernel instances (stream and batch) for constraint length k = 4.
#include "vit_decoder_mx.h"

namespace vit {
void *pick_kernel_mx_k4(int beta, int in, bool batch, bool quad) { return pick_kernel_mx_k<4>(beta, in, batch, quad); }
}  // namespace vit
