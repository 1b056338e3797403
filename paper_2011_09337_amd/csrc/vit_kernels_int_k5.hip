// vit_kernels_int_k5.hip -- integer kernel instances (stream and batch) for constraint length k = 5.
#include "vit_decoder_int.h"

namespace vit {
void *pick_kernel_int_k5(int beta, bool top, int in, bool batch) { return pick_kernel_int_k<5>(beta, top, in, batch); }
}  // namespace vit
