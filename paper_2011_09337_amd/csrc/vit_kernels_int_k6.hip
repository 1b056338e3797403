// vit_kernels_int_k6.hip -- integer kernel instances (stream and batch) for constraint length k = 6.
#include "vit_decoder_int.h"

namespace vit {
void *pick_kernel_int_k6(int beta, bool top, int in, bool batch) { return pick_kernel_int_k<6>(beta, top, in, batch); }
}  // namespace vit
