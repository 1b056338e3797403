// vit_kernels_row_k5.hip -- FP32 kernel instances of four blocks a wave (stream and batch) for constraint length k = 5.
#include "vit_decoder_row.h"

namespace vit {
void *pick_kernel_row_k5(int beta, bool batch) { return pick_kernel_row_k<5>(beta, batch); }
}  // namespace vit
