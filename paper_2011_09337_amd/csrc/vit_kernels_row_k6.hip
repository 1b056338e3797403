// vit_kernels_row_k6.hip -- FP32 kernel instances of four blocks a wave (stream and batch) for constraint length k = 6.
#include "vit_decoder_row.h"

namespace vit {
void *pick_kernel_row_k6(int beta, bool batch) { return pick_kernel_row_k<6>(beta, batch); }
}  // namespace vit
