// The last fp32 product of a model of at most 16 classes, with the softmax and the loss (gemm_f32_product.h).
#include "gemm_f32_product.h"

namespace dynb {

void launch_gemm_f32_head(const GemmArgs& a, const HeadArgs& head, unsigned tiles, void* stream) {
  hipLaunchKernelGGL((gemm_f32_kernel<MODE_FWD, 1, HeadArgs>), dim3(tiles), dim3(64), 0, (hipStream_t)stream, a, head);
}

}  // namespace dynb
