// FusedMM on the matrix cores, FP32 operands (apart from the rest so that the sources compile side by side)
#include "dense.hpp"
#include "kernels_dense.hpp"

namespace csrk {
DenseKernel dense_fused_kernel_f32(int ct, int ds) { return dense_fused_kernel<3>(ct, ds); }
DenseKernel dense_again_fused_f32(int ct, int ds) {
#define CSRK_DENSE_CASE(CT, DS) \
    if (ct == CT && ds == DS) return {dense_kernel<CT, DS, 3, true>, DenseCfg<CT, DS, 3>::kBytes};
    CSRK_DENSE_CASE(12, 1)
    CSRK_DENSE_CASE(12, 2)
    CSRK_DENSE_CASE(16, 1)
    CSRK_DENSE_CASE(16, 2)
#undef CSRK_DENSE_CASE
    return {nullptr, 0};
}
}  // namespace csrk
