// The finishing kernels of matrix-core calls, in a file of their own so that the files compile side by side.
#include "kernels_dense_finish.hpp"

namespace csrk {
namespace {

template <typename E, bool FUSED>
DenseKernel finish_kernel(bool vec, int ct, bool halves) {
    constexpr int V = 16 / sizeof(E);
    if constexpr (sizeof(E) == 4)
        if (halves) return vec ? DenseKernel{dense_finish<E, FUSED, V, 256 / V, true>, 0} : DenseKernel{dense_finish<E, FUSED, 1, kWave, true>, 0};
    if (!vec) return {dense_finish<E, FUSED, 1, kWave>, 0};
    if (ct <= 2) return {dense_finish<E, FUSED, V, 32 / V>, 0};
    if (ct <= 4) return {dense_finish<E, FUSED, V, 64 / V>, 0};
    if (ct <= 8) return {dense_finish<E, FUSED, V, 128 / V>, 0};
    return {dense_finish<E, FUSED, V, 256 / V>, 0};
}

}  // namespace

DenseKernel dense_finish_kernel(bool bf16, bool fused, bool vec, int ct, bool halves) {
    return bf16 ? (fused ? finish_kernel<bf16_t, true>(vec, ct, false) : finish_kernel<bf16_t, false>(vec, ct, false))
                : (fused ? finish_kernel<float, true>(vec, ct, halves) : finish_kernel<float, false>(vec, ct, halves));
}

}  // namespace csrk
