// What the entry points see of the matrix-core kernels (kernels_dense.hpp): which calls they can take, at what cost, with
// how much scratch, and the launch itself.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace csrk {

struct DenseArgs;

enum DenseOp { kDenseSpmm, kDenseSddmm, kDenseFused };

struct DenseShape {
    DenseOp op;
    bool bf16;              // the dense operands' type; otherwise float
    int M, K, N, D;         // N: output columns (0 for SDDMM), D: length of the dot products (0 for SPMM)
    bool ones = false;      // SDDMM: no stored values
};

struct DenseConfig {
    int ct;                 // 16-column pieces of the output per workgroup
    int ds;                 // 32-element steps of the dot products
    int segs, seg_k;        // K in `segs` ranges of `seg_k` columns
    bool halves;            // FP32 in half-precision pieces (kernels_dense_wide.hpp)
    double us;              // what the call is expected to take
    size_t bytes;           // of scratch
};

// false: not a shape for these kernels
bool dense_config(const DenseShape &s, int cus, DenseConfig *c);

// SDDMM: in slabs of scores (kernels_dense_sddmm.hpp)
bool sddmm_in_slabs(const DenseShape &s);
// What an SDDMM call with that share of S's cells stored is expected to take where it is done in slabs of scores; false: it is not.
bool sddmm_slab_us(const DenseShape &s, const DenseConfig &c, int cus, double density, double *us);

// `scratch`: 256-byte aligned, config's size.  Nothing is allocated and nothing read back; may be captured.
hipError_t dense_run(const DenseShape &s, const DenseConfig &c, const int32_t *rowptr, const int32_t *colidx, const float *vals,
                     const void *A, const void *B, const void *C, float *out, void *scratch, hipStream_t stream);

// the kernels of one kind: what to launch and with how much LDS
struct DenseKernel {
    void (*fn)(DenseArgs);
    int lds_bytes;
    int threads = 512;
};
DenseKernel dense_fused_kernel_f32(int ct, int ds);
DenseKernel dense_fused_kernel_bf16(int ct, int ds);
// the same kernel for calls whose results after half-precision pieces would mostly be computed again
DenseKernel dense_again_fused_f32(int ct, int ds);
// Wavefronts of a workgroup of the finishing kernel (kernels_dense_finish.hpp says what each is worth)
constexpr int finish_waves(bool halves, bool fused) { return halves ? (fused ? 8 : 16) : 4; }
// `vec`: 128-bit accesses of all dense operands and the output
DenseKernel dense_finish_kernel(bool bf16, bool fused, bool vec, int ct, bool halves);

}  // namespace csrk
