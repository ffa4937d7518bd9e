// Launchers of the quad solver's shapes, one translation unit per group of
// shapes (each kernel is large; the groups compile in parallel).
#pragma once

#include "quad_kernel.hpp"

namespace mcc {

// Set the dynamic local-memory limit of a shape's kernels / launch one.
#define MCC_QUAD_PREPARE(TB, NC, FB, KU, W)                                                                      \
    for (const void *fn : {(const void *)quad_kernel<TB, NC, FB, KU, false, false, W>,                           \
                           (const void *)quad_kernel<TB, NC, FB, KU, false, true, W>}) {                         \
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, max_lds_bytes); \
        if (e != hipSuccess) return e;                                                                           \
    }                                                                                                            \
    return hipSuccess;
#define MCC_QUAD_LAUNCH(TB, NC, FB, KU, W)                                                              \
    const dim3 grid((unsigned)((p.n_cells + kQCells - 1) / kQCells)), block(kWave);                     \
    const size_t lds = (size_t)p.stride * kQCells * sizeof(double);                                     \
    if (p.tape)                                                                                         \
        hipLaunchKernelGGL((quad_kernel<TB, NC, FB, KU, false, true, W>), grid, block, lds, s, p);      \
    else                                                                                                \
        hipLaunchKernelGGL((quad_kernel<TB, NC, FB, KU, false, false, W>), grid, block, lds, s, p);     \
    return hipGetLastError();

// The shapes (TB, NC, FB): dense (at most 16, 24 and 32 species), and a
// 32-row tail behind one to four blocks of front positions.
#define MCC_QUAD_SHAPES(X) X(1, 16, 0) X(2, 24, 0) X(2, 32, 0) X(2, 32, 1) X(2, 32, 2) X(2, 32, 3) X(2, 32, 4)
#define MCC_QUAD_DECLARE(TB, NC, FB)                              \
    hipError_t quad_prepare_##TB##_##NC##_##FB(int max_lds_bytes); \
    hipError_t quad_launch_##TB##_##NC##_##FB(const QuadParams &p, hipStream_t s);
MCC_QUAD_SHAPES(MCC_QUAD_DECLARE)
#define MCC_QUAD_DEFINE(TB, NC, FB, KU, W)                                                                      \
    hipError_t quad_prepare_##TB##_##NC##_##FB(int max_lds_bytes) { MCC_QUAD_PREPARE(TB, NC, FB, KU, W) }        \
    hipError_t quad_launch_##TB##_##NC##_##FB(const QuadParams &p, hipStream_t s) { MCC_QUAD_LAUNCH(TB, NC, FB, KU, W) }

}  // namespace mcc
