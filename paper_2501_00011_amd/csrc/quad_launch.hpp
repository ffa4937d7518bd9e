// Launchers of the quad solver's shapes, one translation unit per group of
// shapes (each kernel is large; the groups compile in parallel).
#pragma once

#include "quad_kernel.hpp"

namespace mcc {

// Set the dynamic local-memory limit of a shape's kernels / launch one.  The
// Multi-cells form is compiled for the shapes without a tail: no batch with a
// tail of 32 rows has a Multi-cells solver.
#define MCC_QUAD_PREPARE(TB, NC, FB, KU, W)                                                                      \
    for (const void *fn : {(const void *)quad_kernel<TB, NC, FB, KU, false, false, W>,                           \
                           (const void *)quad_kernel<TB, NC, FB, KU, false, true, W>,                            \
                           (const void *)quad_kernel<TB, NC, FB, KU, (FB == 0), false, W>}) {                    \
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
#define MCC_QUAD_LAUNCH_MC(TB, NC, FB, KU, W)                                                                      \
    if constexpr (FB == 0) {                                                                                       \
        QuadParams q = p;                                                                                          \
        void *args[] = {(void *)&q};                                                                               \
        return hipLaunchCooperativeKernel((const void *)quad_kernel<TB, NC, FB, KU, (FB == 0), false, W>,          \
                                          dim3((unsigned)((p.n_cells + kQCells - 1) / kQCells)), dim3(kWave), args, \
                                          (size_t)p.stride * kQCells * sizeof(double), s);                         \
    }                                                                                                              \
    return hipErrorInvalidValue;
// Wavefronts of the Multi-cells form that a compute unit holds.
#define MCC_QUAD_RESIDENT(TB, NC, FB, KU, W)                                                                      \
    if constexpr (FB == 0)                                                                                        \
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(                                                      \
            waves, (const void *)quad_kernel<TB, NC, FB, KU, (FB == 0), false, W>, kWave, lds_bytes);             \
    *waves = 0;                                                                                                   \
    return hipSuccess;

// The shapes (TB, NC, FB): dense (at most 16, 24 and 32 species), and a
// 32-row tail behind one to four blocks of front positions.
#define MCC_QUAD_SHAPES(X) X(1, 16, 0) X(2, 24, 0) X(2, 32, 0) X(2, 32, 1) X(2, 32, 2) X(2, 32, 3) X(2, 32, 4)
#define MCC_QUAD_DECLARE(TB, NC, FB)                              \
    hipError_t quad_prepare_##TB##_##NC##_##FB(int max_lds_bytes); \
    hipError_t quad_launch_##TB##_##NC##_##FB(const QuadParams &p, hipStream_t s); \
    hipError_t quad_launch_mc_##TB##_##NC##_##FB(const QuadParams &p, hipStream_t s); \
    hipError_t quad_resident_##TB##_##NC##_##FB(size_t lds_bytes, int *waves);
MCC_QUAD_SHAPES(MCC_QUAD_DECLARE)
#define MCC_QUAD_DEFINE(TB, NC, FB, KU, W)                                                                      \
    hipError_t quad_prepare_##TB##_##NC##_##FB(int max_lds_bytes) { MCC_QUAD_PREPARE(TB, NC, FB, KU, W) }        \
    hipError_t quad_launch_##TB##_##NC##_##FB(const QuadParams &p, hipStream_t s) { MCC_QUAD_LAUNCH(TB, NC, FB, KU, W) } \
    hipError_t quad_launch_mc_##TB##_##NC##_##FB(const QuadParams &p, hipStream_t s) { MCC_QUAD_LAUNCH_MC(TB, NC, FB, KU, W) } \
    hipError_t quad_resident_##TB##_##NC##_##FB(size_t lds_bytes, int *waves) { MCC_QUAD_RESIDENT(TB, NC, FB, KU, W) }

}  // namespace mcc
