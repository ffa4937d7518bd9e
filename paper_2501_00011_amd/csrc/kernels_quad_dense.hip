// Quad solver kernels: see quad_kernel.hpp.
#include "quad_launch.hpp"

namespace mcc {
MCC_QUAD_DEFINE(1, 16, 0, 8, 2)
MCC_QUAD_DEFINE(2, 24, 0, 8, 2)
MCC_QUAD_DEFINE(2, 32, 0, 8, 2)
}  // namespace mcc

namespace mcc {

hipError_t prepare_quad_kernels(const QuadTables &q, int max_lds_bytes)
{
#define MCC_CASE(tb, nc, fb) \
    if (q.TB == tb && q.NC == nc && q.FB == fb) return quad_prepare_##tb##_##nc##_##fb(max_lds_bytes);
    MCC_QUAD_SHAPES(MCC_CASE)
#undef MCC_CASE
    return hipErrorInvalidValue;
}

hipError_t quad_multicell_capacity(const QuadTables &q, int device, int64_t *max_cells)
{
    *max_cells = 0;
    if (!q.ok) return hipSuccess;
    int waves = 0, n_cu = 0;
    hipError_t e = hipErrorInvalidValue;
#define MCC_CASE(tb, nc, fb)                          \
    if (q.TB == tb && q.NC == nc && q.FB == fb) \
        e = quad_resident_##tb##_##nc##_##fb((size_t)q.stride * kQCells * sizeof(double), &waves);
    MCC_QUAD_SHAPES(MCC_CASE)
#undef MCC_CASE
    if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device);
    if (e == hipSuccess) *max_cells = (int64_t)waves * n_cu * kQCells;
    return e;
}

hipError_t launch_quad_multicell(const QuadTables &q, const QuadParams &p, hipStream_t s)
{
    if (p.n_cells == 0) return hipSuccess;
#define MCC_CASE(tb, nc, fb) \
    if (q.TB == tb && q.NC == nc && q.FB == fb) return quad_launch_mc_##tb##_##nc##_##fb(p, s);
    MCC_QUAD_SHAPES(MCC_CASE)
#undef MCC_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_quad(const QuadTables &q, const QuadParams &p, hipStream_t s)
{
    if (p.n_cells == 0) return hipSuccess;
    if (p.n_cells > 0x7fffffff) return hipErrorInvalidValue;
#define MCC_CASE(tb, nc, fb) \
    if (q.TB == tb && q.NC == nc && q.FB == fb) return quad_launch_##tb##_##nc##_##fb(p, s);
    MCC_QUAD_SHAPES(MCC_CASE)
#undef MCC_CASE
    return hipErrorInvalidValue;
}

}  // namespace mcc
