// One BDF outer step per cell, four cells per wavefront: a cell is a row of 16
// lanes.  (Method and per-cell control: as bdf_kernel in kernels_solve.hip.)
//
// Why rows of 16.  With one cell per wavefront the solver is bound by issue:
// most of a step attempt is chains of small operations -- a broadcast of one
// pivot's value, a handful of multiply-adds below it -- in which few of the 64
// lanes have work, and two cells fill a SIMD's issue slots.  A row of 16 lanes
// is the unit within which one instruction can broadcast a lane's FP64 value
// and multiply-add it (row_newbcast DPP on v_fmac_f64), so the same
// instruction serves four cells, a broadcast costs nothing, and one fetch of
// the mechanism's tables (L2) serves four cells.
//
// Rows of the system live in blocks of 16 (lane = row): the dense tail's blocks
// and the sparse front's.  Registers hold the per-species vectors (one double
// per block) and the dense tail (up to 32 x 32: one double per block and
// column), so that its factorisation and its part of the sweeps read no local
// memory; local memory holds the front's factors, y and the rates (10 KB for
// 72 species: 16 cells per compute unit, one wavefront per SIMD).
//
// Measured against the one-cell-per-wavefront kernel: 10,000 cells of 72
// species, one 180 s step (cells longest first, 32-row tail) 156 -> 91 ms;
// 30,000 cells of 20 species, 60 s 97 -> 33 ms; 10 cells of 20 species
// 8.4 -> 5.5 ms.  A wavefront's step attempt takes 106,000 cycles for four
// cells of 72 species (the other kernel: 105,000 for one, two sharing a SIMD):
// 14,700 instructions at 4.4 cycles each, a wavefront alone on its SIMD
// issuing at most one per four, and about 35,000 cycles of waits on dependent
// local-memory reads and table fetches.
//
// Spilled registers.  The tail, the middle pivots' multipliers and the state
// are more than a wavefront's 512 registers (256 without a front, two
// wavefronts on a SIMD): 36 to 187 of them spill behind a front, 83 for 72
// species, none to 119 without.  A spill saves and restores each lane's own
// value, under the branch it stands in.  That is safe here because nothing that
// reads other lanes (DPP, ballots, readlane) stands in a branch that divides a
// row: conditions around it are values of the cell, the same on a row's 16
// lanes, and DPP stays within the row.  The assembly below begins with the wait
// states a DPP source needs after any write, a reload's among them.  The taping
// build is allocated apart (132 spills for 72 species): the tests ask for the same
// bits from both, in every shape.  (A reverse-mode build of kernels_solve.hip
// that spilled once gave wrong sums for a reason not found; it is refused there.)
//
// The four cells of a wavefront take their step attempts together.  Whatever
// differs between them -- step size, order, acceptance, the end of the outer
// step -- is a per-lane value, equal on a row's 16 lanes; a finished cell's
// row idles until the last of the four is done.  No cell's arithmetic depends
// on its neighbours.
#pragma once

#include <type_traits>
#include <utility>

#include "grid_exchange.hpp"

namespace mcc {
namespace {

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// A wavefront's local-memory accesses are performed in the order it issues
// them: a hand-over between lanes needs only the compiler to keep that order.
__device__ __forceinline__ void lds_handover() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// This lane's place in its row, taken afresh where a phase begins: the lane
// masks formed from it then stay within the phase (the compiler would move
// them out of the step loop and spill them).
__device__ __forceinline__ int lane16()
{
    int l = (int)threadIdx.x & 15;
    asm volatile("" : "+v"(l));
    return l;
}

// The value of lane J of this lane's row of 16.  (Assembly rather than the
// builtin: the wait states a DPP source needs after it is written are counted
// by the compiler for its own instructions only, and the value often comes
// straight from the multiply-adds below.)
template <int J>
__device__ __forceinline__ double row_bcast(double v)
{
    double r;
    asm("s_nop 1\nv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v), "n"(J));
    return r;
}

// A table entry at uniform byte offset u and this lane's byte offset l.
template <class V>
__device__ __forceinline__ V ld(const void *base, uint32_t u, uint32_t l)
{
    return *reinterpret_cast<const V *>(static_cast<const char *>(base) + u + l);
}

template <int CTRL>
__device__ __forceinline__ double row_move(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// Reduction over the row's 16 lanes; every exchange combines two equal partial
// results, so all lanes of the row end with the same bits.  (The empty asm
// keeps a product that forms v from being contracted into the first sum, which
// would round differently on the two lanes of a pair.)
template <class Op>
__device__ __forceinline__ double row_reduce(double v, Op op)
{
    asm("" : "+v"(v));
    v = op(v, row_move<0xb1>(v));   // quad_perm [1, 0, 3, 2]
    v = op(v, row_move<0x4e>(v));   // quad_perm [2, 3, 0, 1]
    v = op(v, row_move<0x141>(v));  // row_half_mirror
    return op(v, row_move<0x140>(v));  // row_mirror
}
__device__ __forceinline__ double row_sum(double v)
{
    return row_reduce(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double row_min(double v)
{
    return row_reduce(v, [](double a, double b) { return fmin(a, b); });
}
__device__ __forceinline__ bool row_any(bool b)
{
    const unsigned long long m = __ballot(b);
    const unsigned half = (threadIdx.x & 32) ? (unsigned)(m >> 32) : (unsigned)m;
    return ((half >> (threadIdx.x & 16)) & 0xffffu) != 0;
}

// 1/x of a pivot: the hardware's estimate refined by two Newton steps, within
// about an ulp.
__device__ __forceinline__ double pivot_rcp(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
// of a pivot u, tested on 1/u: u zero, below 1e-300 or not finite
__device__ __forceinline__ bool pivot_bad(double inv) { return !(fabs(inv) <= 1e300); }

__device__ __noinline__ double quad_pow(double x, double y) { return pow(x, y); }

// gamma_j = sum_{i=1..j} 1/i
__device__ __forceinline__ double bdf_gamma(int j)
{
    double g = 0.0;
#pragma unroll
    for (int i = 1; i <= kMaxOrder; ++i) g = i <= j ? g + 1.0 / i : g;
    return g;
}

// Entry e (a constant) of 16-bit local-memory indices packed two to a word:
// index * 8 + the cell's byte address in one multiply-add.
__device__ __forceinline__ uint32_t field_addr(uint32_t w, int hi, uint32_t base)
{
    uint32_t a;
    if (hi)
        asm("v_mad_u32_u16 %0, %1, 8, %2 op_sel:[1,0,0,0]" : "=v"(a) : "v"(w), "v"(base));
    else
        asm("v_mad_u32_u16 %0, %1, 8, %2" : "=v"(a) : "v"(w), "v"(base));
    return a;
}
__device__ __forceinline__ __attribute__((address_space(3))) double &lds_at(uint32_t a)
{
    return *reinterpret_cast<__attribute__((address_space(3))) double *>(static_cast<uintptr_t>(a));
}
__device__ __forceinline__ double field(uint32_t w, int hi, uint32_t base) { return lds_at(field_addr(w, hi, base)); }

// a[q] -= (lane q of the row's u) * m, q = 0..15.  A DPP source is read two
// wait states after anything written before it (s_nop 1).
#define MCC_DPP(acc, src, m, lane) \
    "v_fmac_f64_dpp " acc ", -" src ", " m " row_newbcast:" lane " row_mask:0xf bank_mask:0xf\n"
__device__ __forceinline__ void fms_lanes16(double *a, double u, double m)
{
    asm("s_nop 1\n" MCC_DPP("%0", "%16", "%17", "0")
            MCC_DPP("%1", "%16", "%17", "1")
            MCC_DPP("%2", "%16", "%17", "2")
            MCC_DPP("%3", "%16", "%17", "3")
            MCC_DPP("%4", "%16", "%17", "4")
            MCC_DPP("%5", "%16", "%17", "5")
            MCC_DPP("%6", "%16", "%17", "6")
            MCC_DPP("%7", "%16", "%17", "7")
            MCC_DPP("%8", "%16", "%17", "8")
            MCC_DPP("%9", "%16", "%17", "9")
            MCC_DPP("%10", "%16", "%17", "10")
            MCC_DPP("%11", "%16", "%17", "11")
            MCC_DPP("%12", "%16", "%17", "12")
            MCC_DPP("%13", "%16", "%17", "13")
            MCC_DPP("%14", "%16", "%17", "14")
            MCC_DPP("%15", "%16", "%17", "15")
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15])
        : "v"(u), "v"(m));
}
// a[q] -= (lane K of the row's s[q]) * m for CNT (16, 8, 4, 2 or 1) columns; own: s = a
template <int K, int CNT>
__device__ __forceinline__ void fms_own(double *a, double m)
{
    if constexpr (CNT == 16)
        asm("s_nop 1\n" MCC_DPP("%0", "%0", "%16", "%17")
                MCC_DPP("%1", "%1", "%16", "%17")
                MCC_DPP("%2", "%2", "%16", "%17")
                MCC_DPP("%3", "%3", "%16", "%17")
                MCC_DPP("%4", "%4", "%16", "%17")
                MCC_DPP("%5", "%5", "%16", "%17")
                MCC_DPP("%6", "%6", "%16", "%17")
                MCC_DPP("%7", "%7", "%16", "%17")
                MCC_DPP("%8", "%8", "%16", "%17")
                MCC_DPP("%9", "%9", "%16", "%17")
                MCC_DPP("%10", "%10", "%16", "%17")
                MCC_DPP("%11", "%11", "%16", "%17")
                MCC_DPP("%12", "%12", "%16", "%17")
                MCC_DPP("%13", "%13", "%16", "%17")
                MCC_DPP("%14", "%14", "%16", "%17")
                MCC_DPP("%15", "%15", "%16", "%17")
            : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15])
            : "v"(m), "n"(K));
    else if constexpr (CNT == 8)
        asm("s_nop 1\n" MCC_DPP("%0", "%0", "%8", "%9") MCC_DPP("%1", "%1", "%8", "%9") MCC_DPP("%2", "%2", "%8", "%9")
                MCC_DPP("%3", "%3", "%8", "%9") MCC_DPP("%4", "%4", "%8", "%9") MCC_DPP("%5", "%5", "%8", "%9")
                    MCC_DPP("%6", "%6", "%8", "%9") MCC_DPP("%7", "%7", "%8", "%9")
            : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
            : "v"(m), "n"(K));
    else if constexpr (CNT == 4)
        asm("s_nop 1\n" MCC_DPP("%0", "%0", "%4", "%5") MCC_DPP("%1", "%1", "%4", "%5") MCC_DPP("%2", "%2", "%4", "%5")
                MCC_DPP("%3", "%3", "%4", "%5")
            : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3])
            : "v"(m), "n"(K));
    else if constexpr (CNT == 2)
        asm("s_nop 1\n" MCC_DPP("%0", "%0", "%2", "%3") MCC_DPP("%1", "%1", "%2", "%3") : "+v"(a[0]), "+v"(a[1]) : "v"(m), "n"(K));
    else
        asm("s_nop 1\n" MCC_DPP("%0", "%0", "%1", "%2") : "+v"(a[0]) : "v"(m), "n"(K));
}
template <int K, int CNT>
__device__ __forceinline__ void fms_from(double *a, const double *s, double m)
{
    if constexpr (CNT == 16)
        asm("s_nop 1\n" MCC_DPP("%0", "%16", "%32", "%33")
                MCC_DPP("%1", "%17", "%32", "%33")
                MCC_DPP("%2", "%18", "%32", "%33")
                MCC_DPP("%3", "%19", "%32", "%33")
                MCC_DPP("%4", "%20", "%32", "%33")
                MCC_DPP("%5", "%21", "%32", "%33")
                MCC_DPP("%6", "%22", "%32", "%33")
                MCC_DPP("%7", "%23", "%32", "%33")
                MCC_DPP("%8", "%24", "%32", "%33")
                MCC_DPP("%9", "%25", "%32", "%33")
                MCC_DPP("%10", "%26", "%32", "%33")
                MCC_DPP("%11", "%27", "%32", "%33")
                MCC_DPP("%12", "%28", "%32", "%33")
                MCC_DPP("%13", "%29", "%32", "%33")
                MCC_DPP("%14", "%30", "%32", "%33")
                MCC_DPP("%15", "%31", "%32", "%33")
            : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15])
            : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]), "v"(s[4]), "v"(s[5]), "v"(s[6]), "v"(s[7]), "v"(s[8]), "v"(s[9]), "v"(s[10]), "v"(s[11]), "v"(s[12]), "v"(s[13]), "v"(s[14]), "v"(s[15]), "v"(m), "n"(K));
    else if constexpr (CNT == 8)
        asm("s_nop 1\n" MCC_DPP("%0", "%8", "%16", "%17") MCC_DPP("%1", "%9", "%16", "%17")
                MCC_DPP("%2", "%10", "%16", "%17") MCC_DPP("%3", "%11", "%16", "%17") MCC_DPP("%4", "%12", "%16", "%17")
                    MCC_DPP("%5", "%13", "%16", "%17") MCC_DPP("%6", "%14", "%16", "%17") MCC_DPP("%7", "%15", "%16", "%17")
            : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
            : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]), "v"(s[4]), "v"(s[5]), "v"(s[6]), "v"(s[7]), "v"(m), "n"(K));
    else if constexpr (CNT == 4)
        asm("s_nop 1\n" MCC_DPP("%0", "%4", "%8", "%9") MCC_DPP("%1", "%5", "%8", "%9") MCC_DPP("%2", "%6", "%8", "%9")
                MCC_DPP("%3", "%7", "%8", "%9")
            : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3])
            : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]), "v"(m), "n"(K));
    else if constexpr (CNT == 2)
        asm("s_nop 1\n" MCC_DPP("%0", "%2", "%4", "%5") MCC_DPP("%1", "%3", "%4", "%5")
            : "+v"(a[0]), "+v"(a[1])
            : "v"(s[0]), "v"(s[1]), "v"(m), "n"(K));
    else
        asm("s_nop 1\n" MCC_DPP("%0", "%1", "%2", "%3") : "+v"(a[0]) : "v"(s[0]), "v"(m), "n"(K));
}

// b[q] -= (lane K of the row's x) * m[q], q < N
template <int K, int N>
__device__ __forceinline__ void fms_col(double *b, double x, const double *m)
{
    static_assert(N >= 1 && N <= 6, "");
    if constexpr (N == 1)
        asm("s_nop 1\n" MCC_DPP("%0", "%1", "%2", "%3") : "+v"(b[0]) : "v"(x), "v"(m[0]), "n"(K));
    else if constexpr (N == 2)
        asm("s_nop 1\n" MCC_DPP("%0", "%2", "%3", "%5") MCC_DPP("%1", "%2", "%4", "%5")
            : "+v"(b[0]), "+v"(b[1])
            : "v"(x), "v"(m[0]), "v"(m[1]), "n"(K));
    else if constexpr (N == 3)
        asm("s_nop 1\n" MCC_DPP("%0", "%3", "%4", "%7") MCC_DPP("%1", "%3", "%5", "%7") MCC_DPP("%2", "%3", "%6", "%7")
            : "+v"(b[0]), "+v"(b[1]), "+v"(b[2])
            : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "n"(K));
    else if constexpr (N == 4)
        asm("s_nop 1\n" MCC_DPP("%0", "%4", "%5", "%9") MCC_DPP("%1", "%4", "%6", "%9") MCC_DPP("%2", "%4", "%7", "%9")
                MCC_DPP("%3", "%4", "%8", "%9")
            : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3])
            : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "n"(K));
    else if constexpr (N == 5)
        asm("s_nop 1\n" MCC_DPP("%0", "%5", "%6", "%11") MCC_DPP("%1", "%5", "%7", "%11")
                MCC_DPP("%2", "%5", "%8", "%11") MCC_DPP("%3", "%5", "%9", "%11") MCC_DPP("%4", "%5", "%10", "%11")
            : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4])
            : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "n"(K));
    else
        asm("s_nop 1\n" MCC_DPP("%0", "%6", "%7", "%13") MCC_DPP("%1", "%6", "%8", "%13")
                MCC_DPP("%2", "%6", "%9", "%13") MCC_DPP("%3", "%6", "%10", "%13") MCC_DPP("%4", "%6", "%11", "%13")
                    MCC_DPP("%5", "%6", "%12", "%13")
            : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4]), "+v"(b[5])
            : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]), "n"(K));
}

// The same with x = b[0] itself (its own update last; lane K's m[0] is zero)
template <int K, int N>
__device__ __forceinline__ void fms_col_own(double *b, const double *m)
{
    static_assert(N >= 1 && N <= 6, "");
    if constexpr (N == 1)
        asm("s_nop 1\n" MCC_DPP("%0", "%0", "%1", "%2") : "+v"(b[0]) : "v"(m[0]), "n"(K));
    else if constexpr (N == 2)
        asm("s_nop 1\n" MCC_DPP("%1", "%0", "%3", "%4") MCC_DPP("%0", "%0", "%2", "%4")
            : "+v"(b[0]), "+v"(b[1])
            : "v"(m[0]), "v"(m[1]), "n"(K));
    else if constexpr (N == 3)
        asm("s_nop 1\n" MCC_DPP("%1", "%0", "%4", "%6") MCC_DPP("%2", "%0", "%5", "%6") MCC_DPP("%0", "%0", "%3", "%6")
            : "+v"(b[0]), "+v"(b[1]), "+v"(b[2])
            : "v"(m[0]), "v"(m[1]), "v"(m[2]), "n"(K));
    else if constexpr (N == 4)
        asm("s_nop 1\n" MCC_DPP("%1", "%0", "%5", "%8") MCC_DPP("%2", "%0", "%6", "%8") MCC_DPP("%3", "%0", "%7", "%8")
                MCC_DPP("%0", "%0", "%4", "%8")
            : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3])
            : "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "n"(K));
    else if constexpr (N == 5)
        asm("s_nop 1\n" MCC_DPP("%1", "%0", "%6", "%10") MCC_DPP("%2", "%0", "%7", "%10")
                MCC_DPP("%3", "%0", "%8", "%10") MCC_DPP("%4", "%0", "%9", "%10") MCC_DPP("%0", "%0", "%5", "%10")
            : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4])
            : "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "n"(K));
    else
        asm("s_nop 1\n" MCC_DPP("%1", "%0", "%7", "%12") MCC_DPP("%2", "%0", "%8", "%12")
                MCC_DPP("%3", "%0", "%9", "%12") MCC_DPP("%4", "%0", "%10", "%12") MCC_DPP("%5", "%0", "%11", "%12")
                    MCC_DPP("%0", "%0", "%6", "%12")
            : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4]), "+v"(b[5])
            : "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]), "n"(K));
}

template <int TB, int NC, int FB, int KU>
struct Quad {
    static constexpr int NB = TB + FB;
    static constexpr int NBP = (NB + 3) / 4 * 4;
    static constexpr bool kFull = FB > 0;  // the tail has exactly NC columns

    const QuadParams &p;
    uint32_t base;  // local-memory byte address of this lane's cell
    int i;          // lane of the row
    double kr[KU];  // rate constants of this lane's reactions (16 u + i)
    double T[TB][NC], dinv[TB];

    __device__ __forceinline__ Quad(const QuadParams &pp, const double *smem)
        : p(pp), base((uint32_t)(uintptr_t)smem + (uint32_t)((threadIdx.x >> 4) * pp.stride * 8)), i((int)threadIdx.x & 15)
    {
    }

    // Launch parameters read afresh where a phase begins, as in the
    // one-cell-per-wavefront solver: keeping them all in scalar registers
    // across the step loop spills.
    typedef const __attribute__((address_space(4))) QuadParams KParams;
    static __device__ __forceinline__ KParams &params_here()
    {
        KParams *q = (KParams *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(q));
        return *q;
    }

    // y, compact by position: the front, then the tail (whose unused rows
    // follow it, and which is written last: the front's unused rows overlap it)
    __device__ __forceinline__ void put_y(KParams &p, const double (&v)[NB])
    {
        lds_handover();
        const uint32_t a = base + 8u * (uint32_t)(p.off_y + i);
#pragma unroll
        for (int f = 0; f < FB; ++f) lds_at(a + 128u * f) = v[f];
        lds_handover();
        const uint32_t at = a + 8u * (uint32_t)p.F;
#pragma unroll
        for (int t = 0; t < TB; ++t) lds_at(at + 128u * t) = v[FB + t];
        lds_handover();
    }

    // Reaction rates (PART false) or rate partials times -c (PART true) at v,
    // lane per reaction, four rounds of 16 together (the table ends in idle
    // rounds that write to the write-only cell).
    template <bool PART>
    __device__ __forceinline__ void rates(KParams &p, const double (&v)[NB], double nc)
    {
        const uint32_t il = 16u * i;
        const int n = p.n_rx;
        uint4 a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = ld<uint4>(p.rx, 256u * u, il);
        put_y(p, v);
#pragma unroll
        for (int u0 = 0; u0 < KU; u0 += 4) {
            if (u0 >= n) break;
            double ya[4], yb[4], yc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                ya[u] = field(a[u].x, 0, base);
                yb[u] = field(a[u].x, 1, base);
                yc[u] = field(a[u].y, 0, base);
            }
            uint4 cur[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                cur[u] = a[u];
                if (u0 + 4 < KU) a[u] = ld<uint4>(p.rx, 256u * (u0 + 4 + u), il);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (PART) {
                    const double k = nc * kr[u0 + u], kb = k * yb[u], ka = k * ya[u];
                    lds_at(field_addr(cur[u].z, 0, base)) = kb * yc[u];
                    lds_at(field_addr(cur[u].z, 1, base)) = ka * yc[u];
                    lds_at(field_addr(cur[u].w, 0, base)) = ka * yb[u];
                } else {
                    double r = kr[u0 + u] * ya[u];
                    r *= yb[u];
                    r *= yc[u];
                    lds_at(field_addr(cur[u].y, 1, base)) = r;
                }
            }
        }
        lds_handover();
    }

    // f at v: rates, then every row's sum of nu r, two terms of every block's
    // rows per iteration.
    __device__ __forceinline__ void deriv(const double (&v)[NB], double (&f)[NB])
    {
        KParams &p = params_here();
        struct Rec {
            double2 c[NB];
            uint4 w[NBP / 4];
        };
        const int n = p.fg_iters;
        const uint32_t lc = 16u * i, li = 4u * NBP * i;
        auto load = [&](int it) {
            Rec r;
#pragma unroll
            for (int b = 0; b < NB; ++b) r.c[b] = ld<double2>(p.fg_coef, (uint32_t)(it * NB + b) * 256u, lc);
#pragma unroll
            for (int x = 0; x < NBP / 4; ++x) r.w[x] = ld<uint4>(p.fg_idx, (uint32_t)it * (64u * NBP) + 16u * x, li);
            return r;
        };
        Rec r0 = load(0), r1 = load(1);
        rates<false>(p, v, 0.0);
        double acc[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = 0.0;
        auto use = [&](const Rec &r) {
            double x0[NB], x1[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint4 &w4 = r.w[b / 4];
                const uint32_t w = b % 4 == 0 ? w4.x : b % 4 == 1 ? w4.y : b % 4 == 2 ? w4.z : w4.w;
                x0[b] = field(w, 0, base);
                x1[b] = field(w, 1, base);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] += r.c[b].x * x0[b];
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] += r.c[b].y * x1[b];
        };
        for (int it = 0; it < n; it += 2) {
            use(r0);
            r0 = load(it + 2);
            use(r1);
            r1 = load(it + 3);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) f[b] = acc[b];
    }

    // One set of Newton-matrix entries from the rate partials (which carry the
    // factor -c): m = sum of coef * partial (+ 1 on the diagonal).  A record's
    // partials are read while the one before it is finished.
    // The first four records are fetched ahead (nm_fetch), each later one four
    // records before its use.
    struct NmRec {
        double2 c0, c1;
        uint4 w;
    };
    __device__ __forceinline__ NmRec nm_load(const uint32_t *recs, int r) const
    {
        static_assert(sizeof(QNmRec) == 48, "");
        const uint32_t u = (uint32_t)r * (16 * sizeof(QNmRec)), il = 16u * i;
        return NmRec{ld<double2>(recs, u, il), ld<double2>(recs, u + 256, il), ld<uint4>(recs, u + 512, il)};
    }
    __device__ __forceinline__ void nm_fetch(const uint32_t *recs, NmRec (&r)[4]) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = nm_load(recs, q);
    }
    __device__ __forceinline__ void nm_set(const uint32_t *recs, int n, int two, int one, NmRec (&rec)[4])
    {
        using Rec = NmRec;
        auto load = [&](int r) { return nm_load(recs, r); };
        struct X {
            double x0, x1, x2, x3;
        };
        auto read = [&](const Rec &r) {
            return X{field(r.w.x, 0, base), field(r.w.x, 1, base), field(r.w.y, 0, base), field(r.w.y, 1, base)};
        };
        Rec r0 = rec[0], r1 = rec[1], r2 = rec[2], r3 = rec[3];
        X x0 = read(r0);
        double acc = 0.0;
        auto chain = [&](const Rec &r, const X &x) {
            acc += r.c0.x * x.x0;
            acc += r.c0.y * x.x1;
            acc += r.c1.x * x.x2;
            acc += r.c1.y * x.x3;
            const uint32_t kind = (uint32_t)__builtin_amdgcn_readfirstlane((int)r.w.w) >> 16;
            if (kind != kQNmMore) {
                lds_at(field_addr(r.w.z, 0, base)) = acc + (kind == kQNmDiag ? 1.0 : 0.0);
                acc = 0.0;
            }
        };
        auto pairs = [&](const Rec &r, const X &x) {
            lds_at(field_addr(r.w.z, 0, base)) = r.c0.x * x.x0 + r.c0.y * x.x1;
            lds_at(field_addr(r.w.z, 1, base)) = r.c1.x * x.x2 + r.c1.y * x.x3;
        };
        auto single = [&](const Rec &r, const X &x) {
            lds_at(field_addr(r.w.z, 0, base)) = r.c0.x * x.x0;
            lds_at(field_addr(r.w.z, 1, base)) = r.c0.y * x.x1;
            lds_at(field_addr(r.w.w, 0, base)) = r.c1.x * x.x2;
            lds_at(field_addr(r.w.w, 1, base)) = r.c1.y * x.x3;
        };
        auto run = [&](int r, int end, auto &&f) {
            for (; r < end; r += 4) {
                X x1 = read(r1);
                f(r0, x0);
                r0 = load(r + 4);
                x0 = read(r2);
                f(r1, x1);
                r1 = load(r + 5);
                x1 = read(r3);
                f(r2, x0);
                r2 = load(r + 6);
                x0 = read(r0);
                f(r3, x1);
                r3 = load(r + 7);
            }
        };
        run(0, two, chain);
        run(two, one, pairs);
        run(one, n, single);
        lds_handover();
    }

    // zeros into a list of entries (its first vector fetched ahead)
    __device__ __forceinline__ void zero(const uint16_t *list, int n, uint4 w)
    {
        for (int q = 0; q < n; ++q) {
            const uint4 next = ld<uint4>(list, 256u * (q + 1), 16u * i);
            const uint32_t a[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int x = 0; x < 8; ++x) lds_at(field_addr(a[x / 2], x % 2, base)) = 0.0;
            w = next;
        }
        lds_handover();
    }

    // Assembles M = I - c J(v) and factorises it; returns this lane's part of
    // "a pivot is zero, tiny or not finite".
    __device__ __forceinline__ bool factor(const double (&v)[NB], double c)
    {
        KParams &p = params_here();
        NmRec nr[4];
        nm_fetch(p.nm[0], nr);
        rates<true>(p, v, -c);
        // first part, tail, second part (see QuadTables)
        int unit = 0;
#pragma unroll 1
        for (int part = 0; part < (FB > 0 ? 2 : 1); ++part) {
            uint4 z{};
            LuRec lr[2];
            if constexpr (FB > 0) {
                z = ld<uint4>(p.fill[part], 0, 16u * i);
                lr[0] = lu_load(p, unit);
                lr[1] = lu_load(p, unit + 1);
            }
            nm_set(p.nm[part], p.nm_recs[part], p.nm_two[part], p.nm_one[part], nr);
            uint4 tm[TB * NC / 8];
            if (part == 0)
#pragma unroll
                for (int e = 0; e < TB * NC / 8; ++e) tm[e] = ld<uint4>(p.tmap, 256u * e, 16u * i);
            if constexpr (FB > 0) {
                zero(p.fill[part], p.n_fill[part], z);  // (the second part's held rate partials until here)
                if (part == 0) nm_fetch(p.nm[1], nr);
                front(p, unit, p.n_lu[part], lr);
                unit += p.n_lu[part];
            }
            if (part == 0) {
#pragma unroll
                for (int e = 0; e < TB * NC; e += 8) {
                    const uint4 w = tm[e / 8];
                    double *t = &T[e / NC][e % NC];
                    t[0] = field(w.x, 0, base);
                    t[1] = field(w.x, 1, base);
                    t[2] = field(w.y, 0, base);
                    t[3] = field(w.y, 1, base);
                    t[4] = field(w.z, 0, base);
                    t[5] = field(w.z, 1, base);
                    t[6] = field(w.w, 0, base);
                    t[7] = field(w.w, 1, base);
                }
                lds_handover();
            }
        }
        bool bad = false;
        if constexpr (FB > 0) {
            uint4 first[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) first[q] = ld<uint4>(p.mid_load, 256u * (q < 2 ? q : q + 4), 16u * i);
            schur(p);
            middle(p, first);
#pragma unroll
            for (int f = 0; f < FB; ++f) bad |= pivot_bad(field(ld<uint16_t>(p.dmap, 32u * f, 2u * i), 0, base));
        }
        return (dense(p) ? 1 : 0) | (bad ? 1 : 0);
    }

    // The front's entries, level by level (see build_quad); the first two units
    // are fetched ahead, each later one two units before its use.
    struct LuRec {
        uint4 h, s[kQLuSteps];
        uint32_t flags;
    };
    __device__ __forceinline__ LuRec lu_load(KParams &p, int u) const
    {
        static_assert(sizeof(QLuUnit) == 80 && kQLuEnt == 4 && kQLuSteps == 4, "");
        const uint32_t at = (uint32_t)u * (16 * sizeof(QLuUnit)), il = 16u * i;
        const auto *flags = (const __attribute__((address_space(4))) uint32_t *)p.lu_flags;  // uniform: scalar loads
        LuRec r;
        r.h = ld<uint4>(p.lu, at, il);
#pragma unroll
        for (int s = 0; s < kQLuSteps; ++s) r.s[s] = ld<uint4>(p.lu, at + 256u + 256u * s, il);
        r.flags = flags[u];
        return r;
    }
    __device__ __forceinline__ void front(KParams &p, int first, int n, LuRec (&rec)[2])
    {
        using Rec = LuRec;
        auto load = [&](int u) { return lu_load(p, u); };
        double a[4] = {0.0, 0.0, 0.0, 0.0};
        auto use = [&](const Rec &r) {
            const uint32_t fl = r.flags;
            const int ns = fl & 15;
            uint32_t d[4];
            double sc[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) d[e] = field_addr(e < 2 ? r.h.x : r.h.y, e & 1, base);
            if (!(fl & kQLuCont))
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = lds_at(d[e]);
#pragma unroll
            for (int e = 0; e < 4; ++e) sc[e] = field(e < 2 ? r.h.z : r.h.w, e & 1, base);
            auto terms = [&](auto CNT) {
                constexpr int cnt = decltype(CNT)::value;
                double l[cnt][4], u[cnt][4];
#pragma unroll
                for (int s = 0; s < cnt; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t w = e == 0 ? r.s[s].x : e == 1 ? r.s[s].y : e == 2 ? r.s[s].z : r.s[s].w;
                        l[s][e] = field(w, 0, base);
                        u[s][e] = field(w, 1, base);
                    }
#pragma unroll
                for (int s = 0; s < cnt; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[e] -= l[s][e] * u[s][e];
            };
            if (ns > 2) terms(std::integral_constant<int, 4>{});
            else if (ns == 2) terms(std::integral_constant<int, 2>{});
            else if (ns == 1) terms(std::integral_constant<int, 1>{});
            if (!(fl & kQLuMore)) {
                double x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = a[e] * sc[e];
                if (fl & (15 * kQLuD)) {  // diagonals: few units have any
                    asm volatile("");     // (a branch, not a select over four reciprocals)
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = fl & (kQLuD << e) ? pivot_rcp(a[e]) : x[e];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) lds_at(d[e]) = x[e];
            }
            lds_handover();
        };
        Rec r0 = rec[0], r1 = rec[1];
        for (int u = first; u < first + n; u += 2) {
            use(r0);
            r0 = load(u + 2);
            use(r1);
            r1 = load(u + 3);
        }
    }

    // T -= L_TF U_FT over the pivots split .. m0 - 1, one at a time: a pivot's L
    // in this lane's tail rows times its U in the tail columns, which the row's
    // lanes hold.  Two pivots per trip, the operands of one read while the
    // other's update runs, and no branch in the trip: around a branch the
    // compiler moves the tail between registers (an odd pivot count ends with
    // an all-zero pivot).
    __device__ __forceinline__ void schur(KParams &p)
    {
        if constexpr (TB == 2 && NC == 32) {
            const int n = p.m0 - p.split;
            const uint32_t il = 8u * i;
            auto idx = [&](int k) { return ld<uint2>(p.schur, 128u * (uint32_t)k, il); };
            struct Val {
                double l0, l1, u0, u1;
            };
            auto get = [&](const uint2 &w) { return Val{field(w.x, 0, base), field(w.x, 1, base), field(w.y, 0, base), field(w.y, 1, base)}; };
            auto step = [&](const Val &v) {
                fms_lanes16(&T[0][0], v.u0, v.l0);
                fms_lanes16(&T[1][0], v.u0, v.l1);
                fms_lanes16(&T[0][16], v.u1, v.l0);
                fms_lanes16(&T[1][16], v.u1, v.l1);
            };
            uint2 w1 = idx(1), w2 = idx(2), w3 = idx(3);
            Val v0 = get(idx(0));
            for (int k = 0; k < n; k += 2) {
                const Val v1 = get(w1);
                w1 = w3;
                w3 = idx(k + 5);
                step(v0);
                v0 = get(w2);
                w2 = idx(k + 4);
                step(v1);
            }
        }
    }

    // a[c] -= (lane KK's u[c]) * m for columns C0 .. CE - 1 (CE a multiple of 8); OWN: a and u are the same row block
    template <int KK, int C0, int CE, bool OWN>
    static __device__ __forceinline__ void eliminate(double *a, const double *u, double m)
    {
        constexpr int c1 = (C0 + 1) / 2 * 2, c2 = (C0 + 3) / 4 * 4, c3 = (C0 + 7) / 8 * 8, c4 = (C0 + 15) / 16 * 16;
        auto go = [&](auto C, auto CNT) {
            constexpr int c = decltype(C)::value, n = decltype(CNT)::value;
            if constexpr (OWN) fms_own<KK, n>(&a[c], m);
            else fms_from<KK, n>(&a[c], &u[c], m);
        };
        if constexpr (C0 < CE && C0 < c1) go(std::integral_constant<int, C0>{}, std::integral_constant<int, 1>{});
        if constexpr (c1 < CE && c1 < c2) go(std::integral_constant<int, c1>{}, std::integral_constant<int, 2>{});
        if constexpr (c2 < CE && c2 < c3) go(std::integral_constant<int, c2>{}, std::integral_constant<int, 4>{});
        if constexpr (c3 < CE && c3 < c4) go(std::integral_constant<int, c3>{}, std::integral_constant<int, 8>{});
        if constexpr (c4 < CE)
            static_for<(CE - c4 + 15) / 16>([&](auto B) {
                constexpr int c = c4 + 16 * decltype(B)::value;
                go(std::integral_constant<int, c>{}, std::integral_constant<int, (CE - c < 16 ? 8 : 16)>{});
            });
    }

    // The middle pivots (front positions m0 ..), right-looking, in registers:
    // their rows in the middle and tail columns, the tail's rows in the middle
    // columns, and the tail itself.  The factors go to the places the sweeps
    // read.  Sixteen nearly dense pivots cost 1,900 multiply-adds of one
    // instruction each here; formed entry by entry from local memory they took
    // four instructions per multiply-add, three times the time.
    __device__ __forceinline__ void middle(KParams &p, const uint4 (&first)[6])
    {
        if constexpr (FB > 0) {
            const int i = lane16();
            // 16 registers of a map to or from local memory
            auto load16 = [&](const uint4 *m, double *r) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint32_t a[4] = {m[q].x, m[q].y, m[q].z, m[q].w};
#pragma unroll
                    for (int x = 0; x < 8; ++x) r[8 * q + x] = field(a[x / 2], x % 2, base);
                }
            };
            auto store16 = [&](const uint4 *m, const double *r) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint32_t a[4] = {m[q].x, m[q].y, m[q].z, m[q].w};
#pragma unroll
                    for (int x = 0; x < 8; ++x) lds_at(field_addr(a[x / 2], x % 2, base)) = r[8 * q + x];
                }
            };
            auto map = [&](const uint16_t *t, int v) { return ld<uint4>(t, 256u * v, 16u * i); };
            uint4 mu[4], ms[6];  // maps, fetched a phase ahead
            // the middle columns: multipliers of the middle rows (M, its diagonal
            // 1 / U_kk) and of the tail rows (Lt)
            double M[16], Lt[2][16];
            load16(&first[0], M);
            load16(&first[2], Lt[0]);
            load16(&first[4], Lt[1]);
#pragma unroll
            for (int q = 0; q < 4; ++q) mu[q] = map(p.mid_load, 2 + q);
#pragma unroll
            for (int q = 0; q < 6; ++q) ms[q] = map(p.mid_store, q < 2 ? q : q + 4);
            static_for<16>([&](auto Q) {
                constexpr int K = decltype(Q)::value;
                const double inv = pivot_rcp(row_bcast<K>(M[K]));
                const double l = i > K ? M[K] * inv : 0.0;
                eliminate<K, K + 1, 16, true>(M, M, l);
                M[K] = i > K ? l : (i == K ? inv : M[K]);
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    Lt[b][K] *= inv;
                    eliminate<K, K + 1, 16, false>(Lt[b], M, Lt[b][K]);
                }
            });
            lds_handover();
            store16(&ms[0], M);
            store16(&ms[2], Lt[0]);
            store16(&ms[4], Lt[1]);
#pragma unroll
            for (int q = 0; q < 4; ++q) ms[q] = map(p.mid_store, 2 + q);
            lds_handover();
            // the tail columns, half of them at a time: the middle rows of U, then the tail
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                double U[16];
                load16(&mu[2 * h], U);
                static_for<16>([&](auto Q) {
                    constexpr int K = decltype(Q)::value;
                    const double l = i > K ? M[K] : 0.0;
                    fms_own<K, 16>(U, l);
                    eliminate<K, 0, 16, false>(&T[0][16 * h], U, Lt[0][K]);
                    eliminate<K, 0, 16, false>(&T[1][16 * h], U, Lt[1][K]);
                });
                lds_handover();
                store16(&ms[2 * h], U);
                lds_handover();
            }
        }
    }

    // The tail, right-looking, in registers: L below the diagonal, U above,
    // 1 / U_kk in dinv.
    __device__ __forceinline__ bool dense(KParams &p)
    {
        const int n = p.Mt, i = lane16();
#pragma unroll
        for (int t = 0; t < TB; ++t) dinv[t] = 1.0;
        static_for<NC / 4>([&](auto G) {
            constexpr int k0 = 4 * decltype(G)::value;
            if (!kFull && k0 >= n) return;
            static_for<4>([&](auto Q) {
                constexpr int K = k0 + decltype(Q)::value, rk = K / 16, kk = K % 16;
                if (!kFull && K >= n) return;
                const double inv = pivot_rcp(row_bcast<kk>(T[rk][K]));
                dinv[rk] = i == kk ? inv : dinv[rk];
                const double l = i > kk ? T[rk][K] * inv : 0.0;
                T[rk][K] = i > kk ? l : T[rk][K];
                eliminate<kk, K + 1, NC, true>(T[rk], T[rk], l);
                if constexpr (rk + 1 < TB) {
                    T[rk + 1][K] *= inv;
                    eliminate<kk, K + 1, NC, false>(T[rk + 1], T[rk], T[rk + 1][K]);
                }
            });
        });
        bool bad = false;
#pragma unroll
        for (int t = 0; t < TB; ++t) bad |= pivot_bad(dinv[t]);
        return bad;
    }

    // b <- (LU)^-1 b.  Columns in elimination order; a column's value is
    // broadcast within the row by the multiply-adds that use it.  The front's
    // entries are read four columns ahead of their use, their places (the sweep
    // maps) a half block of columns ahead.
    __device__ __forceinline__ void solve(double (&b)[NB])
    {
        KParams &p = params_here();
        const int i = lane16(), F = p.F;
        const uint32_t il = 16u * i;
        // entries of columns 4 z .. 4 z + 3 of a map vector of eight
        auto get4 = [&](const uint4 &w, int z, double *v, int stride) {
            const uint32_t a = z ? w.z : w.x, c = z ? w.w : w.y;
            v[0] = field(a, 0, base);
            v[stride] = field(a, 1, base);
            v[2 * stride] = field(c, 0, base);
            v[3 * stride] = field(c, 1, base);
        };
        double di[FB > 0 ? FB : 1];
        if constexpr (FB > 0) {
            constexpr int G = 4 * FB;  // groups of four columns
            uint4 map[2][NB];
            double v[2][4][NB];
            auto fetch = [&](auto H) {
                constexpr int h = decltype(H)::value, cb = h / 2, nw = NB - cb;
                constexpr int v0 = 2 * (cb * NB - cb * (cb - 1) / 2) + (h % 2) * nw;  // vectors of the half blocks before
#pragma unroll
                for (int w = 0; w < nw; ++w) map[h % 2][w] = ld<uint4>(p.fwd, 256u * (v0 + w), il);
            };
            auto read = [&](auto GG) {
                constexpr int g = decltype(GG)::value, nw = NB - g / 4;
#pragma unroll
                for (int w = 0; w < nw; ++w) get4(map[g / 2 % 2][w], g % 2, &v[g % 2][0][w], NB);
            };
            fetch(std::integral_constant<int, 0>{});
            uint32_t dw[FB];
#pragma unroll
            for (int f = 0; f < FB; ++f) dw[f] = ld<uint16_t>(p.dmap, 32u * f, 2u * i);
            fetch(std::integral_constant<int, 1>{});
            read(std::integral_constant<int, 0>{});
#pragma unroll
            for (int f = 0; f < FB; ++f) di[f] = field(dw[f], 0, base);
            static_for<G>([&](auto GG) {
                constexpr int g = decltype(GG)::value, cb = g / 4;
                if constexpr (g + 1 < G) read(std::integral_constant<int, g + 1>{});
                if constexpr (g % 2 == 1 && g / 2 + 2 < 2 * FB) fetch(std::integral_constant<int, g / 2 + 2>{});
                __builtin_amdgcn_sched_barrier(0);
                if (cb + 1 < FB || 4 * g < F)
                    static_for<4>([&](auto C) {
                        constexpr int c = decltype(C)::value;
                        fms_col_own<(g % 4) * 4 + c, NB - cb>(&b[cb], v[g % 2][c]);
                    });
            });
        }
        double *t = b + FB;
        uint4 mapt[2][FB > 0 ? FB : 1];
        auto fetch_t = [&](auto GI) {
            constexpr int gi = decltype(GI)::value;
#pragma unroll
            for (int w = 0; w < FB; ++w) mapt[gi % 2][w] = ld<uint4>(p.bwt, 256u * (gi * FB + w), il);
        };
        if constexpr (FB > 0) {
            fetch_t(std::integral_constant<int, 0>{});
            fetch_t(std::integral_constant<int, 1>{});
        }
        // tail, forward
        static_for<NC / 4>([&](auto G) {
            constexpr int k0 = 4 * decltype(G)::value;
            if (!kFull && k0 >= p.Mt) return;
            static_for<4>([&](auto Q) {
                constexpr int K = k0 + decltype(Q)::value, rk = K / 16, kk = K % 16, n = TB - rk;
                double m[TB];
                m[0] = i > kk ? T[rk][K] : 0.0;
                if constexpr (n > 1) m[1] = T[rk + 1][K];
                fms_col_own<kk, n>(&t[rk], m);
            });
        });
        uint4 mapf[2][FB > 0 ? FB : 1];  // of the last part: fetched ahead of this one
        auto fetch_f = [&](auto HH) {
            constexpr int h = 2 * FB - 1 - decltype(HH)::value, cb = h / 2;
            constexpr int v0 = FB * (FB + 1) - (cb + 1) * (cb + 2) + (h % 2 ? 0 : cb + 1);
#pragma unroll
            for (int w = 0; w <= cb; ++w) mapf[h % 2][w] = ld<uint4>(p.bwf, 256u * (v0 + w), il);
        };
        if constexpr (FB > 0) {
            fetch_f(std::integral_constant<int, 0>{});
            fetch_f(std::integral_constant<int, 1>{});
        }
        // tail columns, backward, on the front's rows too
        double vt[2][4][FB + TB];
        auto read_t = [&](auto GI) {  // groups of four columns, last first
            constexpr int g = decltype(GI)::value;
#pragma unroll
            for (int w = 0; w < FB; ++w) get4(mapt[g / 2 % 2][w], 1 - g % 2, &vt[g % 2][0][w], FB + TB);
        };
        read_t(std::integral_constant<int, 0>{});
        static_for<NC / 4>([&](auto GI) {
            constexpr int g = decltype(GI)::value, k0 = NC - 4 * (g + 1);
            if constexpr (g + 1 < NC / 4) read_t(std::integral_constant<int, g + 1>{});
            if constexpr (FB > 0 && g % 2 == 1 && g / 2 + 2 < NC / 8) fetch_t(std::integral_constant<int, g / 2 + 2>{});
            if constexpr (FB > 0) __builtin_amdgcn_sched_barrier(0);
            if (!kFull && k0 >= p.Mt) return;
            static_for<4>([&](auto CC) {
                constexpr int c = 3 - decltype(CC)::value, K = k0 + c, rk = K / 16, kk = K % 16;
                double *m = vt[g % 2][c];
                if constexpr (rk > 0) m[FB] = T[0][K];
                m[FB + rk] = i < kk ? T[rk][K] : 0.0;
                fms_col<kk, FB + rk + 1>(b, t[rk] * dinv[rk], m);
            });
        });
#pragma unroll
        for (int q = 0; q < TB; ++q) t[q] *= dinv[q];
        // front columns, backward
        if constexpr (FB > 0) {
            constexpr int G = 4 * FB;
            double v[2][4][FB];
            auto read = [&](auto GG) {
                constexpr int g = G - 1 - decltype(GG)::value;
#pragma unroll
                for (int w = 0; w <= g / 4; ++w) get4(mapf[g / 2 % 2][w], g % 2, &v[g % 2][0][w], FB);
            };
            read(std::integral_constant<int, 0>{});
            static_for<G>([&](auto GG) {
                constexpr int gg = decltype(GG)::value, g = G - 1 - gg, cb = g / 4;
                if constexpr (gg + 1 < G) read(std::integral_constant<int, gg + 1>{});
                if constexpr (gg % 2 == 1 && gg / 2 + 2 < 2 * FB) fetch_f(std::integral_constant<int, gg / 2 + 2>{});
                __builtin_amdgcn_sched_barrier(0);
                if (cb + 1 < FB || 4 * g < F)
                    static_for<4>([&](auto CC) {
                        constexpr int c = 3 - decltype(CC)::value;
                        fms_col<(g % 4) * 4 + c, cb + 1>(b, b[cb] * di[cb], v[g % 2][c]);
                    });
            });
#pragma unroll
            for (int f = 0; f < FB; ++f) b[f] *= di[f];
        }
    }
};

// D'_i = sum_j T_ij D_j for a change of spacing by rho (see rescale_entry in
// kernels_solve.hip), the identity beyond the order.
__device__ __forceinline__ double resample_entry(int e, int order, double rho)
{
    const int i = e / (kMaxOrder + 1), j = e % (kMaxOrder + 1);
    double acc = 0.0, u = 1.0;  // u = (-1)^l C(i, l)
#pragma unroll
    for (int l = 0; l <= kMaxOrder; ++l) {
        if (l > 0) u = rint(u * (l - 1 - i) * (1.0 / l));  // an integer of magnitude at most 10
        const double x = rho * l;
        double num = 1.0;
#pragma unroll
        for (int m = 1; m <= kMaxOrder; ++m) num = m <= j ? num * ((m - 1) - x) : num;
        acc = l <= order ? fma(num, u, acc) : acc;
    }
    int fact = 1;
#pragma unroll
    for (int m = 2; m <= kMaxOrder; ++m) fact = m <= j ? fact * m : fact;
    const double v = acc / fact;
    return i > order ? (i == j ? 1.0 : 0.0) : (j > order ? 0.0 : v);
}

__device__ __forceinline__ double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}

// The sum over a wavefront's four cells of a value that a row's lanes share.
__device__ __forceinline__ double cells_sum(double v)
{
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Multi-cells (MC): one system over all cells, so every wavefront has the same
// t, h, order and decisions, and only the norms and the failure flags cross
// wavefronts.  An exchange costs about as much as the rest of a Newton
// iteration, so one serves an iteration: the norm of the correction travels
// with the flags of that iteration's f and of the factorisation, and with the
// norms that the error test and the order selection would need if the
// iteration turned out to be the last.  20 species, per attempt, against one
// cell per wavefront with a grid barrier for every sum and flag: 343 -> 17 us
// with 500 cells, 1290 -> 26 us with 2,000.
struct NoExchange {
    __device__ __forceinline__ NoExchange(double *, int) {}
    __device__ __forceinline__ uint32_t sum(double (&)[4], uint32_t flags) { return flags; }
};

// State kept between the launches of the per-launch form, after the backward
// differences: see bdf_kernel; [16] and [17]: a re-sampling decided but not
// yet applied, and its factor.
template <int TB, int NC, int FB, int KU, bool MC, bool TAPE, int W>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(W, W))) void quad_kernel(QuadParams p)
{
    extern __shared__ double smem[];
    using Q = Quad<TB, NC, FB, KU>;
    constexpr int NB = Q::NB, KO = kMaxOrder;
    const int i = (int)threadIdx.x & 15;
    const int64_t slot = (int64_t)blockIdx.x * kQCells + (threadIdx.x >> 4);
    const bool has = slot < p.n_cells;
    const int64_t cell = has ? (p.order ? p.order[slot] : slot) : 0;
    const int K = p.opts.steps_per_launch;
    double *st_d = K > 0 ? p.state + cell * p.state_stride : nullptr;
    double *st_s = K > 0 ? st_d + (KO + 3) * NB * 16 : nullptr;
    bool live = has, resumed = false;
    if (K > 0 && has && st_s[0] == (double)p.call_id) {
        if (st_s[1] == 2.0) live = false;  // finished in an earlier launch of this outer step
        else resumed = true;
    }
    if (!MC && !__any(live)) return;
    Q C(p, smem);
    std::conditional_t<MC, GridExchange<4>, NoExchange> grid(p.mc_slots, (int)gridDim.x);
    const int N = p.N;
    const double n_inv = 1.0 / (MC ? (double)N * (double)p.n_cells : (double)N);
    auto ssq = [&](const double (&v)[NB], const double (&w)[NB]) -> double {
        double q = 0.0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const double x = v[b] * w[b];
            q += x * x;
        }
        return row_sum(q);
    };
    auto norm = [&](const double (&v)[NB], const double (&w)[NB]) -> double { return sqrt(ssq(v, w) * n_inv); };
    // Multi-cells: the wavefront's part of a sum, of a flag
    auto part = [&](const double (&v)[NB], const double (&w)[NB]) -> double { return cells_sum(has ? ssq(v, w) : 0.0); };
    auto flag = [&](bool x) -> uint32_t { return __any(has && x) ? 1u : 0u; };
    const mcc_solver_opts &o = p.opts;
    const double dt = p.dt;
    const int maxord = o.max_order;

    if (i == 0) {
        lds_at(C.base + 8 * kQZero) = 0.0;
        lds_at(C.base + 8 * kQTrash) = 0.0;
        lds_at(C.base + 8 * kQOne) = 1.0;
    }
#pragma unroll
    for (int u = 0; u < KU; ++u) {
        const int j = 16 * u + i;
        C.kr[u] = j < p.R && live ? p.k[(int64_t)j * p.ld + cell] : 0.0;
    }
    int sp[NB];
    // D[0..5] the backward differences; d1 the last Newton correction at this
    // order and spacing (the difference of order + 1)
    double D[KO + 1][NB], d1[NB], f[NB], w[NB], ypred[NB], psi[NB], d[NB], tmp[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        sp[b] = p.vsp[b * 16 + i];
#pragma unroll
        for (int j = 0; j < KO + 1; ++j) D[j][b] = resumed && live ? st_d[(j * NB + b) * 16 + i] : 0.0;
        d1[b] = resumed && live ? st_d[((KO + 1) * NB + b) * 16 + i] : 0.0;
        if (!resumed && live && sp[b] >= 0) D[0][b] = p.y[(int64_t)sp[b] * p.ld + cell];
    }
    auto nonfinite = [&](const double (&v)[NB]) {
        int x = 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) x |= !isfinite(v[b]);
        return x;
    };
    int steps = 0, rejects = 0, newton_fails = 0, newton_iters = 0, f_evals = 0, lu_count = 0;
    int status = MCC_CELL_OK, order = 1, n_equal = 0, attempts = 0, steps_here = 0;
    double h = 0.0, t = 0.0, h_uncut = 0.0, h_next = 0.0, pfac = 1.0;
    bool bad = false, pend = false, susp = false;
    double *tp = TAPE ? p.tape + cell * p.tape_stride : nullptr;
    int64_t tpos = TAPE && resumed ? (int64_t)st_s[15] : 0;
    auto record = [&](bool on, int type, int ord, double x, bool with_state) {
        if (!TAPE || !on || tpos < 0) return;
        if (tpos + kTapeScalars + (with_state ? N : 0) > p.tape_stride) {
            tpos = -1;
            return;
        }
        if (i == 0) tp[tpos] = type;
        tpos += 1;
        if (with_state) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if (sp[b] >= 0) tp[tpos + sp[b]] = D[0][b];
            tpos += N;
        }
        if (i == 0) {
            tp[tpos] = ord;
            tp[tpos + 1] = x;
            tp[tpos + 2] = type;
        }
        tpos += 3;
    };
    if (resumed) {
        t = st_s[2];
        h = st_s[3];
        order = (int)st_s[4];
        n_equal = (int)st_s[5];
        attempts = (int)st_s[6];
        steps = (int)st_s[7];
        rejects = (int)st_s[8];
        newton_fails = (int)st_s[9];
        newton_iters = (int)st_s[10];
        f_evals = (int)st_s[11];
        lu_count = (int)st_s[13];
        status = (int)st_s[14];
        pend = st_s[16] != 0.0;
        pfac = st_s[17];
    }
    const bool fresh = (live || MC) && !resumed;
    if (__any(fresh)) {
        const double h_warm = !MC && o.warm_start && fresh ? p.stats[cell].h_next : 0.0;
        C.deriv(D[0], f);
        bool nf = row_any((nonfinite(D[0]) | nonfinite(f)) != 0);
        double sys[4] = {0.0, 0.0, 0.0, 0.0};
        if constexpr (MC) {
#pragma unroll
            for (int b = 0; b < NB; ++b) w[b] = sp[b] >= 0 ? 1.0 / (o.rtol * fabs(D[0][b]) + o.atol) : 0.0;
            sys[0] = part(D[0], w);
            sys[1] = part(f, w);
            nf = grid.sum(sys, flag(nf)) != 0;
        }
        bool cold = false;
        if (fresh) {
            f_evals++;
            if (nf) {
                status = MCC_CELL_NONFINITE;
                order = 0;
                bad = true;
            } else if (h_warm > 0.0 && isfinite(h_warm)) {
                h = fmin(h_warm, dt);
            } else {
                cold = true;
            }
        }
        if (__any(cold)) {
#pragma unroll
            for (int b = 0; b < NB; ++b) w[b] = sp[b] >= 0 ? 1.0 / (o.rtol * fabs(D[0][b]) + o.atol) : 0.0;
            const double n0 = MC ? sqrt(sys[0] * n_inv) : norm(D[0], w), n1 = MC ? sqrt(sys[1] * n_inv) : norm(f, w);
            const double h0 = (n0 < 1e-5 || n1 < 1e-5) ? 1e-6 * dt : 0.01 * n0 / n1;
#pragma unroll
            for (int b = 0; b < NB; ++b) ypred[b] = D[0][b] + h0 * f[b];
            C.deriv(ypred, tmp);
#pragma unroll
            for (int b = 0; b < NB; ++b) tmp[b] -= f[b];
            if constexpr (MC) {
                sys[0] = part(tmp, w);
                grid.sum(sys, 0);
            }
            const double n2 = (MC ? sqrt(sys[0] * n_inv) : norm(tmp, w)) / h0;
            const double dm = n1 > n2 ? n1 : n2;
            const double h1 = dm <= 1e-15 ? fmax(1e-6, 1e-3 * h0) : sqrt(0.01 / dm);
            if (cold) {
                f_evals++;
                h = fmin(100.0 * h0, fmin(h1, dt));
                if (!(h > 0.0) || !isfinite(h)) {
                    status = MCC_CELL_NONFINITE;
                    order = 0;
                    h = 0.0;
                    bad = true;
                }
            }
        }
        if (fresh && !bad) {
#pragma unroll
            for (int b = 0; b < NB; ++b) D[1][b] = h * f[b];
        }
        record(fresh && !bad, 0, 0, h, false);
    }

    bool act = (live || MC) && !bad;
    while (__any(act)) {
        // re-samplings of the differences: the one decided by the last
        // attempt, then the one that cuts a step to land on dt
        bool landing = false;
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            bool need;
            double rho = 1.0;
            if (pass == 0) {
                need = act && pend;
                if (need) {
                    rho = pfac;
                    pend = false;
                }
            } else {
                if (act && attempts >= o.max_steps) {
                    status = MCC_CELL_TOO_MUCH_WORK;
                    act = false;
                }
                if (act) attempts++;
                need = act && h >= dt - t;
                if (need) {
                    h_uncut = h;
                    rho = (dt - t) / h;
                }
            }
            if (!__any(need)) continue;
            const uint32_t ta = C.base + 8u * (uint32_t)p.off_r;
            constexpr int M6 = KO + 1;
            lds_handover();
#pragma unroll 1
            for (int e = i; e < M6 * M6; e += 16) lds_at(ta + 8u * e) = resample_entry(e, order, rho);
            lds_handover();
            if (need) {
                double nd[M6][NB];
#pragma unroll
                for (int a = 0; a < M6; ++a) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) nd[a][b] = 0.0;
#pragma unroll
                    for (int j = 0; j < M6; ++j) {
                        const double x = lds_at(ta + 8u * (a * M6 + j));
#pragma unroll
                        for (int b = 0; b < NB; ++b) nd[a][b] += x * D[j][b];
                    }
                }
#pragma unroll
                for (int a = 0; a < M6; ++a)
#pragma unroll
                    for (int b = 0; b < NB; ++b) D[a][b] = nd[a][b];
            }
            lds_handover();
            record(need, 1, order, rho, false);
            if (pass == 1 && need) {
                h = dt - t;
                n_equal = 0;
                landing = true;
            }
        }
        if (!__any(act)) break;

        const double gk = bdf_gamma(order);
        const double igk = 1.0 / gk, c = h / gk;
        double on[KO + 1];  // 1 up to the order, 0 beyond: a select folded into the multiply-adds
#pragma unroll
        for (int j = 0; j <= KO; ++j) on[j] = j <= order ? 1.0 : 0.0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            double yp = 0.0, ps = 0.0;
#pragma unroll
            for (int j = 0; j <= KO; ++j) yp += on[j] * D[j][b];
#pragma unroll
            for (int j = 1; j <= KO; ++j) ps += (on[j] * bdf_gamma(j)) * D[j][b];
            ypred[b] = yp;
            psi[b] = ps * igk;
            // (the inverse of infinity would be NaN, by its Newton steps; 2^-1021 is zero once squared)
            w[b] = sp[b] >= 0 ? pivot_rcp(fmin(o.rtol * fabs(D[0][b]) + o.atol, 0x1p1021)) : 0.0;
            d[b] = 0.0;
        }
        if (act) lu_count++;
        bool singular = row_any(C.factor(ypred, c));
        bool conv = false, nact = act && !singular;
        double nrm_old = 0.0;
        double sys[4] = {0.0, 0.0, 0.0, 0.0};  // Multi-cells: squares of the correction, of d, D[order] and d - d1 with it
        if constexpr (MC) {
            const bool failed = singular;
            singular = false;
            nact = act;
#pragma unroll 1
            for (int it = 0; it < o.max_newton && __any(nact); ++it) {
#pragma unroll
                for (int b = 0; b < NB; ++b) tmp[b] = ypred[b] + d[b];
                C.deriv(tmp, f);
                const bool nf = row_any(nonfinite(f) != 0);
#pragma unroll
                for (int b = 0; b < NB; ++b) tmp[b] = c * f[b] - psi[b] - d[b];
                C.solve(tmp);
                sys[0] = part(tmp, w);
#pragma unroll
                for (int b = 0; b < NB; ++b) d[b] += tmp[b];
                sys[1] = part(d, w);
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    tmp[b] = d[b];
#pragma unroll
                    for (int j = 1; j <= KO; ++j) tmp[b] = fma(j == order ? 1.0 : 0.0, D[j][b], tmp[b]);
                }
                sys[2] = part(tmp, w);
#pragma unroll
                for (int b = 0; b < NB; ++b) tmp[b] = d[b] - d1[b];
                sys[3] = part(tmp, w);
                const uint32_t flags = grid.sum(sys, flag(failed) | 2 * flag(nf));
                if (it == 0 && (flags & 1)) {
                    singular = true;
                    break;
                }
                if (act) f_evals++;
                if (flags & 2) break;
                if (act) newton_iters++;
                const double nrm = sqrt(sys[0] * n_inv), rho = it >= 1 ? nrm / nrm_old : 0.0;
                if (!isfinite(nrm) || rho >= 1.0) break;
                if (nrm == 0.0 || (it >= 1 && rho / (1.0 - rho) * nrm < o.eta_newton)) {
                    conv = true;
                    break;
                }
                nrm_old = nrm;
            }
        }
#pragma unroll 1
        for (int it = 0; !MC && it < o.max_newton; ++it) {
            if (!__any(nact)) break;
#pragma unroll
            for (int b = 0; b < NB; ++b) tmp[b] = ypred[b] + d[b];
            C.deriv(tmp, f);
            if (nact) f_evals++;
            const bool nf = row_any(nonfinite(f) != 0);
            nact = nact && !nf;
#pragma unroll
            for (int b = 0; b < NB; ++b) tmp[b] = c * f[b] - psi[b] - d[b];
            C.solve(tmp);
            if (nact) newton_iters++;
            const double nrm = norm(tmp, w);
            nact = nact && isfinite(nrm);
            double rho = 0.0;
            if (it >= 1) {
                rho = nrm / nrm_old;
                nact = nact && !(rho >= 1.0);
            }
            if (nact) {
#pragma unroll
                for (int b = 0; b < NB; ++b) d[b] += tmp[b];
                if (nrm == 0.0 || (it >= 1 && rho / (1.0 - rho) * nrm < o.eta_newton)) {
                    conv = true;
                    nact = false;
                }
            }
            nrm_old = nrm;
        }
        double err = 0.0;
        if (__any(act && conv)) err = (MC ? sqrt(sys[1] * n_inv) : norm(d, w)) / (order + 1);
        const bool reject = act && conv && err > 1.0;
        const bool accept = act && conv && !reject;
        const bool fail = act && !conv;
        if (accept) {
            t = landing ? dt : t + h;
            if (t >= dt) h_next = landing ? h_uncut : h;
            steps++;
            steps_here++;
            n_equal++;
        }
        double d2[NB];  // the correction's change against the one before (the difference of order + 2)
        {
            // D_j += D_{j+1} from the order down, the new difference of order + 1
            // being d; the factors are 1 or 0 (an attempt that was not accepted)
            double m[KO + 1];
#pragma unroll
            for (int j = 0; j <= KO; ++j) m[j] = accept && j <= order ? 1.0 : 0.0;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                double sum = accept ? d[b] : 0.0;
#pragma unroll
                for (int j = KO; j >= 0; --j) {
                    const double old = D[j][b];
                    D[j][b] = fma(m[j], sum, old);
                    sum = fma(m[j], old, sum);
                }
                d2[b] = d[b] - d1[b];
                d1[b] = accept ? d[b] : d1[b];
            }
        }
        record(accept, 2, order, h / bdf_gamma(order), true);
        const bool select = accept && t < dt && n_equal >= order + 1;
        if (accept && t >= dt) act = false;
        double e_low = INFINITY, e_high = INFINITY;
        if (__any(select)) {
            double m[KO + 1];
#pragma unroll
            for (int j = 1; j <= KO; ++j) m[j] = j == order ? 1.0 : 0.0;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                tmp[b] = 0.0;
#pragma unroll
                for (int j = 1; j <= KO; ++j) tmp[b] = fma(m[j], D[j][b], tmp[b]);
            }
            const double el = (MC ? sqrt(sys[2] * n_inv) : norm(tmp, w)) / order;
            const double eh = (MC ? sqrt(sys[3] * n_inv) : norm(d2, w)) / (order + 2);
            if (order > 1) e_low = el;
            if (order < maxord) e_high = eh;
        }
        if (__any(select || reject)) {
            // the three powers on three lanes of the row: one call of the power function
            const int q = i == 1 ? order : (i == 2 ? order + 2 : order + 1);
            const double x = i == 1 ? e_low : (i == 2 ? e_high : err);
            const double r = quad_pow(select || reject ? x : 1.0, -1.0 / q);
            const double r_cur = row_bcast<0>(r);
            const double r1 = row_bcast<1>(r), r2 = row_bcast<2>(r);
            if (reject) {
                rejects++;
                pfac = fmax(o.safety * r_cur, o.fac_min);
            }
            if (select) {
                const double r_low = order > 1 ? r1 : 0.0, r_high = order < maxord ? r2 : 0.0;
                double best = r_cur;
                int new_order = order;
                if (r_low > best) { best = r_low; new_order = order - 1; }
                if (r_high > best) { best = r_high; new_order = order + 1; }
                pfac = o.safety * best;
                if (pfac > o.fac_max) pfac = o.fac_max;
                if (new_order > order)  // d1 becomes the highest difference
#pragma unroll
                    for (int j = 2; j <= KO; ++j)
#pragma unroll
                        for (int b = 0; b < NB; ++b) D[j][b] = j == new_order ? d1[b] : D[j][b];
                order = new_order;
            }
        }
        if (fail) {
            newton_fails++;
            pfac = o.fac_newton_fail;
        }
        if (reject || select || fail) {
            pend = true;
            h *= pfac;
            n_equal = 0;
            if ((reject || fail) && (h < o.h_min_rel * dt || t + h == t)) {
                status = reject ? MCC_CELL_ERR_FAIL : (singular ? MCC_CELL_SINGULAR : MCC_CELL_CONV_FAIL);
                act = false;
            }
        }
        if (K > 0 && act && accept && steps_here >= K) {  // per-launch form: the rest in a later launch
            susp = true;
            act = false;
        }
    }

    if (susp) {
#pragma unroll
        for (int j = 0; j < KO + 2; ++j)
#pragma unroll
            for (int b = 0; b < NB; ++b) st_d[(j * NB + b) * 16 + i] = j <= KO ? D[j < KO ? j : KO][b] : d1[b];
        if (i == 0) {
            st_s[0] = (double)p.call_id;
            st_s[1] = 1.0;
            st_s[2] = t;
            st_s[3] = h;
            st_s[4] = order;
            st_s[5] = n_equal;
            st_s[6] = attempts;
            st_s[7] = steps;
            st_s[8] = rejects;
            st_s[9] = newton_fails;
            st_s[10] = newton_iters;
            st_s[11] = f_evals;
            st_s[13] = lu_count;
            st_s[14] = status;
            if (TAPE) st_s[15] = (double)tpos;
            st_s[16] = pend ? 1.0 : 0.0;
            st_s[17] = pfac;
            atomicAdd(p.pending, 1);
        }
    }
    const bool done = live && !susp;
    double lm = INFINITY;
    bool nf = false;
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (done && status != MCC_CELL_NONFINITE && sp[b] >= 0) {
            p.y[(int64_t)sp[b] * p.ld + cell] = D[0][b];
            lm = fmin(lm, D[0][b]);
            nf |= !isfinite(D[0][b]);
        }
    lm = row_min(lm);
    nf = row_any(nf);
    if constexpr (MC) {
        double none[4] = {0.0, 0.0, 0.0, 0.0};
        nf = grid.sum(none, flag(nf)) != 0;
    }
    if (done && i == 0) {
        const double ymin = status == MCC_CELL_OK ? lm : 0.0;
        if (status == MCC_CELL_OK && nf) status = MCC_CELL_NONFINITE;
        p.status[cell] = status;
        if (TAPE) p.tape_len[cell] = tpos;
        if (p.stats) {
            mcc_cell_stats st;
            st.steps = steps;
            st.rejects = rejects;
            st.newton_fails = newton_fails;
            st.newton_iters = newton_iters;
            st.f_evals = f_evals;
            st.jac_evals = lu_count;
            st.lu_count = lu_count;
            st.order = order;
            st.h_last = h;
            st.y_min = ymin;
            st.h_next = status == MCC_CELL_OK ? h_next : h;
            p.stats[cell] = st;
        }
        if (K > 0) {
            st_s[0] = (double)p.call_id;
            st_s[1] = 2.0;
        }
    }
}

}  // namespace
}  // namespace mcc
