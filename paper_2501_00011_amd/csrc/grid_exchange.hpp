// Multi-cells: sums over every wavefront of a cooperative launch (one
// wavefront per workgroup, all resident).
//
// A grid barrier takes 5 us for a few wavefronts and 50 to 200 us for 500 to
// 2,000, and a solve needs thousands of sums, so the sums carry their own synchronisation: a wavefront publishes each
// value in two 64-bit words of its own slot, one half of the double in the
// high 32 bits beside the number of the exchange (and flags) in the low ones.
// A word is written and read whole, so a reader that finds the number it
// waits for has the value, with no fence and no second round trip.  Everyone
// reads all slots and adds them in one fixed order: every wavefront obtains
// the same bits and takes the same decisions.  Two slot arrays alternate: a
// wavefront publishes exchange r + 2 only after it has read r + 1 of
// everyone, hence after everyone has read r.  Slots are accessed with
// device-scope atomics, coherent across the XCDs' separate L2 caches.
//
// Measured, per step attempt, grid barriers against this: 72 species (eight or
// so sums an attempt) 79 -> 53 us with 64 cells and 703 -> 77 us with 1,000.
#pragma once

#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>

#include "mcc_internal.hpp"

namespace mcc {

template <int V>  // values per exchange (1, 2 or 4)
struct GridExchange {
    static constexpr int kWords = 2 * V, kPer = kWave / V, kFlight = 4;
    unsigned long long *slots;  // [2][n][kWords]
    int n;
    uint32_t round = 0;
    bool lost = false;

    // Slots may hold the numbers of an earlier launch (a replayed graph repeats
    // them): clear the own ones before anyone publishes.
    __device__ __forceinline__ GridExchange(double *mem, int waves) : slots((unsigned long long *)mem), n(waves)
    {
        const int l = (int)threadIdx.x;
        if (l < 2 * kWords)
            __hip_atomic_store(&slots[((size_t)(l / kWords) * n + blockIdx.x) * kWords + l % kWords], 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        cooperative_groups::this_grid().sync();
    }

    // v (the same on the wavefront's lanes) becomes the sums over all
    // wavefronts; returns the union of their flags (two bits).  A wait is
    // bounded (some seconds, only ever reached if another launch writes the
    // same slots): then, and from then on, the sums are NaN and every flag set.
    __device__ __forceinline__ uint32_t sum(double (&v)[V], uint32_t flags)
    {
        const int l = (int)threadIdx.x, q = l % V;
        ++round;
        unsigned long long *b = slots + (size_t)(round & 1) * n * kWords;
        const uint32_t tag = round << 2;
        if (l < kWords) {
            unsigned long long x = 0;
#pragma unroll
            for (int a = 0; a < V; ++a) {
                const unsigned long long y = (unsigned long long)__double_as_longlong(v[a]);
                if (l / 2 == a) x = l & 1 ? y << 32 : y & 0xffffffff00000000ull;
            }
            __hip_atomic_store(&b[(size_t)blockIdx.x * kWords + l], x | tag | flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        double acc = 0.0;
        uint32_t seen = 0;
        for (int s0 = 0; s0 < n && !lost; s0 += kFlight * kPer) {
            unsigned long long hi[kFlight], lo[kFlight];
            bool ok;
            int spins = 0;
            do {
                ok = true;
#pragma unroll
                for (int u = 0; u < kFlight; ++u) {
                    const int s = s0 + u * kPer + l / V;
                    hi[u] = lo[u] = tag;
                    if (s < n) {
                        hi[u] = __hip_atomic_load(&b[(size_t)s * kWords + 2 * q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        lo[u] = __hip_atomic_load(&b[(size_t)s * kWords + 2 * q + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
#pragma unroll
                for (int u = 0; u < kFlight; ++u)
                    ok = ok && ((uint32_t)hi[u] & ~3u) == tag && ((uint32_t)lo[u] & ~3u) == tag;
                lost = ++spins > (1 << 21);
            } while (!__all(ok) && !lost);
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {  // beyond the last slot: zero
                acc += __longlong_as_double((long long)((hi[u] & 0xffffffff00000000ull) | (lo[u] >> 32)));
                seen |= (uint32_t)hi[u] & 3u;
            }
        }
#pragma unroll
        for (int m = V; m < kWave; m *= 2) acc += __shfl_xor(acc, m);
#pragma unroll
        for (int a = 0; a < V; ++a) v[a] = lost ? NAN : __shfl(acc, a);
        return lost ? 3u : (__any(seen & 1u) ? 1u : 0u) | (__any(seen & 2u) ? 2u : 0u);
    }
};

}  // namespace mcc
