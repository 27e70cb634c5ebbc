// Change of the precision messages between two buffers (the freeze test),
// shared by the lattice, batched and space-time solvers.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace gabp {

// Relative change |a - b| / max(|a|, |b|) of two elements whose bits differ;
// +inf for a non-finite element.
struct LatticeRel {
    __device__ __forceinline__ static float of(double a, double b) {
        const double d = fabs(a - b), m = fmax(fabs(a), fabs(b));
        return !isfinite(d) || !isfinite(m) ? INFINITY : d == 0.0 ? 0.0f : (float)(d / m);
    }
};

// --------------------------------------------------------------------------
// One wave's share of the test over n elements (a multiple of 16 / sizeof(T),
// 16-byte aligned): the wave-th of `waves` waves.  *count grows by the number of
// elements whose bits differ (64-bit: n may exceed 2^32), *maxrel becomes the
// largest of their relative changes, as the bits of a non-negative float, so
// that unsigned comparison orders them; both are independent of the order of
// the atomics.  The precision messages freeze only if at most `limit` elements
// changed, so once a wave knows of more - its own, or *count, which the others
// add to - it stops reading: then *count is some number above `limit` and
// *maxrel says nothing.  Before the messages settle a test so takes the time of
// its first loads (4 us at any size; with every element read, a division per
// changed one and an atomic per wave it took 136 us on 261 x 187 nodes and 814
// on 8192 x 4096); once they have, every element is read once, at the copy rate.
// --------------------------------------------------------------------------
template <typename T, typename Rel>
__device__ __forceinline__ void prec_change_wave(const T *__restrict__ a, const T *__restrict__ b,
                                                 int64_t n, int wave, int waves, uint64_t limit,
                                                 unsigned long long *__restrict__ count,
                                                 uint32_t *__restrict__ maxrel) {
    constexpr int V = 16 / (int)sizeof(T), U = 2;
    struct alignas(16) Vec {
        T v[V];
    };
    const Vec *av = (const Vec *)a, *bv = (const Vec *)b;
    const int64_t nv = n / V, stride = (int64_t)waves * 64 * U;
    const int lane = (int)(threadIdx.x & 63u);
    uint64_t mine = 0;      // of this wave
    float mr = 0.0f;
    for (int64_t k = (int64_t)wave * 64 * U + lane; k - lane < nv; k += stride) {
        const uint64_t known = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__any(known > limit)) return;      // uniform
        Vec x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = k + 64 * u < nv ? k + 64 * u : 0;
            x[u] = av[q];
            y[u] = bv[q];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) {
                bool diff;
                if constexpr (sizeof(T) == 4)
                    diff = __float_as_uint(x[u].v[v]) != __float_as_uint(y[u].v[v]);
                else
                    diff = __double_as_longlong(x[u].v[v]) != __double_as_longlong(y[u].v[v]);
                diff = diff && k + 64 * u < nv;
                const uint64_t who = __ballot(diff);
                mine += (uint64_t)__popcll(who);
                if (who != 0 && mine <= limit && diff)
                    mr = fmaxf(mr, Rel::of((double)x[u].v[v], (double)y[u].v[v]));
            }
        if (mine > limit) break;
    }
    if (mine == 0) return;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mr = fmaxf(mr, __shfl_xor(mr, o, 64));
    if (lane == 0) {
        atomicAdd(count, (unsigned long long)mine);
        atomicMax(maxrel, __float_as_uint(mr));
    }
}

// Blocks of 256 threads for a test over n elements of the given size.
inline int prec_change_blocks(int64_t n, int esize) {
    const int64_t want = (n + 2048 * 4 / esize - 1) / (2048 * 4 / esize);
    return (int)(want < 1024 ? (want > 0 ? want : 1) : 1024);
}

}  // namespace gabp
