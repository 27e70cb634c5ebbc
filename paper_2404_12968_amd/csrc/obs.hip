// Folding point observations into node terms (Section "Including
// Observations"): every observation k of cell c contributes w_k = 1/s_k^2 to
// the node precision p_c and w_k y_k to the node information h_c; several
// observations of one cell multiply their likelihoods, so their terms add.
//
// Deterministic: the thread that owns the first observation of a run of one cell
// sums the run in input order, starting from 0.  The node terms therefore do not
// depend on thread timing (floating-point atomics would), and equal a sequential
// sum in input order.  Shared by the lattice, batched and space-time set-up paths.
//
// The observations are first folded as they come, in one launch: right wherever
// all observations of a cell follow one another, in whatever order the cells are.
// A run that meets a cell already taken raises a flag, which the caller looks at
// when it next waits; only then are the observations brought into their cells'
// order by a stable radix sort over the bits that a cell number has, and folded
// anew.  Set-up without a sort and with one before every fold: 64^2 with 5 %
// observed 64 and 94 us, 2048^2 283 and 440, a batch of 24 0.37 and 1.4 ms.
// Cells repeated out of order (10 %) take both passes.  The first does little then:
// its workgroups, and the node terms after it, end once the flag is up.  The sort
// takes its memory from planes that only checks write, and takes the fewer bits; what
// is left is one wait more: 64^2 93 us (94 with the sort first), 256^2 162 (142),
// 1024^2 238 (219), 2048^2 498 (500), a batch of 24 on the device 1.15 ms (1.74).
// Allocating costs more: 1 us up to some hundred KB, 100 us with its release from 2 MB.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <hipcub/hipcub.hpp>

#include "internal.h"

#pragma clang fp contract(off)

namespace gabp {

namespace {

// Positions before the sort, and the observed cells' terms back to zero after a
// pass that found repeated ones.
__global__ __launch_bounds__(256) void k_obs_index(int64_t n, const int64_t *__restrict__ cell,
                                                   int64_t ncells, int32_t nx, int32_t pitch,
                                                   int32_t *__restrict__ idx,
                                                   double *__restrict__ p_plane,
                                                   double *__restrict__ h_plane) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    idx[k] = (int32_t)k;
    const int64_t c = cell[k];
    if (c < 0 || c >= ncells) return;
    const int64_t i = (c / nx) * (int64_t)pitch + c % nx;
    p_plane[i] = 0.0;
    h_plane[i] = 0.0;
}

// Thread per position s; the first of each run of equal cells sums the run.  With
// idx_s the cells are sorted and position s is observation idx_s[s]; without, s
// itself, and `repeated` is raised when a run's cell was taken by another run
// (its precision is no longer 0; a precision is positive), which makes the
// planes worthless.
// Cell c maps to the pitched index (c / nx) * pitch + c % nx, which
// serves both the lattice (row y) and the space-time grid (row n * ny + y,
// slices pitch * ny apart).
__global__ __launch_bounds__(256) void k_obs_fold(int64_t n, const int64_t *__restrict__ cell_s,
                                                  const int32_t *__restrict__ idx_s,
                                                  const double *__restrict__ yv,
                                                  const double *__restrict__ var, double sigma2,
                                                  int64_t ncells, int32_t nx, int32_t pitch,
                                                  double *__restrict__ p_plane,
                                                  double *__restrict__ h_plane,
                                                  uint32_t *__restrict__ err_flag,
                                                  uint32_t *__restrict__ repeated) {
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    // nothing that follows is used once it is raised
    if (repeated &&
        __hip_atomic_load(repeated, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)
        return;
    const int64_t c = cell_s[s];
    if (s > 0 && cell_s[s - 1] == c) return;
    if (c < 0 || c >= ncells) {
        *err_flag = 1u;
        return;
    }
    double p = 0.0, h = 0.0;
    for (int64_t r = s; r < n && cell_s[r] == c; ++r) {
        const int64_t k = idx_s ? (int64_t)idx_s[r] : r;
        const double s2 = var ? var[k] : sigma2;
        const double y = yv[k];
        if (!(s2 > 0.0) || !isfinite(s2) || !isfinite(y)) {
            *err_flag = 1u;
            return;
        }
        const double w = 1.0 / s2;
        p += w;
        h += w * y;
    }
    const int64_t i = (c / nx) * (int64_t)pitch + c % nx;
    const unsigned long long free_cell = 0;
    if (atomicCAS((unsigned long long *)&p_plane[i], free_cell,
                  (unsigned long long)__double_as_longlong(p)) != free_cell) {
        if (repeated) *repeated = 1u;
        return;
    }
    h_plane[i] = h;
}

}  // namespace

hipError_t launch_obs_fold(int64_t n, const int64_t *cell, const double *y, const double *var,
                           double sigma2, int64_t ncells, int32_t nx, int32_t pitch,
                           double *p_plane, double *h_plane, uint32_t *err_flag,
                           uint32_t *repeated, void *room, size_t room_bytes, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (n > INT32_MAX) return hipErrorInvalidValue;
    const unsigned nb = (unsigned)((n + 255) / 256);
    if (repeated) {
        hipLaunchKernelGGL(k_obs_fold, dim3(nb), dim3(256), 0, s, n, cell,
                           (const int32_t *)nullptr, y, var, sigma2, ncells, nx, pitch, p_plane,
                           h_plane, err_flag, repeated);
        return hipGetLastError();
    }
    // sorted cells, positions before and after, the sort's own
    int64_t *cell_s = nullptr;
    int32_t *idx = nullptr, *idx_s = nullptr;
    size_t tmp_bytes = 0;
    int bits = 1;                   // of a cell inside the grid; others are refused
    while (bits < 63 && (ncells - 1) >> bits != 0) ++bits;
    hipError_t e = hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_bytes, cell, cell_s, idx,
                                                      idx_s, (int)n, 0, bits, s);
    const size_t cells_b = ((size_t)n * sizeof(int64_t) + 255) / 256 * 256;
    const size_t idx_b = ((size_t)n * sizeof(int32_t) + 255) / 256 * 256;
    const size_t bytes = cells_b + 2 * idx_b + tmp_bytes + 256;
    const bool own = bytes > room_bytes;
    char *mem = (char *)room;
    if (e == hipSuccess && own) {
        mem = nullptr;
        e = hipMalloc((void **)&mem, bytes);
    }
    void *tmp = nullptr;
    if (e == hipSuccess) {
        cell_s = (int64_t *)mem;
        idx = (int32_t *)(mem + cells_b);
        idx_s = (int32_t *)(mem + cells_b + idx_b);
        tmp = mem + cells_b + 2 * idx_b;
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_obs_index, dim3(nb), dim3(256), 0, s, n, cell, ncells, nx, pitch, idx,
                           p_plane, h_plane);
        e = hipGetLastError();
    }
    if (e == hipSuccess)
        e = hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, cell, cell_s, idx, idx_s, (int)n,
                                               0, bits, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_obs_fold, dim3(nb), dim3(256), 0, s, n, (const int64_t *)cell_s,
                           (const int32_t *)idx_s, y, var, sigma2, ncells, nx, pitch, p_plane,
                           h_plane, err_flag, (uint32_t *)nullptr);
        e = hipGetLastError();
    }
    if (!own) {
        if (e == hipSuccess) e = hipMemsetAsync(room, 0, bytes, s);
        return e;
    }
    const hipError_t es = hipStreamSynchronize(s);
    if (e == hipSuccess) e = es;
    (void)hipFree(mem);
    return e;
}

}  // namespace gabp
