// Several information-only iterations of one tile in one launch (temporal
// blocking over a shrinking region).
#pragma once

#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include "iter_node.h"
#include "lattice.h"
#include "numerics.h"
#include "pair_tile.h"

#pragma clang fp contract(off)

namespace gabp {

// --------------------------------------------------------------------------
// S iterations of a tile.  A workgroup of NT threads holds a region of RW x RH
// nodes, NPT = RW RH / NT to a thread: the tile and a halo of R (S - 1) nodes
// around it (R: the stencil radius).  Iteration t+1 of every region node comes
// from memory (its incoming and previous outgoing messages, gains and data
// term are loaded once); the new messages go to LDS, sender-indexed, and stay
// with the gains in registers.  Each further iteration reads its incoming
// messages from LDS and is right on a region smaller by R on every side;
// iteration t+S is right on the tile and is written out.  Every node goes
// through theta_update, so the result is bitwise that of S single launches.
// Region position (lx, ly) is global (x0 + lx, y0 + ly), wrapped on periodic
// axes; positions outside a non-periodic axis hold zero messages.  IO: the
// caller guarantees that every region node and its neighbours lie inside the
// grid; the boundary code is compiled out.
//
// LDS: deg planes of (RH + R) rows of RW, R rows in front.  A read past a row's
// end lands in another row: only nodes outside the right region make one, and
// their values are used no more.
// --------------------------------------------------------------------------
template <int ALPHA, int RW, int RH>
struct DeepRegion {
    static constexpr int R = ALPHA == 1 ? 1 : 2, DEG = ALPHA == 1 ? 4 : 12;
    static constexpr int PL = (RH + R) * RW;                 // LDS plane
    static constexpr int kLds = DEG * PL + R * RW;
    static constexpr __host__ __device__ int halo(int S) { return R * (S - 1); }
    static constexpr __host__ __device__ int tw(int S) { return RW - 2 * halo(S); }
    static constexpr __host__ __device__ int th(int S) { return RH - 2 * halo(S); }
};

// --------------------------------------------------------------------------
// Region and iterations per launch for a lattice: the smallest region with at
// least `least` iterations per launch whose tiles all run at once (one to a
// CU; then as many iterations as that allows, at most `most`), else the type's
// last region with its `bulk` iterations.  A launch costs a few microseconds
// that do not depend on S, so small lattices want S large; past one tile per CU a
// larger halo is more tiles.  Microseconds per iteration, two per launch
// (best tile height) -> this rule:
//   FP32 13-point  64^2 5.3 -> 1.4, 256^2 5.9 -> 1.9, 512^2 7.0 -> 5.0,
//                  1024^2 20.4 -> 14.5, 2048^2 75.6 -> 57.8, 8192 x 4096 511 -> 448
//   FP32 5-point   64^2 2.6 -> 0.66, 512^2 2.9 -> 1.44, 1024^2 7.5 -> 3.6,
//                  2048^2 23.7 -> 11.9, 8192 x 4096 164 -> 96
//   FP64 5-point   64^2 2.8 -> 0.77, 512^2 4.1 -> 1.95, 1024^2 13.2 -> 6.9,
//                  2048^2 47.5 -> 24.2, 8192 x 4096 359 -> 195
//   FP64 13-point  64^2 6.5 -> 2.2, 512^2 12.5 -> 8.3, 1024^2 38.8 -> 31.4,
//                  2048^2 164 -> 122, 8192 x 4096 1149 -> 994
// --------------------------------------------------------------------------
struct DeepChoice {
    int rw, rh;                // region
    int least, most, bulk;     // iterations per launch, see above
};
constexpr DeepChoice kDeepF32A2[] = {{32, 32, 3, 7, 0}, {64, 32, 5, 5, 5}};
constexpr DeepChoice kDeepF32A1[] = {{32, 32, 8, 12, 0}, {64, 32, 6, 12, 0}, {64, 64, 8, 12, 8}};
constexpr DeepChoice kDeepF64A2[] = {{32, 32, 3, 6, 3}};
constexpr DeepChoice kDeepF64A1[] = {{32, 32, 6, 12, 0}, {64, 32, 6, 12, 6}};

struct DeepPlan {
    int region;   // index into the type's choices
    int S;        // iterations per launch
};

inline const DeepChoice *deep_choices(int dtype, int alpha, int &n) {
    if (dtype == 0) {
        n = alpha == 1 ? 3 : 2;
        return alpha == 1 ? kDeepF32A1 : kDeepF32A2;
    }
    n = alpha == 1 ? 2 : 1;
    return alpha == 1 ? kDeepF64A1 : kDeepF64A2;
}

inline int64_t deep_tiles(int alpha, int nx, int ny, int rw, int rh, int S) {
    const int h = 2 * (alpha == 1 ? 1 : 2) * (S - 1), tw = rw - h, th = rh - h;
    return (int64_t)((nx + tw - 1) / tw) * ((ny + th - 1) / th);
}

// Iterations before launch k of `launches` that share n iterations evenly.
inline int deep_part(int n, int launches, int k) { return (int)((int64_t)n * k / launches); }

inline DeepPlan deep_pick(const DeepChoice *c, int n, int alpha, int nx, int ny, int cus) {
    for (int k = 0; k < n; ++k)
        for (int S = c[k].most; S >= c[k].least; --S)
            if (deep_tiles(alpha, nx, ny, c[k].rw, c[k].rh, S) <= cus) return {k, S};
    return {n - 1, c[n - 1].bulk};
}

inline DeepPlan deep_plan(int dtype, int alpha, int nx, int ny, int cus) {
    int n;
    const DeepChoice *c = deep_choices(dtype, alpha, n);
    return deep_pick(c, n, alpha, nx, ny, cus);
}

// Record the earliest of a wave's invalid iterations (t + bad, bad != 0).
__device__ __forceinline__ void record_first(int bad, uint32_t t, uint32_t *diverged_at) {
    if (!__any(bad != 0)) return;
    int first = bad != 0 ? bad : INT_MAX;
    for (int k = 32; k >= 1; k >>= 1) first = min(first, __shfl_xor(first, k, 64));
    if ((threadIdx.x & 63u) == 0u) record_divergence(diverged_at, t + (uint32_t)first);
}

// n <= S iterations on the tiles for S.  Returns the first of them (1-based) in
// which this thread computed an invalid message of a node that the result
// depends on; 0: none.  `stop` (a divergence recorded by an earlier launch;
// uniform) is looked at only after the loads are on their way.
template <typename T, int ALPHA, int RW, int RH, int NT, bool IO>
__device__ __forceinline__ int deep_tile(const Lattice &L, const T *__restrict__ m_in,
                                         T *__restrict__ m_out, const T *__restrict__ gain,
                                         const T *__restrict__ bw, T eta, int S, int n, int tx,
                                         int ty, bool stop, T *lds) {
    using Rg = DeepRegion<ALPHA, RW, RH>;
    constexpr int DEG = Rg::DEG, R = Rg::R, PL = Rg::PL, NPT = RW * RH / NT, RPP = NT / RW;
    static_assert(NT % RW == 0 && RW * RH % NT == 0, "whole rows per pass over the region");
    const int x0 = tx * Rg::tw(S) - Rg::halo(S), y0 = ty * Rg::th(S) - Rg::halo(S);
    const int lx = (int)threadIdx.x % RW, ly0 = (int)threadIdx.x / RW;
    const T c = (T)L.c, keep = (T)1 - eta;
    T ot[NPT][DEG], g[NPT][DEG], b[NPT];
    bool here[NPT];
    int bad = 0;
    T *own = lds + R * RW + (int)threadIdx.x;
    // whether row ly is still computed in iteration s, and node (lx, ly) right
    auto live = [&](int ly, int s) { return ly >= R * (s - 1) && ly < RH - R * (s - 1); };
    auto right = [&](int ly, int s) {
        return live(ly, s) && lx >= R * (s - 1) && lx < RW - R * (s - 1);
    };
    // a thread's new messages: kept, and in LDS for the next iteration.  The
    // products with zero add up to zero exactly when every message is finite.  An
    // edge that does not exist adds an invalid value only where an infinite belief
    // makes the node's other messages invalid too, or there is no other: a grid of
    // one node has no messages, and nothing to report.
    const bool edges = IO || L.nx > 1 || L.ny > 1;
    auto finish = [&](int k, int s, const T *out) {
        const int ly = ly0 + k * RPP;
        T z = 0;
#pragma unroll
        for (int d = 0; d < DEG; ++d) {
            ot[k][d] = out[d];
            z = fmadd(out[d], (T)0, z);
        }
        if (!(z == (T)0) && edges && right(ly, s) && bad == 0) bad = s;
        if (s < n) {
#pragma unroll
            for (int d = 0; d < DEG; ++d) own[d * PL + k * NT] = out[d];
        }
    };
    {
        T tin[NPT][DEG];
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            int gx = x0 + lx, gy = y0 + ly0 + k * RPP;
            bool ok[DEG];
            here[k] = true;
            if (!IO) {
                if (gx < 0 || gx >= L.nx) {
                    if (L.bcx == BC_PERIODIC) gx = wrap_coord(gx, L.nx);
                    else here[k] = false;
                }
                if (gy < 0 || gy >= L.ny) {
                    if (L.bcy == BC_PERIODIC) gy = wrap_coord(gy, L.ny);
                    else here[k] = false;
                }
            }
            if (here[k]) {
                theta_gather<T, ALPHA, IO>(L, m_in, gain, bw, gx, gy, tin[k], ot[k], g[k], b[k], ok);
            } else {
                b[k] = 0;
#pragma unroll
                for (int d = 0; d < DEG; ++d) tin[k][d] = ot[k][d] = g[k][d] = 0;
            }
        }
        __builtin_amdgcn_s_setprio(0);
        if (stop) return 0;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            T out[DEG];
            theta_update<T, DEG>(tin[k], ot[k], g[k], b[k], c, eta, keep, out);
            finish(k, 1, out);
        }
    }
#pragma unroll 1
    for (int s = 2; s <= n; ++s) {
        __syncthreads();
        T tin[NPT][DEG];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if (!live(ly0 + k * RPP, s)) continue;
#pragma unroll
            for (int d = 0; d < DEG; ++d)
                tin[k][d] = own[(d ^ 1) * PL + k * NT + dir_dy(d) * RW + dir_dx(d)];
        }
        if (s < n) __syncthreads();
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if (!live(ly0 + k * RPP, s)) continue;
            T out[DEG];
            theta_update<T, DEG>(tin[k], ot[k], g[k], b[k], c, eta, keep, out);
            if (!IO && !here[k]) {
#pragma unroll
                for (int d = 0; d < DEG; ++d) out[d] = 0;
            }
            finish(k, s, out);
        }
    }
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int ly = ly0 + k * RPP, x = x0 + lx, y = y0 + ly;
        if (!right(ly, S) || x >= L.nx || y >= L.ny) continue;
        const uint32_t i = (uint32_t)(y * L.pitch + x);
#pragma unroll
        for (int d = 0; d < DEG; ++d) {
            int xn, yn;
            if (IO || neighbour(L, x, y, d, xn, yn))
                __builtin_nontemporal_store(ot[k][d], &(m_out + (size_t)(DEG + d) * L.plane)[i]);
        }
    }
    return bad;
}

}  // namespace gabp
