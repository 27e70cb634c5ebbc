// Several full iterations (precision and information messages) of one tile in
// one launch: the temporal blocking of deep_tile.h for the phase before the
// precision messages freeze.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "deep_tile.h"
#include "iter_node.h"
#include "lattice.h"
#include "numerics.h"

#pragma clang fp contract(off)

namespace gabp {

// --------------------------------------------------------------------------
// S full iterations of a tile, on the region and with the node order of
// deep_tile.  A thread keeps its nodes' outgoing messages and diagonal in
// registers; new messages go to LDS.  Every node runs iter_node's arithmetic in
// iter_node's order, so the result is bitwise that of S single launches.
//
// SPLIT: precision and information messages take turns in one set of deg LDS
// planes (four barriers an iteration instead of two): two sets of FP64
// 13-point planes of a 32 x 32 region do not fit.
// --------------------------------------------------------------------------
template <int ALPHA, int RW, int RH, bool SPLIT>
constexpr int deep_full_lds() {
    using Rg = DeepRegion<ALPHA, RW, RH>;
    return (SPLIT ? 1 : 2) * Rg::DEG * Rg::PL + Rg::R * RW;
}

// --------------------------------------------------------------------------
// Region and iterations per launch, by the rule of deep_tile.h on the regions
// below.  A single full iteration is bound by memory on large lattices (200
// bytes a node in FP32 with 13 points) and by its launch and its chain of loads
// on small ones; S of them read and write the messages once.  Past one tile per
// CU, one node to a thread in a 64-wide region was the fastest in FP32 (its rows
// are whole lines); two to a thread need too many registers with 13 points.
// Microseconds per iteration, single launches -> this rule (Neumann, launches
// back to back):
//   FP32 13-point  64^2 5.4 -> 2.7, 256^2 6.2 -> 3.1, 512^2 13.3 -> 9.9,
//                  1024^2 46 -> 32, 2048^2 174 -> 123, 8192 x 4096 1279 -> 968
//   FP32 5-point   64^2 3.4 -> 0.95, 256^2 3.7 -> 1.2, 512^2 5.3 -> 2.7,
//                  1024^2 20 -> 7.6, 2048^2 59 -> 27, 8192 x 4096 420 -> 185
//   FP64 13-point  64^2 6.6 -> 3.9, 256^2 7.8 -> 5.9, 512^2 26 -> 21,
//                  1024^2 84 -> 74, 2048^2 336 -> 284
//   FP64 5-point   64^2 3.7 -> 1.3, 256^2 4.2 -> 1.8, 512^2 8.9 -> 3.8,
//                  1024^2 33 -> 14, 2048^2 118 -> 49
// The 24 x 24 region is for FP64 with 5 points up to 128^2, where one tile per CU
// leaves an iteration to the CU's FP64 rate and barriers: 9 waves to a workgroup
// instead of 16.  Against the 32 x 32 one, calls of 10, 50 and 200 iterations: 24^2 1.50,
// 1.35, 1.28 (1.81, 1.56, 1.42), 64^2 1.50, 1.37, 1.30 (1.86, 1.60, 1.44), 90 x 61 1.51,
// 1.40, 1.30 (1.88, 1.62, 1.46), 128^2 1.55, 1.40, 1.32 (1.83, 1.61, 1.47).  Nine
// iterations at most keep one tile per CU up to that size; eight of them (136^2) take
// 2.03 in calls of 10 and 1.39 in calls of 200, against 1.94 and 1.48.
// --------------------------------------------------------------------------
constexpr DeepChoice kFullF32A2[] = {{32, 32, 3, 5, 0}, {64, 16, 3, 3, 3}};
constexpr DeepChoice kFullF32A1[] = {{32, 32, 6, 12, 0}, {64, 16, 5, 5, 5}};
constexpr DeepChoice kFullF64A2[] = {{32, 16, 2, 3, 0}, {32, 24, 3, 3, 3}};
constexpr DeepChoice kFullF64A1[] = {{24, 24, 9, 9, 0}, {32, 32, 6, 12, 0}, {64, 32, 6, 6, 6}};

inline const DeepChoice *full_choices(int dtype, int alpha, int &n) {
    if (dtype == 0) {
        n = 2;
        return alpha == 1 ? kFullF32A1 : kFullF32A2;
    }
    n = alpha == 1 ? 3 : 2;
    return alpha == 1 ? kFullF64A1 : kFullF64A2;
}

inline DeepPlan deep_full_plan(int dtype, int alpha, int nx, int ny, int cus) {
    int n;
    const DeepChoice *c = full_choices(dtype, alpha, n);
    return deep_pick(c, n, alpha, nx, ny, cus);
}

// n <= S iterations on the tiles for S.  Returns the first of them (1-based) in
// which this thread computed an invalid message of a node that the result
// depends on (a cavity precision that is not positive or a message that is not
// finite); 0: none.
template <typename T, int ALPHA, int RW, int RH, int NT, bool SPLIT, bool IO>
__device__ __forceinline__ int deep_full_tile(const Lattice &L, const T *__restrict__ m_in,
                                              T *__restrict__ m_out, const T *__restrict__ adiag,
                                              const T *__restrict__ bw, T eta, int S, int n,
                                              int tx, int ty, bool stop, T *lds) {
    using Rg = DeepRegion<ALPHA, RW, RH>;
    constexpr int DEG = Rg::DEG, R = Rg::R, PL = Rg::PL, NPT = RW * RH / NT, RPP = NT / RW;
    constexpr int NQ = ALPHA == 2 && !IO ? 4 : 1;   // couplings that depend on the node
    static_assert(NT % RW == 0 && RW * RH % NT == 0, "whole rows per pass over the region");
    const int x0 = tx * Rg::tw(S) - Rg::halo(S), y0 = ty * Rg::th(S) - Rg::halo(S);
    const int lx = (int)threadIdx.x % RW, ly0 = (int)threadIdx.x / RW;
    const T c = (T)L.c, keep = (T)1 - eta;
    T ol[NPT][DEG], ot[NPT][DEG], a[NPT], b[NPT], qn[NPT][NQ];
    uint32_t okm[NPT];
    int bad = 0;
    T *own = lds + R * RW + (int)threadIdx.x;
    constexpr int INFO = SPLIT ? 0 : DEG * PL;
    // whether row ly is still computed in iteration s, and node (lx, ly) right
    auto live = [&](int ly, int s) { return ly >= R * (s - 1) && ly < RH - R * (s - 1); };
    auto right = [&](int ly, int s) {
        return live(ly, s) && lx >= R * (s - 1) && lx < RW - R * (s - 1);
    };
    auto has = [&](int k, int d) { return IO || (okm[k] >> d & 1u) != 0u; };
    // nodes with every neighbour two cells inside the grid: l_i is the same
    const T inner = (T)L.kappa2 + (T)2 * (T)L.ihx2 + (T)2 * (T)L.ihy2;
    auto coupling = [&](int k, int d) {
        if (NQ == 4 && d < 4) return qn[k][d];
        return q_over_c_ell<T, ALPHA>(L, d, inner, inner);
    };
    // precision half: gains of the node's edges, and its new precision messages
    auto precision = [&](int k, const T *lin, T *g, bool &wrong) {
        T sl = 0, z = 0;
#pragma unroll
        for (int d = 0; d < DEG; ++d) sl += lin[d];
        const T bl = fmadd(c, sl, a[k]);
#pragma unroll
        for (int d = 0; d < DEG; ++d) {
            const T q = coupling(k, d), lc = bl - lin[d];
            g[d] = edge_gain(q, lc);
            const T dl = fmadd(eta, g[d] * q, keep * ol[k][d]);
            wrong |= has(k, d) && !(lc > (T)0);
            ol[k][d] = has(k, d) ? dl : (T)0;
            z = fmadd(ol[k][d], (T)0, z);   // zero exactly when every message is finite
        }
        wrong |= !(z == (T)0);
    };
    auto information = [&](int k, const T *tin, const T *g, bool &wrong) {
        T st = 0, z = 0;
#pragma unroll
        for (int d = 0; d < DEG; ++d) st += tin[d];
        const T bt = fmadd(c, st, b[k]);
#pragma unroll
        for (int d = 0; d < DEG; ++d) {
            const T tc = bt - tin[d];
            const T dt = fmadd(eta, g[d] * tc, keep * ot[k][d]);
            ot[k][d] = has(k, d) ? dt : (T)0;
            z = fmadd(ot[k][d], (T)0, z);
        }
        wrong |= !(z == (T)0);
    };
    auto put = [&](int k, const T *m, int base) {
#pragma unroll
        for (int d = 0; d < DEG; ++d) own[base + d * PL + k * NT] = m[d];
    };
    auto get = [&](int k, T *m, int base) {
#pragma unroll
        for (int d = 0; d < DEG; ++d)
            m[d] = own[base + (d ^ 1) * PL + k * NT + dir_dy(d) * RW + dir_dx(d)];
    };
    {
        T lin[NPT][DEG], tin[NPT][DEG];
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            int gx = x0 + lx, gy = y0 + ly0 + k * RPP;
            bool here = true;
            if (!IO) {
                if (gx < 0 || gx >= L.nx) {
                    if (L.bcx == BC_PERIODIC) gx = wrap_coord(gx, L.nx);
                    else here = false;
                }
                if (gy < 0 || gy >= L.ny) {
                    if (L.bcy == BC_PERIODIC) gy = wrap_coord(gy, L.ny);
                    else here = false;
                }
            }
            okm[k] = 0;
            if (here) {
                const uint32_t i = (uint32_t)(gy * L.pitch + gx);
                uint32_t j[DEG];
                int xs[DEG], ys[DEG];
                bool ok[DEG];
                node_nbrs<DEG, IO>(L, gx, gy, j, xs, ys, ok);
#pragma unroll
                for (int d = 0; d < DEG; ++d) lin[k][d] = (m_in + (size_t)(d ^ 1) * L.plane)[j[d]];
#pragma unroll
                for (int d = 0; d < DEG; ++d) ol[k][d] = (m_in + (size_t)d * L.plane)[i];
#pragma unroll
                for (int d = 0; d < DEG; ++d)
                    tin[k][d] = (m_in + (size_t)(DEG + (d ^ 1)) * L.plane)[j[d]];
#pragma unroll
                for (int d = 0; d < DEG; ++d) ot[k][d] = (m_in + (size_t)(DEG + d) * L.plane)[i];
                a[k] = adiag[i];
                b[k] = bw[i];
                if (!IO) {
                    const T li = NQ == 4 ? ell<T>(L, gx, gy) : (T)0;
#pragma unroll
                    for (int d = 0; d < DEG; ++d) {
                        lin[k][d] = ok[d] ? lin[k][d] : (T)0;
                        tin[k][d] = ok[d] ? tin[k][d] : (T)0;
                        okm[k] |= (ok[d] ? 1u : 0u) << d;
                        if (NQ == 4 && d < 4) qn[k][d] = q_over_c<T, ALPHA>(L, d, li, xs[d], ys[d]);
                    }
                }
            } else {
                a[k] = b[k] = 0;
#pragma unroll
                for (int d = 0; d < DEG; ++d) lin[k][d] = tin[k][d] = ol[k][d] = ot[k][d] = 0;
#pragma unroll
                for (int d = 0; d < NQ; ++d) qn[k][d] = 0;
            }
        }
        __builtin_amdgcn_s_setprio(0);
        if (stop) return 0;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int ly = ly0 + k * RPP;
            bool wrong = false;
            T g[DEG];
            precision(k, lin[k], g, wrong);
            information(k, tin[k], g, wrong);
            if (wrong && right(ly, 1) && bad == 0) bad = 1;
            if (n > 1) {
                put(k, ol[k], 0);
                if (!SPLIT) put(k, ot[k], INFO);
            }
        }
    }
#pragma unroll 1
    for (int s = 2; s <= n; ++s) {
        __syncthreads();
        T lin[NPT][DEG], tin[NPT][DEG], g[NPT][DEG];
        bool wrong[NPT];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if (!live(ly0 + k * RPP, s)) continue;
            get(k, lin[k], 0);
            if (!SPLIT) get(k, tin[k], INFO);
        }
        if (SPLIT) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NPT; ++k) put(k, ot[k], 0);
        } else if (s < n) {
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            wrong[k] = false;
            if (!live(ly0 + k * RPP, s)) continue;
            precision(k, lin[k], g[k], wrong[k]);
        }
        if (SPLIT) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NPT; ++k)
                if (live(ly0 + k * RPP, s)) get(k, tin[k], 0);
            if (s < n) __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int ly = ly0 + k * RPP;
            if (!live(ly, s)) continue;
            information(k, tin[k], g[k], wrong[k]);
            if (wrong[k] && right(ly, s) && bad == 0) bad = s;
            if (s < n) {
                put(k, ol[k], 0);
                if (!SPLIT) put(k, ot[k], INFO);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int ly = ly0 + k * RPP, x = x0 + lx, y = y0 + ly;
        if (!right(ly, S) || x >= L.nx || y >= L.ny) continue;
        const uint32_t i = (uint32_t)(y * L.pitch + x);
#pragma unroll
        for (int d = 0; d < DEG; ++d) {
            if (!has(k, d)) continue;
            __builtin_nontemporal_store(ol[k][d], &(m_out + (size_t)d * L.plane)[i]);
            __builtin_nontemporal_store(ot[k][d], &(m_out + (size_t)(DEG + d) * L.plane)[i]);
        }
    }
    return bad;
}

}  // namespace gabp
