// Iteration kernels of the space-time solver (include/gabp_st.h): the GMRF of
// the stochastic heat equation discretised by Crank-Nicolson steps (paper:
// Appendix "Extension to Spatiotemporal Systems"), solved by the damped,
// re-weighted flooding iteration on its 38-neighbour graph.
//
// Precision closed form.  With G the graph Laplacian of the grid (unit
// spacing; G_ii = g_i, the number of in-grid axis neighbours of i, G_ij = -1
// for grid neighbours), Lap_h = -G/h^2 and every block of M is a polynomial
// in G: A = a1 I + a2 G, B = a1 I - a2 G, L = l1 I + l2 G with a1 = 1/dt,
// a2 = nu/(2 h^2), l1 = a0 kappa^2, l2 = a0/h^2.  The blocks of
// Q = S M^T M (S = dt h^2 / sigma_u^2) are then polynomials p I + q G + r G^2:
//     slice 0:        S (L^2 + B^2)      (S L^2 when there is one slice)
//     slices 1..N-2:  S (A^2 + B^2)
//     slice N-1:      S A^2
//     between n, n+1: -S A B = -S (a1^2 I - a2^2 G^2)
// and the entries of p I + q G + r G^2 follow from those of G and G^2 (the
// grid graph is bipartite, so grid neighbours share no neighbour):
//     (i, i):               p + q g_i + r (g_i^2 + g_i)
//     one step:             -q - r (g_i + g_j)
//     two steps on an axis: r
//     diagonal:             2 r
// The host folds the three products of each block into one (p, q, r) in
// FP64; kernels evaluate the entries from it, the position and the slice.
//
// Storage.  Sender-indexed SoA planes as in the lattice kernels: plane d at
// node i holds the message from i to i + off_d (d = 0..37, opposite d ^ 1),
// precisions in planes 0..37 and information in planes 38..75.  A node's
// plane index is n * slice + y * pitch + x with slice = pitch * ny.
//
// Launch shape.  A workgroup of 64 x 4 threads per slice owns one 64 x 4 tile
// of one slice (or of SL consecutive slices), a row to a wave; the workgroup
// order (wg_tile) keeps the tiles that share halo rows and slices on one XCD at
// nearly the same time.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lattice.h"
#include "numerics.h"
#include "prec_change.h"

#pragma clang fp contract(off)

namespace gabp {
namespace st {


constexpr int kDeg = 38;

// Direction tables: d < 12 lie in the slice (the lattice directions of
// lattice.h); d = 12 + 2k is (o_k, +1), d = 13 + 2k is (-o_k, -1), with
// o_0 = (0, 0) and o_k the lattice direction k - 1.
__host__ __device__ constexpr int cross_k(int d) { return (d - 12) >> 1; }
__host__ __device__ constexpr int sdx(int d) {
    return d < 12 ? dir_dx(d)
                  : cross_k(d) == 0 ? 0 : ((d & 1) ? -dir_dx(cross_k(d) - 1) : dir_dx(cross_k(d) - 1));
}
__host__ __device__ constexpr int sdy(int d) {
    return d < 12 ? dir_dy(d)
                  : cross_k(d) == 0 ? 0 : ((d & 1) ? -dir_dy(cross_k(d) - 1) : dir_dy(cross_k(d) - 1));
}
__host__ __device__ constexpr int sdt(int d) { return d < 12 ? 0 : ((d & 1) ? -1 : 1); }
// spatial relation of direction d: 0 same position, 1 one step, 2 two steps
// along an axis, 3 diagonal
__host__ __device__ constexpr int scls(int d) {
    return d < 12 ? (d < 4 ? 1 : d < 8 ? 2 : 3)
                  : cross_k(d) == 0 ? 0 : (cross_k(d) - 1 < 4 ? 1 : cross_k(d) - 1 < 8 ? 2 : 3);
}

struct Grid {
    int32_t nx, ny, nt, pitch;
    int32_t bcx, bcy, tiles_x, tiles_y;
    int64_t slice;              // elements between slices (pitch * ny)
    int64_t plane;              // elements between planes
    double blk[4][3];           // (p, q, r) of blocks: slice 0, middle, last, coupling
    double lsq[3];              // (p, q, r) of S L^2, the initial condition's precision
    double c, inv_c;
};

__device__ __forceinline__ int axis_g(int v, int n, int bc) {
    return bc == BC_PERIODIC ? 2 : (int)(v > 0) + (int)(v < n - 1);
}

__device__ __forceinline__ int slice_kind(const Grid &G, int t) {
    return t == 0 ? 0 : (t == G.nt - 1 ? 2 : 1);
}

// Entry of p I + q G + r G^2 for a relation class (g_j only for one step).
template <typename T>
__device__ __forceinline__ T coef(const double *pqr, int cls, T gi, T gj) {
    const T p = (T)pqr[0], q = (T)pqr[1], r = (T)pqr[2];
    if (cls == 0) return p + q * gi + r * (gi * gi + gi);
    if (cls == 1) return -q - r * (gi + gj);
    if (cls == 2) return r;
    return r + r;
}

// Neighbour of (x, y, t) in direction d: wraps periodic axes; false when it
// lies outside the grid.
__device__ __forceinline__ bool nbr(const Grid &G, int x, int y, int t, int d, int &xn, int &yn,
                                    int &tn) {
    xn = x + sdx(d);
    yn = y + sdy(d);
    tn = t + sdt(d);
    if ((unsigned)tn >= (unsigned)G.nt) return false;
    if (G.bcx == BC_PERIODIC) {
        xn = xn < 0 ? xn + G.nx : (xn >= G.nx ? xn - G.nx : xn);
    } else if ((unsigned)xn >= (unsigned)G.nx) {
        return false;
    }
    if (G.bcy == BC_PERIODIC) {
        yn = yn < 0 ? yn + G.ny : (yn >= G.ny ? yn - G.ny : yn);
    } else if ((unsigned)yn >= (unsigned)G.ny) {
        return false;
    }
    return true;
}

// --------------------------------------------------------------------------
// One flooding iteration of node (x, y, t) (as the lattice kernels):
//   Lam_i = A_ii + c sum_k Lam_{k->i},  th_i = b_i + c sum_k th_{k->i}
//   for each neighbour j: Lam_c = Lam_i - Lam_{j->i}, th_c = th_i - th_{j->i},
//   g = -(Q_ij/c)/Lam_c, new (g Q_ij/c, g th_c), damped with the previous
//   outgoing message (Appendix "Re-weighted message updates"; Section
//   "Update Damping").
//
// Boundaries cost no masks on the incoming messages: every coordinate wraps,
// on any axis.  On a periodic axis that is the neighbour; on another one the
// node reached lies at the far end, and its message in the opposite
// direction leaves the grid there, a slot that is always zero.  A wave is one
// row of one slice, so that the rows and slices reached are scalars and only
// the five column offsets are per lane (Reach).  What remains of the boundary
// is whether an outgoing edge exists and the neighbour counts in Q_ij; waves
// whose edges all exist (`inner`, uniform) skip both.
// --------------------------------------------------------------------------
__device__ __forceinline__ int wrap(int v, int n) {   // v in [-2, n + 1]
    v = v < 0 ? v + n : (v >= n ? v - n : v);
    return min(max(v, 0), n - 1);                     // n = 1: two steps wrap twice
}

// What lies `bytes` behind a wave-uniform address.  With a 32-bit offset an
// access takes the address from scalar registers and one register per lane, and
// needs no 64-bit arithmetic.
template <typename T>
__device__ __forceinline__ T *behind(T *row, uint32_t bytes) {
    return (T *)((char *)row + bytes);
}
template <typename T>
__device__ __forceinline__ const T *behind(const T *row, uint32_t bytes) {
    return (const T *)((const char *)row + bytes);
}

struct Reach {
    uint32_t row[3][5];   // element offset of row y + dy of slice t + dt, wrapped
    int col[5];           // column x + dx, wrapped (per lane)
    uint32_t at[5];       // its byte offset in a row
    __device__ __forceinline__ Reach(const Grid &G, int x, int y, int t, uint32_t esize) {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            col[k] = wrap(x + k - 2, G.nx);
            at[k] = (uint32_t)col[k] * esize;
            asm volatile("" : "+v"(at[k]));   // not a 64-bit index to the compiler
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint32_t s = (uint32_t)wrap(t + q - 1, G.nt) * (uint32_t)G.slice;
#pragma unroll
            for (int k = 0; k < 5; ++k) row[q][k] = s + (uint32_t)(wrap(y + k - 2, G.ny) * G.pitch);
        }
    }
    // incoming message of direction d, plane at m
    template <typename T>
    __device__ __forceinline__ T in(const T *__restrict__ m, int d) const {
        return *behind(m + row[sdt(d) + 1][sdy(d) + 2], at[sdx(d) + 2]);
    }
};

// Belief parameter: a + c * sum_d v[d], summed in direction order.
template <typename T>
__device__ __forceinline__ T belief(T a, const T *v, T c) {
    T s = 0;
#pragma unroll
    for (int d = 0; d < kDeg; ++d) s += v[d];
    return fmadd(c, s, a);
}

// Q_ij / c for direction d (closed forms at the top of this file); gi and gj
// are the two nodes' neighbour counts (gj for one step only), pq_same /
// pq_cross the slice's blocks.
template <typename T>
__device__ __forceinline__ T q_dir(const Grid &G, int d, T gi, T gj, const T *pq_same,
                                   const T *pq_cross) {
    const T *pqr = d < 12 ? pq_same : pq_cross;
    T q;
    if (scls(d) == 0) q = pqr[0] + pqr[1] * gi + pqr[2] * (gi * gi + gi);
    else if (scls(d) == 1) q = -pqr[1] - pqr[2] * (gi + gj);
    else if (scls(d) == 2) q = pqr[2];
    else q = pqr[2] + pqr[2];
    return q * (T)G.inv_c;
}

// --------------------------------------------------------------------------
// Frozen precision messages.  The precision recursion involves neither the
// information messages nor the data, so once one iteration leaves every
// precision message unchanged, all later ones do too.  The edge gains
// g = -(Q_ij/c)/Lam_c are then stored once (MODE_GAIN) and the iteration
// updates only the information messages (MODE_THETA):
//   th_i = b_i + c sum_d th_{k->i},  out_d = (1 - eta) out_d + eta g_d (th_i - th_{j->i}).
// All three modes share Reach, belief and q_dir, so the information-only
// iteration is bitwise the full one's.  New messages are written with
// non-temporal stores (nothing reads them in the same launch; 4-5 % faster)
// and the gains, read once per iteration, are loaded non-temporally (4 %
// more on the information-only kernel; on the lattice's two-iteration tiles
// the same hint costs 4 %, so it is used here only).
// --------------------------------------------------------------------------
enum { MODE_FULL = 0, MODE_GAIN = 1, MODE_THETA = 2 };

// Edges of a node: INNER, every neighbour exists and has four in its slice.
template <typename T, bool INNER>
struct Edges {
    const Grid &G;
    const T *pq_same, *pq_cross;
    int x, y, t;
    T gi, gs[4];   // neighbour counts of the node and of its four axis neighbours
    __device__ __forceinline__ Edges(const Grid &g, const Reach &R, const T *same, const T *cross,
                                     int x_, int y_, int t_)
        : G(g), pq_same(same), pq_cross(cross), x(x_), y(y_), t(t_) {
        gi = INNER ? (T)4 : count(x, y);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            gs[k] = INNER ? (T)4 : count(R.col[dir_dx(k) + 2], wrap(y + dir_dy(k), G.ny));
    }
    __device__ __forceinline__ T count(int xn, int yn) const {
        return (T)(axis_g(xn, G.nx, G.bcx) + axis_g(yn, G.ny, G.bcy));
    }
    __device__ __forceinline__ T q(int d) const {
        const int step = sdx(d) == 1 ? 0 : sdx(d) == -1 ? 1 : sdy(d) == 1 ? 2 : 3;
        return q_dir<T>(G, d, gi, scls(d) == 1 ? gs[step] : (T)0, pq_same, pq_cross);
    }
    __device__ __forceinline__ bool ok(int d) const {
        if (INNER) return true;
        const bool px = G.bcx == BC_PERIODIC, py = G.bcy == BC_PERIODIC;
        return (bool)((int)((unsigned)(t + sdt(d)) < (unsigned)G.nt) &
                      ((int)py | (int)((unsigned)(y + sdy(d)) < (unsigned)G.ny)) &
                      ((int)px | (int)((unsigned)(x + sdx(d)) < (unsigned)G.nx)));
    }
};

// A node's previous outgoing messages (MODE_THETA: the gains in place of the precision
// messages).  Those of the first AHEAD directions are loaded beside the incoming
// messages, direction d's of the others when direction d - AHEAD is computed.
template <typename T, int MODE, int AHEAD>
struct Own {
    T l[AHEAD > 0 ? kDeg : 1], t[AHEAD > 0 ? kDeg : 1];
    __device__ __forceinline__ void load(int d, const T *__restrict__ m_in,
                                         const T *__restrict__ gain, int64_t plane, uint32_t rc,
                                         uint32_t xb) {
        if constexpr (AHEAD > 0) {
            const size_t at = (size_t)d * plane + rc, at2 = (size_t)(kDeg + d) * plane + rc;
            l[d] = *behind((MODE == MODE_THETA ? gain : m_in) + at, xb);
            t[d] = *behind(m_in + at2, xb);
        }
    }
};

// New messages of a node from its gathered incoming ones and its beliefs (bl
// unused in MODE_THETA, bt and tin in MODE_GAIN).  The planes' addresses are
// made again (`plane` is a copy the compiler cannot tell from another value)
// rather than kept from the gather: 76 pairs of scalar registers spill.
template <typename T, int MODE, bool INNER, int AHEAD>
__device__ __forceinline__ void st_out(const Edges<T, INNER> &E, int64_t plane, uint32_t rc, uint32_t xb,
                                       const T *__restrict__ m_in, T *__restrict__ m_out,
                                       T *__restrict__ gain, T eta, const T *lin, const T *tin,
                                       T bl, T bt, Own<T, MODE, AHEAD> &own, bool &bad) {
    const T keep = (T)1 - eta;
    T z = (T)0;   // MODE_THETA: stays zero exactly when every new message is finite
#pragma unroll
    for (int d = 0; d < kDeg; ++d) {
        if (AHEAD > 0 && d + AHEAD < kDeg) {
            own.load(d + AHEAD, m_in, gain, plane, rc, xb);
            __builtin_amdgcn_sched_barrier(0);
        }
        const bool ok = E.ok(d);
        const size_t at = (size_t)d * plane + rc, at2 = (size_t)(kDeg + d) * plane + rc;
        if constexpr (MODE == MODE_FULL) {
            const T q = E.q(d);
            const T lc = bl - lin[d];
            const T tc = bt - tin[d];
            const T g = edge_gain(q, lc);
            const T ol = AHEAD > 0 ? own.l[AHEAD > 0 ? d : 0] : *behind(m_in + at, xb);
            const T ot = AHEAD > 0 ? own.t[AHEAD > 0 ? d : 0] : *behind(m_in + at2, xb);
            T dl = fmadd(eta, g * q, keep * ol);
            T dt = fmadd(eta, g * tc, keep * ot);
            bad |= ok && (!(lc > (T)0) || !isfinite(dl) || !isfinite(dt));
            dl = ok ? dl : (T)0;
            dt = ok ? dt : (T)0;
            __builtin_nontemporal_store(dl, behind(m_out + at, xb));
            __builtin_nontemporal_store(dt, behind(m_out + at2, xb));
        } else if constexpr (MODE == MODE_GAIN) {
            const T g = edge_gain(E.q(d), bl - lin[d]);
            *behind(gain + at, xb) = ok ? g : (T)0;
        } else {
            // edges that do not exist: gain and previous message are zero
            const T g = AHEAD > 0 ? own.l[AHEAD > 0 ? d : 0] : __builtin_nontemporal_load(behind(gain + at, xb));
            const T ot = AHEAD > 0 ? own.t[AHEAD > 0 ? d : 0] : *behind(m_in + at2, xb);
            const T dt = fmadd(eta, g * (bt - tin[d]), keep * ot);
            z = fmadd(dt, (T)0, z);
            __builtin_nontemporal_store(dt, behind(m_out + at2, xb));
        }
    }
    if (MODE == MODE_THETA) bad = !(z == (T)0);
}

// Workgroup -> (tile x, tile y, first slice).  A workgroup covers one 64 x 4
// tile on SL consecutive slices (4 waves per slice): the messages that pass
// between those slices are read twice inside one workgroup.  Tiles are
// grouped in bands of kGroupRows tile rows; within a band the order is slice
// group by slice group, each row by row.  With the XCD remap each XCD runs a
// contiguous range of this order, so a tile's vertical neighbours (same
// slices) are at most a few tile rows away and its slice neighbours one
// band-slice (tiles_x * kGroupRows workgroups) away: both halos are read
// while still in L2.
// Band height, measured on 512 x 512 x 64 (information-only iteration, ms):
// 2 rows 1.540, 4 rows 1.473, 8 rows 1.443, 16 rows 1.424, 32 rows 1.486,
// 128 rows (one band) 1.700.
constexpr int kGroupRows = 16;

// Band and slice-group order over a box of tiles_x x tiles_y tiles and nt
// slices: workgroup b -> (tx, ty, first slice) relative to the box.
template <int SL>
__device__ __forceinline__ void wg_tile(int b, int tiles_x, int tiles_y, int nt, int &tx, int &ty,
                                        int &t0) {
    const int groups = (nt + SL - 1) / SL;
    const int full = kGroupRows * tiles_x * groups;         // workgroups of a full band
    const int g = b / full;
    const int r = b - g * full;
    const int hg = min(kGroupRows, tiles_y - g * kGroupRows);   // tile rows of this band
    const int per_slice = hg * tiles_x;
    const int sg = r / per_slice;
    const int r2 = r - sg * per_slice;
    const int tyi = r2 / tiles_x;
    tx = r2 - tyi * tiles_x;
    ty = g * kGroupRows + tyi;
    t0 = sg * SL;
}

// One launch of a mode over the grid, SL slices per workgroup.  Bound by memory
// on large grids: 512 x 512 x 64 in FP32, 2.21 ms per full iteration (10.3 GB read and
// written once at least: 4.6 TB/s; 2.64 ms when boundary tiles took a masked
// path in a second launch) and 1.42 ms per information-only one (7.6 GB, 5.4 TB/s,
// above what a device copy streams).  AHEAD: a node's previous messages (and
// gains) are loaded beside the incoming ones, of so many directions (Own), every load
// before the first use, at the price of registers.  The full iteration has it in FP32
// for all 38: 183 VGPRs, two waves per SIMD, against 112 and four, yet 25 -> 18 us on
// 100 x 75 x 12, 675 -> 567 on 256 x 256 x 64, 2380 -> 2208 on 512 x 512 x 64; held to
// three waves it spills (670 and 2675).  In FP64 for six at a time, as many as fit into
// the 256 VGPRs of two waves (248; 204 with none, 36 spilled with 12): 100 x 75 x 12
// 37.3 -> 30.0, 256 x 256 x 16 419 -> 297, 128 x 128 x 64 417 -> 280, periodic 130 x
// 130 x 10 67 -> 60.5.
// diverged_at[0] records the first iteration whose launch met an invalid value;
// launches of later iterations return at once (the launch of the iteration that met
// it completes, so its output buffer holds that iteration).  MODE_GAIN passes
// it = 0.
template <typename T, int MODE, int SL, int AHEAD>
__global__ __launch_bounds__(256 * SL,
                             sizeof(T) == 8 || AHEAD > 0 ? 2 : MODE == MODE_THETA ? 8 : 4) void k_iter(
    Grid G, const T *__restrict__ m_in, T *__restrict__ m_out, T *__restrict__ gain,
    const T *__restrict__ aw, const T *__restrict__ bw, T eta, uint32_t *__restrict__ diverged_at,
    uint32_t it) {
    const uint32_t seen = *diverged_at;
    if (MODE != MODE_GAIN && seen != 0u && seen < it) return;
    int tx, ty, t0;
    wg_tile<SL>(xcd_remap((int)blockIdx.x, (int)gridDim.x), G.tiles_x, G.tiles_y, G.nt, tx, ty, t0);
    // one row of one slice per wave
    const int t = __builtin_amdgcn_readfirstlane(t0 + (int)(threadIdx.x >> 8));
    const int y = __builtin_amdgcn_readfirstlane(ty * 4 + (int)((threadIdx.x >> 6) & 3u));
    const int x = tx * 64 + (int)(threadIdx.x & 63u);
    if (t >= G.nt || y >= G.ny || x >= G.nx) return;
    // the slice's blocks (uniform over the wave) in message precision
    const int kind = slice_kind(G, t);
    const T pq_same[3] = {(T)G.blk[kind][0], (T)G.blk[kind][1], (T)G.blk[kind][2]};
    const T pq_cross[3] = {(T)G.blk[3][0], (T)G.blk[3][1], (T)G.blk[3][2]};
    const bool inner = (G.bcx == BC_PERIODIC || (tx * 64 >= 2 && tx * 64 + 66 <= G.nx)) &&
                       (G.bcy == BC_PERIODIC || (y >= 2 && y + 2 < G.ny)) && t > 0 && t < G.nt - 1;
    const Reach R(G, x, y, t, (uint32_t)sizeof(T));
    const uint32_t rc = R.row[1][2], xb = R.at[2];   // the node's own row and column
    const T c = (T)G.c;
    T lin[kDeg], tin[kDeg], bl = 0, bt = 0;
    // the full iteration's gather at a raised wave priority (as the lattice
    // kernels); the information-only iteration does not gain from it
    if (MODE == MODE_FULL) __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int d = 0; d < kDeg; ++d) {
        if (MODE != MODE_THETA) lin[d] = R.in(m_in + (size_t)(d ^ 1) * G.plane, d);
        if (MODE != MODE_GAIN) tin[d] = R.in(m_in + (size_t)(kDeg + (d ^ 1)) * G.plane, d);
    }
    Own<T, MODE, AHEAD> own;
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) own.load(d, m_in, gain, G.plane, rc, xb);
    const T a = *behind(aw + rc, xb), b = *behind(bw + rc, xb);
    if (AHEAD > 0) __builtin_amdgcn_sched_barrier(0);   // every load is on its way
    if (MODE == MODE_FULL) __builtin_amdgcn_s_setprio(0);
    if (MODE != MODE_THETA) bl = belief(a, lin, c);
    if (MODE != MODE_GAIN) bt = belief(b, tin, c);
    uint32_t pl = (uint32_t)G.plane;      // below 2^31 + 512
    asm volatile("" : "+s"(pl));
    const int64_t plane = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)pl);
    bool bad = false;
    if (MODE == MODE_THETA || inner)
        st_out<T, MODE, true, AHEAD>(Edges<T, true>(G, R, pq_same, pq_cross, x, y, t), plane, rc, xb, m_in,
                              m_out, gain, eta, lin, tin, bl, bt, own, bad);
    else
        st_out<T, MODE, false, AHEAD>(Edges<T, false>(G, R, pq_same, pq_cross, x, y, t), plane, rc, xb, m_in,
                               m_out, gain, eta, lin, tin, bl, bt, own, bad);
    if (MODE != MODE_GAIN && bad) atomicCAS(diverged_at, 0u, it);
}

// The freeze test (prec_change.h); a non-finite element counts as an infinite
// change, and so does one whose two values are zeros of different sign.
struct StRel {
    __device__ __forceinline__ static float of(double u, double v) {
        const double den = fmax(fabs(u), fabs(v));
        const float r = den > 0.0 ? (float)(fabs(u - v) / den) : INFINITY;
        return isnan(r) ? INFINITY : r;
    }
};

template <typename T>
__global__ __launch_bounds__(256) void k_prec_change(const T *__restrict__ a,
                                                     const T *__restrict__ b, int64_t n,
                                                     uint64_t limit,
                                                     unsigned long long *__restrict__ count,
                                                     uint32_t *__restrict__ maxrel_bits) {
    prec_change_wave<T, StRel>(a, b, n, (int)(blockIdx.x * 4 + (threadIdx.x >> 6)),
                               (int)gridDim.x * 4, limit, count, maxrel_bits);
}

}  // namespace st
}  // namespace gabp
