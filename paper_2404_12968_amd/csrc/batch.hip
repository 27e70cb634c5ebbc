// Batched solving of many independent lattice problems of uneven sizes
// (C ABI: gabp_batch_* in include/gabp.h).
//
// Every instance keeps its own sender-indexed message planes and node planes
// inside one workspace.  A device-resident instance table describes them.
// The instances still running are grouped by prior order and phase (full or
// information-only iteration).  One launch takes several iterations of a whole
// group, over a work list of (instance, tile) items (deep_tile.h, deep_full.h);
// the launch boundary is the flooding barrier, so no workgroup ever waits on
// another.  Converged or diverged instances leave the work lists; each instance
// switches to the information-only iteration on its own once its precision
// messages freeze.  A check of all running instances is three launches that
// report to pinned host memory.
//
// The per-node bodies are those of the single-lattice kernels (iter_node.h,
// check_node.h): a batched instance computes bitwise what a lone context
// computes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "check_node.h"
#include "deep_full.h"
#include "deep_tile.h"
#include "gabp.h"
#include "host_common.h"
#include "internal.h"
#include "iter_node.h"
#include "prec_change.h"
#include "lattice.h"
#include "numerics.h"

#pragma clang fp contract(off)

namespace gabp {

// Device record of one instance.
struct BatchInst {
    Lattice L;
    void *msg[2];
    void *gain;
    const void *adiag_w, *b_w;
    double *adiag64, *b64, *mu64, *bel64;
};

// Largest a in [0, n) with prefix[a] <= w (prefix[0] = 0, increasing).
__device__ __forceinline__ int find_item(const int *__restrict__ prefix, int n, int w) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= w) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// One iteration (number t) of every instance of a list, from its buffer `buf` to the
// other: full, or, FROZEN, information-only.  Workgroup g after the XCD remap takes
// work item prefix[0] + g, tile item - prefix[a] of instance act[a] (64 x 4*RPT nodes,
// a row of threads to every fourth row) in the strip order of the lone context's
// kernels, so that each XCD takes a contiguous range of tiles and the rows a tile
// shares with its neighbours are in its L2.
// ALPHA: the instances' prior order, 0 for either.
// The rows are a loop the compiler cannot see through, also where there is one: the
// loads of every prior order, inside and at the boundary, brought in front of their
// branches took 231 registers in FP32 and 256 in FP64 (now 131 and 211, for one order
// of 13 points 128 and 204).  One iteration of 1024^2 alone, call and waits included,
// FP32 73 -> 68 us, FP64 132 -> 105; of 2048 x 1024 with 13 and with 5 points 153 -> 140
// and 321 -> 265 (two launches); information-only 76 -> 52, 110 -> 74, 165 -> 104 and
// 270 -> 195, where a tile of several iterations had taken one.
template <typename T, int RPT, int ALPHA, bool FROZEN>
__global__ __launch_bounds__(256) void k_batch_iter(const BatchInst *__restrict__ inst,
                                                    const int *__restrict__ act,
                                                    const int *__restrict__ prefix, int nact,
                                                    int buf, uint32_t t, T eta,
                                                    uint32_t *__restrict__ diverged_at) {
    constexpr int TH = 4 * RPT;
    const int w = prefix[0] + xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int a = __builtin_amdgcn_readfirstlane(find_item(prefix, nact, w));
    const int I = __builtin_amdgcn_readfirstlane(act[a]);
    const uint32_t seen = diverged_at[I];
    if (seen != 0u && seen < t) return;   // of an earlier iteration: this one is written whole
    const BatchInst &B = inst[I];
    const Lattice L = B.L;
    int tx, ty;
    strip_order(w - prefix[a], L.tiles_x, (L.ny + TH - 1) / TH, tx, ty);
    const int x = tx * 64 + (int)(threadIdx.x & 63u);
    const int y0 = ty * TH + (int)(threadIdx.x >> 6);
    const bool interior = tx * 64 >= 2 && tx * 64 + 66 <= L.nx && ty * TH >= 2 &&
                          ty * TH + TH + 2 <= L.ny;
    const T *m_in = (const T *)B.msg[buf], *bw = (const T *)B.b_w;
    const T *co = (const T *)(FROZEN ? B.gain : B.adiag_w);
    T *m_out = (T *)B.msg[buf ^ 1];
    bool bad = false;
    int rows = RPT;
    asm volatile("" : "+s"(rows));
    if (x < L.nx) {
#pragma unroll 1
        for (int k = 0; k < rows; ++k) {
            const int y = y0 + 4 * k;
            if (y >= L.ny) break;
            if constexpr (FROZEN) {
                if (ALPHA == 1 || (ALPHA == 0 && L.alpha == 1)) {
                    if (interior) iter_theta_node<T, 1, true>(L, m_in, m_out, co, bw, eta, bad, x, y);
                    else iter_theta_node<T, 1, false>(L, m_in, m_out, co, bw, eta, bad, x, y);
                } else {
                    if (interior) iter_theta_node<T, 2, true>(L, m_in, m_out, co, bw, eta, bad, x, y);
                    else iter_theta_node<T, 2, false>(L, m_in, m_out, co, bw, eta, bad, x, y);
                }
            } else {
                if (ALPHA == 1 || (ALPHA == 0 && L.alpha == 1)) {
                    if (interior) iter_node<T, 1, true>(L, m_in, m_out, co, bw, eta, bad, x, y);
                    else iter_node<T, 1, false>(L, m_in, m_out, co, bw, eta, bad, x, y);
                } else {
                    if (interior) iter_node<T, 2, true>(L, m_in, m_out, co, bw, eta, bad, x, y);
                    else iter_node<T, 2, false>(L, m_in, m_out, co, bw, eta, bad, x, y);
                }
            }
        }
    }
    if (bad) diverged_at[I] = t;
}

// Work item of a multi-iteration launch: the tile (tx, ty) of instance I, on the
// tiles for S iterations of a region of RW x RH nodes; items are XCD-remapped so
// that each XCD takes a contiguous range of them.
template <int ALPHA, int RW, int RH>
__device__ __forceinline__ const BatchInst &deep_item(const BatchInst *__restrict__ inst,
                                                      const int *__restrict__ act,
                                                      const int *__restrict__ prefix, int nact,
                                                      int S, int &I, int &tx, int &ty,
                                                      bool &inside) {
    using Rg = DeepRegion<ALPHA, RW, RH>;
    const int w = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int a = __builtin_amdgcn_readfirstlane(find_item(prefix, nact, w));
    I = __builtin_amdgcn_readfirstlane(act[a]);
    const BatchInst &B = inst[I];
    const int cols = (B.L.nx + Rg::tw(S) - 1) / Rg::tw(S), tile = w - prefix[a];
    tx = tile % cols;
    ty = tile / cols;
    const int x0 = tx * Rg::tw(S) - Rg::halo(S), y0 = ty * Rg::th(S) - Rg::halo(S);
    inside = x0 >= Rg::R && x0 + RW + Rg::R <= B.L.nx && y0 >= Rg::R && y0 + RH + Rg::R <= B.L.ny;
    return B;
}

// n <= S information-only iterations of every instance of a list (frozen, prior
// order ALPHA), from iteration t in its buffer `buf` to the other.
// Ten iterations of the frozen instances were four launches of two and two single
// ones, each with its own fill and drain; they are two launches of five.  24
// instances of 64^2 to 400^2 (FP32, 400 iterations, checks included): 21.6 -> 12.8
// ms, of which the information-only launches took 4.4 ms and take 3.6, the others
// 7.9 and 2.7.
template <typename T, int ALPHA, int RW, int RH>
__global__ __launch_bounds__(1024) void k_batch_deep(const BatchInst *__restrict__ inst,
                                                     const int *__restrict__ act,
                                                     const int *__restrict__ prefix, int nact,
                                                     int S, int n, int buf, uint32_t t, T eta,
                                                     uint32_t *__restrict__ diverged_at) {
    __shared__ T lds[DeepRegion<ALPHA, RW, RH>::kLds];
    int I, tx, ty;
    bool inside;
    const BatchInst &B = deep_item<ALPHA, RW, RH>(inst, act, prefix, nact, S, I, tx, ty, inside);
    const uint32_t seen = diverged_at[I];
    const bool stop = seen != 0u && seen <= t;
    const Lattice L = B.L;
    const T *m_in = (const T *)B.msg[buf], *gain = (const T *)B.gain, *bw = (const T *)B.b_w;
    T *m_out = (T *)B.msg[buf ^ 1];
    int bad;
    if (inside)
        bad = deep_tile<T, ALPHA, RW, RH, 1024, true>(L, m_in, m_out, gain, bw, eta, S, n, tx, ty,
                                                      stop, lds);
    else
        bad = deep_tile<T, ALPHA, RW, RH, 1024, false>(L, m_in, m_out, gain, bw, eta, S, n, tx, ty,
                                                       stop, lds);
    record_first(bad, t, &diverged_at[I]);
}

// The same for full iterations.
template <typename T, int ALPHA, int RW, int RH, int NT, bool SPLIT>
__global__ __launch_bounds__(NT) void k_batch_deep_full(const BatchInst *__restrict__ inst,
                                                        const int *__restrict__ act,
                                                        const int *__restrict__ prefix, int nact,
                                                        int S, int n, int buf, uint32_t t, T eta,
                                                        uint32_t *__restrict__ diverged_at) {
    __shared__ T lds[deep_full_lds<ALPHA, RW, RH, SPLIT>()];
    int I, tx, ty;
    bool inside;
    const BatchInst &B = deep_item<ALPHA, RW, RH>(inst, act, prefix, nact, S, I, tx, ty, inside);
    const uint32_t seen = diverged_at[I];
    const bool stop = seen != 0u && seen <= t;
    const Lattice L = B.L;
    const T *m_in = (const T *)B.msg[buf], *ad = (const T *)B.adiag_w, *bw = (const T *)B.b_w;
    T *m_out = (T *)B.msg[buf ^ 1];
    int bad;
    if (inside)
        bad = deep_full_tile<T, ALPHA, RW, RH, NT, SPLIT, true>(L, m_in, m_out, ad, bw, eta, S, n,
                                                                tx, ty, stop, lds);
    else
        bad = deep_full_tile<T, ALPHA, RW, RH, NT, SPLIT, false>(L, m_in, m_out, ad, bw, eta, S, n,
                                                                 tx, ty, stop, lds);
    record_first(bad, t, &diverged_at[I]);
}

// Marginals of every running instance (64 x 4 tiles, the first `blocks`
// workgroups), writing each instance's FP64 mean plane and, until its precision
// messages freeze, its belief precisions.  kProbeBlocks further workgroups for
// each instance of the list actu (running, not frozen) take its freeze test
// (prec_change.h).  Both read buffer `buf`.
constexpr int kProbeBlocks = 64;
template <typename T>
__global__ __launch_bounds__(256) void k_batch_post(const BatchInst *__restrict__ inst,
                                                    const int *__restrict__ act,
                                                    const int *__restrict__ prefix, int nact,
                                                    int total, const int *__restrict__ frozen,
                                                    int buf, int blocks,
                                                    const int *__restrict__ actu, uint64_t limit,
                                                    unsigned long long *__restrict__ count,
                                                    uint32_t *__restrict__ maxrel) {
    if ((int)blockIdx.x >= blocks) {
        const int p = (int)blockIdx.x - blocks;
        const int I = __builtin_amdgcn_readfirstlane(actu[p / kProbeBlocks]);
        const BatchInst &B = inst[I];
        prec_change_wave<T, LatticeRel>((const T *)B.msg[buf], (const T *)B.msg[buf ^ 1],
                                        (int64_t)B.L.deg * B.L.plane,
                                        p % kProbeBlocks * 4 + (int)(threadIdx.x >> 6),
                                        kProbeBlocks * 4, limit, count + I, maxrel + I);
        return;
    }
    const int per = (total + blocks - 1) / blocks;
    const int w1 = min(total, ((int)blockIdx.x + 1) * per);
    for (int w = (int)blockIdx.x * per; w < w1; ++w) {
        const int a = find_item(prefix, nact, w);
        const int I = act[a];
        const BatchInst &B = inst[I];
        const Lattice L = B.L;
        const int tile = w - prefix[a];
        const int x = (tile % L.tiles_x) * 64 + (int)(threadIdx.x & 63u);
        const int y = (tile / L.tiles_x) * 4 + (int)(threadIdx.x >> 6);
        if (x >= L.nx || y >= L.ny) continue;
        const T *m = (const T *)B.msg[buf];
        if (L.alpha == 1) {
            if (frozen[I]) post_node<T, 1, true>(L, m, B.adiag64, B.b64, B.bel64, B.mu64, nullptr, nullptr, nullptr, x, y);
            else post_node<T, 1, false>(L, m, B.adiag64, B.b64, nullptr, B.mu64, nullptr, nullptr, B.bel64, x, y);
        } else {
            if (frozen[I]) post_node<T, 2, true>(L, m, B.adiag64, B.b64, B.bel64, B.mu64, nullptr, nullptr, nullptr, x, y);
            else post_node<T, 2, false>(L, m, B.adiag64, B.b64, nullptr, B.mu64, nullptr, nullptr, B.bel64, x, y);
        }
    }
}

// FP64 residual partial sums, one (r^2, b^2) pair per work item, each summed
// in a fixed order.
__global__ __launch_bounds__(256) void k_batch_resid(const BatchInst *__restrict__ inst,
                                                     const int *__restrict__ act,
                                                     const int *__restrict__ prefix, int nact,
                                                     int total, double *__restrict__ partials) {
    __shared__ double sh[2][4];
    const int per = (total + (int)gridDim.x - 1) / (int)gridDim.x;
    const int w1 = min(total, ((int)blockIdx.x + 1) * per);
    for (int w = (int)blockIdx.x * per; w < w1; ++w) {
        const int a = find_item(prefix, nact, w);
        const BatchInst &B = inst[act[a]];
        const Lattice L = B.L;
        const int tile = w - prefix[a];
        const int tx = tile % L.tiles_x, ty = tile / L.tiles_x;
        const int x = tx * 64 + (int)(threadIdx.x & 63u);
        const int y = ty * 4 + (int)(threadIdx.x >> 6);
        const bool interior = tx * 64 >= 2 && tx * 64 + 66 <= L.nx && ty * 4 >= 2 &&
                              ty * 4 + 6 <= L.ny;
        double rr = 0.0, bb = 0.0;
        if (L.alpha == 1) {
            if (interior) resid_node<1, true>(L, B.mu64, B.adiag64, B.b64, x, y, rr, bb);
            else if (x < L.nx && y < L.ny) resid_node<1, false>(L, B.mu64, B.adiag64, B.b64, x, y, rr, bb);
        } else {
            if (interior) resid_node<2, true>(L, B.mu64, B.adiag64, B.b64, x, y, rr, bb);
            else if (x < L.nx && y < L.ny) resid_node<2, false>(L, B.mu64, B.adiag64, B.b64, x, y, rr, bb);
        }
        rr = wave_sum(rr);
        bb = wave_sum(bb);
        const int wv = (int)(threadIdx.x >> 6);
        __syncthreads();
        if ((threadIdx.x & 63u) == 0u) {
            sh[0][wv] = rr;
            sh[1][wv] = bb;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            partials[2 * (int64_t)w] = (sh[0][0] + sh[0][1]) + (sh[0][2] + sh[0][3]);
            partials[2 * (int64_t)w + 1] = (sh[1][0] + sh[1][1]) + (sh[1][2] + sh[1][3]);
        }
    }
}

// One workgroup per running instance: fixed-order sum of its partials, reported
// to pinned host memory with its divergence and freeze-test words; clears the
// latter.
__global__ __launch_bounds__(256) void k_batch_reduce(const int *__restrict__ act,
                                                      const int *__restrict__ prefix,
                                                      const double *__restrict__ partials,
                                                      const uint32_t *__restrict__ diverged_at,
                                                      unsigned long long *__restrict__ count,
                                                      uint32_t *__restrict__ maxrel,
                                                      double *__restrict__ h_out,
                                                      uint32_t *__restrict__ h_div,
                                                      unsigned long long *__restrict__ h_count,
                                                      uint32_t *__restrict__ h_maxrel) {
    __shared__ double sh[2][4];
    const int a = (int)blockIdx.x;
    const int lo = prefix[a], hi = prefix[a + 1];
    double r = 0.0, b = 0.0;
    for (int k = lo + (int)threadIdx.x; k < hi; k += 256) {
        r += partials[2 * (int64_t)k];
        b += partials[2 * (int64_t)k + 1];
    }
    r = wave_sum(r);
    b = wave_sum(b);
    const int wv = (int)(threadIdx.x >> 6);
    if ((threadIdx.x & 63u) == 0u) {
        sh[0][wv] = r;
        sh[1][wv] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int I = act[a];
        h_out[2 * I] = (sh[0][0] + sh[0][1]) + (sh[0][2] + sh[0][3]);
        h_out[2 * I + 1] = (sh[1][0] + sh[1][1]) + (sh[1][2] + sh[1][3]);
        h_div[I] = diverged_at[I];
        h_count[I] = count[I];
        h_maxrel[I] = maxrel[I];
        count[I] = 0;
        maxrel[I] = 0;
    }
}

}  // namespace gabp

// ==========================================================================
// host side
// ==========================================================================
using gabp::BatchInst;
using gabp::Lattice;
using namespace gabp::host;

namespace {

thread_local std::string g_batch_create_error;

struct InstHost {
    Lattice L;
    int dtype;
    Layout lay;
    size_t base = 0;            // byte offset of the instance's region
    int tiles_check = 0;        // work items of the check kernels (64 x 4)
    bool running = true;
    bool frozen = false;
    int64_t frozen_at = -1;
    int status = GABP_E_NOT_CONVERGED;
    int64_t iters = 0;          // iterations applied to this instance
    double rel = INFINITY;
    double first_rel = -1.0;
    double prev_rel = -1.0;     // residual and iteration count at the check before
    int64_t prev_iters = 0;
    bool prev_valid = false;
    int64_t diverged_at = 0;    // first invalid iteration (0: none)
    int dbuf = -1;              // after a divergence: the buffer holding the kept state
};

// Buffer holding an instance's current messages: its iteration's parity,
// except after a divergence inside a launch of several iterations.
int state_buf(const InstHost &H) { return H.dbuf >= 0 ? H.dbuf : (int)(H.iters & 1); }

// Group of an instance: full iterations (0, 1) or information-only (2, 3), by
// prior order.
int group_of(const InstHost &H, bool frozen) { return (frozen ? 2 : 0) + (H.L.alpha == 1 ? 0 : 1); }

// One run of k iterations since the last check read-back: the iterations in
// multi-iteration launches and their number for each group, the couples of
// two-iteration launches that a divergence is reported by (hold_batch), and each
// instance's iteration and frozen flag at its start (-1: not running).
struct BatchRun {
    int k = 0;
    double eta = 0.0;
    int iters[4] = {0, 0, 0, 0}, deeps[4] = {0, 0, 0, 0};
    int couples = 0;
    std::vector<int64_t> t0;
    std::vector<char> frozen;
};

}  // namespace

struct gabp_batch {
    int n = 0;
    int dtype = 0;
    size_t esize = 4;
    int device = 0;
    hipStream_t ustream = nullptr;   // the caller's stream (may be the null stream)
    hipStream_t stream = nullptr;    // internal stream
    hipEvent_t ev_in = nullptr, ev_out = nullptr;
    char *ws = nullptr;
    size_t ws_bytes = 0;
    bool own_ws = false;
    std::vector<InstHost> h;
    // device arrays (inside the workspace)
    BatchInst *d_inst = nullptr;
    int *d_act = nullptr, *d_pprefix = nullptr, *d_frozen = nullptr;
    int *d_gact = nullptr;      // running, by group, those not frozen first
    int *d_gpre = nullptr, *d_spre = nullptr;   // their items of several and of one iteration
    uint32_t *d_div = nullptr, *d_t = nullptr, *d_err = nullptr;
    unsigned long long *d_cnt = nullptr;   // changed precision messages per instance
    uint32_t *d_mrel = nullptr;            // their largest relative change (float bits)
    double *d_partials = nullptr;
    size_t partial_cap = 0;     // work items of the check kernels
    // pinned host mirror
    double *p_out = nullptr;
    uint32_t *p_div = nullptr, *p_mrel = nullptr, *p_t = nullptr;
    unsigned long long *p_cnt = nullptr;
    int *p_lists = nullptr;     // kStages stagings of the lists,
    int staged = 0;             // of which copies may still read so many
    // rows per thread of the one-iteration kernel: the last iteration before a
    // check, of instances not frozen; one hides its loads best
    int rpt = 1;
    int cus = 256;
    int64_t freeze_slots = 0;   // freeze tolerance (gabp_batch_set_freeze_tolerance)
    double freeze_rel = 0.0;
    int64_t t = 0;              // iterations applied to the running set
    // current work lists
    int nact = 0, ptotal = 0, nu = 0;
    struct Group {
        int off = 0, n = 0;              // in d_gact and d_spre; in d_gpre from off + its index
        int items = 0, singles = 0;
        gabp::DeepPlan plan{0, 1};
        int S = 1;                       // iterations that its tiles are for, at most plan.S
    } group[4];
    bool lists_dirty = true;
    std::vector<BatchRun> runs;   // runs since the last check read-back
    std::string err;
};

namespace {

// Order the internal stream after the caller's stream (entry) and the
// caller's stream after the internal one (exit).
struct StreamJoin {
    gabp_batch *b;
    bool ok;
    explicit StreamJoin(gabp_batch *bb) : b(bb), ok(true) {
        ok = hipSetDevice(b->device) == hipSuccess &&
             hipEventRecord(b->ev_in, b->ustream) == hipSuccess &&
             hipStreamWaitEvent(b->stream, b->ev_in, 0) == hipSuccess;
    }
    ~StreamJoin() {
        if (hipEventRecord(b->ev_out, b->stream) == hipSuccess)
            (void)hipStreamWaitEvent(b->ustream, b->ev_out, 0);
    }
};

gabp_status bfail(gabp_batch *b, gabp_status st, const std::string &m) {
    if (b) b->err = m;
    else g_batch_create_error = m;
    return st;
}

#define BHIP(b, call)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            return bfail((b), GABP_E_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

constexpr int kBatchGrid = 256 * 32;  // persistent grid: ranges of work items per workgroup

int tiles_iter_of(const Lattice &L, int rpt) {
    return L.tiles_x * ((L.ny + 4 * rpt - 1) / (4 * rpt));
}

// lists staging / device layout: act[n] pprefix[n+1] frozen[n] gact[n] gpre[n+4]
// spre[n+1]
constexpr int lists_ints(int n) { return 6 * n + 6; }
constexpr int kStages = 4;
// the workspace's share, as the documented sizes have it
constexpr int lists_room(int n) { return 11 * n + 5; }
static_assert(lists_ints(1) <= lists_room(1), "lists fit their room from n = 1 on");
// flag region: div[n], t, err, mrel[n] (uint32), then cnt[n] (uint64, 8-aligned)
constexpr size_t flag_bytes(int n) { return 4 * (2 * (size_t)n + 2) + 4 + 8 * (size_t)n; }

// Region and iterations per launch of a group: deep_pick's rule on the tiles of
// all its instances together.
gabp::DeepPlan group_plan(const gabp_batch *b, int g, const std::vector<int> &members) {
    const int dt = b->dtype == GABP_F32 ? 0 : 1, alpha = (g & 1) + 1;
    int n;
    const gabp::DeepChoice *c = g < 2 ? gabp::full_choices(dt, alpha, n)
                                      : gabp::deep_choices(dt, alpha, n);
    for (int k = 0; k < n; ++k)
        for (int S = c[k].most; S >= c[k].least; --S) {
            int64_t tiles = 0;
            for (int i : members)
                tiles += gabp::deep_tiles(alpha, b->h[i].L.nx, b->h[i].L.ny, c[k].rw, c[k].rh, S);
            if (tiles <= b->cus) return {k, S};
        }
    return {n - 1, c[n - 1].bulk};
}

// A run of k iterations of a group: the first `iters` in `launches` launches of several
// iterations, the others singly.  Instances not frozen run at least the last one
// singly, so that they end on their two newest iterations in their two buffers (the
// freeze test needs that).  The launches have the parity of their iterations, so that
// an instance's state stays in the buffer its iteration number selects: one iteration
// more runs singly where that makes it so.  Launches of one iteration are left to
// the single kernel, whose tiles have no region around them; and four full iterations
// are three and a single one where they would be two and two: those read and write a
// region twice for what one iteration costs alone (1024^2 FP64, five iterations a call
// 459 -> 414 us; two of two took as long as four single ones).
struct Split {
    int iters = 0, launches = 0;
    // iterations that the tiles are for, the longest launch's: tiles for more have a
    // larger halo than it needs (four frozen iterations of 1024^2 FP32 in two launches
    // 144 -> 107 us, of 700 x 600 with 5 points in one 61 -> 60)
    int tile() const { return launches > 0 ? (iters + launches - 1) / launches : 1; }
};
Split split_run(int g, int k, int S) {
    int n = g < 2 ? k - 1 : k;
    if (n < 3) return {};
    auto launches = [&]() { return (n + S - 1) / S; };
    n -= (launches() ^ n) & 1;
    const int l = launches() + ((launches() ^ n) & 1);
    if (g < 2 && n == 4 && l == 2 && S >= 3) return {3, 1};
    return l < n ? Split{n, l} : Split{};
}

// Work lists of the running instances for a run of k iterations, if they are not
// up to date (host staging, then one copy into the device arrays).
gabp_status upload_lists(gabp_batch *b, int k) {
    bool same = !b->lists_dirty;
    for (int g = 0; g < 4; ++g) {
        const gabp_batch::Group &G = b->group[g];
        const Split q = split_run(g, k, G.plan.S);
        same = same && (G.n == 0 || q.launches == 0 || G.S == q.tile());
    }
    if (same) return GABP_OK;
    const int n = b->n;
    if (b->staged == kStages) {
        BHIP(b, hipStreamSynchronize(b->stream));
        b->staged = 0;
    }
    int *act = b->p_lists + (size_t)b->staged * lists_ints(n), *pp = act + n, *fz = pp + n + 1;
    int *gact = fz + n, *gpre = gact + n, *spre = gpre + n + 4;
    const int *lists = act;
    int na = 0, p = 0;
    std::vector<int> members[4];
    for (int i = 0; i < n; ++i) {
        InstHost &H = b->h[i];
        fz[i] = H.frozen ? 1 : 0;
        if (!H.running) continue;
        act[na] = i;
        pp[na++] = p;
        p += H.tiles_check;
        members[group_of(H, H.frozen)].push_back(i);
    }
    pp[na] = p;
    b->nact = na;
    b->ptotal = p;
    b->nu = (int)(members[0].size() + members[1].size());
    int off = 0, singles = 0;
    for (int g = 0; g < 4; ++g) {
        gabp_batch::Group &G = b->group[g];
        const int dt = b->dtype == GABP_F32 ? 0 : 1, alpha = (g & 1) + 1;
        int nc;
        const gabp::DeepChoice *c = g < 2 ? gabp::full_choices(dt, alpha, nc)
                                          : gabp::deep_choices(dt, alpha, nc);
        if (b->lists_dirty) G.plan = group_plan(b, g, members[g]);
        G.S = split_run(g, k, G.plan.S).tile();
        c += G.plan.region;
        G.off = off;
        G.n = (int)members[g].size();
        const int s0 = singles;
        G.items = 0;
        for (int q = 0; q < G.n; ++q) {
            const Lattice &L = b->h[members[g][q]].L;
            gact[off + q] = members[g][q];
            gpre[off + g + q] = G.items;
            G.items += (int)gabp::deep_tiles(alpha, L.nx, L.ny, c->rw, c->rh, G.S);
            spre[off + q] = singles;
            singles += tiles_iter_of(L, g < 2 ? b->rpt : 1);
        }
        gpre[off + g + G.n] = G.items;
        G.singles = singles - s0;
        off += G.n;
    }
    spre[off] = singles;
    // all lists are contiguous from d_act on
    BHIP(b, hipMemcpyAsync(b->d_act, lists, sizeof(int) * (size_t)lists_ints(n),
                           hipMemcpyHostToDevice, b->stream));
    ++b->staged;
    b->lists_dirty = false;
    return GABP_OK;
}

// Iteration t of groups g0 to g1 (both not frozen or both frozen), one launch.
template <typename T, int ALPHA>
void single_k(gabp_batch *b, int g0, int g1, int64_t t, double eta) {
    const gabp_batch::Group &G0 = b->group[g0], &G1 = b->group[g1];
    const int n = g0 == g1 ? G0.n : G0.n + G1.n;
    const unsigned items = (unsigned)(g0 == g1 ? G0.singles : G0.singles + G1.singles);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(items), dim3(256), 0, b->stream, b->d_inst,
                           b->d_gact + G0.off, b->d_spre + G0.off, n, (int)((t - 1) & 1),
                           (uint32_t)t, (T)eta, b->d_div);
    };
    if (g0 >= 2) go(gabp::k_batch_iter<T, 1, ALPHA, true>);
    else if (b->rpt == 1) go(gabp::k_batch_iter<T, 1, ALPHA, false>);
    else if (b->rpt == 2) go(gabp::k_batch_iter<T, 2, ALPHA, false>);
    else if (b->rpt == 4) go(gabp::k_batch_iter<T, 4, ALPHA, false>);
    else go(gabp::k_batch_iter<T, 8, ALPHA, false>);
}

// Iteration t of group g (5-point) and the one after it (13-point), as far as they are
// named: in one launch while its workgroups run at once (nine instances up to 150 x 120
// FP32 29 us, 35 in two), then each in one, with the registers of its own order only
// (2048 x 1024 of both orders 174 us in one, 141 in two).
gabp_status launch_single(gabp_batch *b, int g, bool five, bool thirteen, int64_t t, double eta) {
    const bool f32 = b->dtype == GABP_F32;
    if (five && thirteen && b->group[g].singles + b->group[g + 1].singles <= 4 * b->cus) {
        (f32 ? single_k<float, 0> : single_k<double, 0>)(b, g, g + 1, t, eta);
    } else {
        if (five) (f32 ? single_k<float, 1> : single_k<double, 1>)(b, g, g, t, eta);
        if (thirteen) (f32 ? single_k<float, 2> : single_k<double, 2>)(b, g + 1, g + 1, t, eta);
    }
    BHIP(b, hipGetLastError());
    return GABP_OK;
}

// n iterations of group g from iteration t in buffer `buf`, one launch.
template <typename T, int ALPHA, int RW, int RH>
void deep_k(gabp_batch *b, int g, int n, int buf, int64_t t, double eta) {
    const gabp_batch::Group &G = b->group[g];
    hipLaunchKernelGGL((gabp::k_batch_deep<T, ALPHA, RW, RH>), dim3((unsigned)G.items), dim3(1024),
                       0, b->stream, b->d_inst, b->d_gact + G.off, b->d_gpre + G.off + g, G.n,
                       G.S, n, buf, (uint32_t)t, (T)eta, b->d_div);
}

template <typename T, int ALPHA, int RW, int RH, int NT, bool SPLIT>
void full_k(gabp_batch *b, int g, int n, int buf, int64_t t, double eta) {
    const gabp_batch::Group &G = b->group[g];
    hipLaunchKernelGGL((gabp::k_batch_deep_full<T, ALPHA, RW, RH, NT, SPLIT>),
                       dim3((unsigned)G.items), dim3(NT), 0, b->stream, b->d_inst,
                       b->d_gact + G.off, b->d_gpre + G.off + g, G.n, G.S, n, buf,
                       (uint32_t)t, (T)eta, b->d_div);
}

gabp_status launch_group(gabp_batch *b, int g, int n, int buf, int64_t t, double eta) {
    const int region = b->group[g].plan.region;
    if (b->dtype == GABP_F32) {
        if (g == 0) (region == 0 ? full_k<float, 1, 32, 32, 1024, false> : full_k<float, 1, 64, 16, 1024, false>)(b, g, n, buf, t, eta);
        else if (g == 1) (region == 0 ? full_k<float, 2, 32, 32, 1024, false> : full_k<float, 2, 64, 16, 1024, false>)(b, g, n, buf, t, eta);
        else if (g == 2) (region == 0 ? deep_k<float, 1, 32, 32> : region == 1 ? deep_k<float, 1, 64, 32> : deep_k<float, 1, 64, 64>)(b, g, n, buf, t, eta);
        else (region == 0 ? deep_k<float, 2, 32, 32> : deep_k<float, 2, 64, 32>)(b, g, n, buf, t, eta);
    } else {
        if (g == 0) (region == 0 ? full_k<double, 1, 24, 24, 576, false> : region == 1 ? full_k<double, 1, 32, 32, 1024, false> : full_k<double, 1, 64, 32, 1024, false>)(b, g, n, buf, t, eta);
        else if (g == 1) (region == 0 ? full_k<double, 2, 32, 16, 512, false> : full_k<double, 2, 32, 24, 768, true>)(b, g, n, buf, t, eta);
        else if (g == 2) (region == 0 ? deep_k<double, 1, 32, 32> : deep_k<double, 1, 64, 32>)(b, g, n, buf, t, eta);
        else deep_k<double, 2, 32, 32>(b, g, n, buf, t, eta);
    }
    BHIP(b, hipGetLastError());
    return GABP_OK;
}

// Record a run of k iterations about to be applied to the running set.
void record_run(gabp_batch *b, int k, double eta) {
    BatchRun r;
    r.k = k;
    r.eta = eta;
    for (int g = 0; g < 4; ++g) {
        if (b->group[g].n == 0) continue;
        const Split q = split_run(g, k, b->group[g].plan.S);
        r.iters[g] = q.iters;
        r.deeps[g] = q.launches;
    }
    r.couples = b->group[2].n + b->group[3].n > 0 && k >= 5 ? (k - 1) / 4 : 0;
    r.t0.resize(b->n);
    r.frozen.resize(b->n);
    for (int i = 0; i < b->n; ++i) {
        r.t0[i] = b->h[i].running ? b->h[i].iters : -1;
        r.frozen[i] = b->h[i].frozen ? 1 : 0;
    }
    b->runs.push_back(std::move(r));
}

// Record and issue k iterations of the running set (on lists for them).
gabp_status run_iters(gabp_batch *b, int k, double eta) {
    gabp_status st = upload_lists(b, k);
    if (st != GABP_OK) return st;
    if (b->nact > 0 && k > 0) {
        record_run(b, k, eta);
        const BatchRun &r = b->runs.back();
        for (int g = 0; g < 4; ++g)
            for (int j = 0; j < r.deeps[g] && st == GABP_OK; ++j) {
                const int i0 = gabp::deep_part(r.iters[g], r.deeps[g], j);
                st = launch_group(b, g, gabp::deep_part(r.iters[g], r.deeps[g], j + 1) - i0,
                                  (int)((b->t + j) & 1), b->t + i0, eta);
            }
        for (int g : {0, 2}) {     // both prior orders, from where both go on singly
            const int i0 = b->group[g].n > 0 ? r.iters[g] : k;
            const int i1 = b->group[g + 1].n > 0 ? r.iters[g + 1] : k;
            for (int i = std::min(i0, i1); i < k && st == GABP_OK; ++i)
                st = launch_single(b, g, i >= i0, i >= i1, b->t + i + 1, eta);
        }
        if (st != GABP_OK) return st;
    }
    b->t += k;
    for (auto &H : b->h)
        if (H.running) {
            H.iters += k;
            if (k > 0) H.prev_valid = true;
        }
    return GABP_OK;
}

// Check of the running set: marginals with the freeze test of the instances not
// frozen (before t = 2 there is no previous iteration to compare with), residual
// partials, per-instance reduction and report to the pinned mirror.
gabp_status launch_check(gabp_batch *b) {
    if (b->nact == 0) return GABP_OK;
    const int grid = std::min(kBatchGrid, std::max(1, b->ptotal));
    const int post = grid + (b->t >= 2 ? b->nu * gabp::kProbeBlocks : 0);
    const int buf = (int)(b->t & 1);
    if (b->dtype == GABP_F32)
        hipLaunchKernelGGL((gabp::k_batch_post<float>), dim3(post), dim3(256), 0, b->stream,
                           b->d_inst, b->d_act, b->d_pprefix, b->nact, b->ptotal, b->d_frozen, buf,
                           grid, b->d_gact, (uint64_t)b->freeze_slots, b->d_cnt, b->d_mrel);
    else
        hipLaunchKernelGGL((gabp::k_batch_post<double>), dim3(post), dim3(256), 0, b->stream,
                           b->d_inst, b->d_act, b->d_pprefix, b->nact, b->ptotal, b->d_frozen, buf,
                           grid, b->d_gact, (uint64_t)b->freeze_slots, b->d_cnt, b->d_mrel);
    hipLaunchKernelGGL(gabp::k_batch_resid, dim3(grid), dim3(256), 0, b->stream, b->d_inst,
                       b->d_act, b->d_pprefix, b->nact, b->ptotal, b->d_partials);
    hipLaunchKernelGGL(gabp::k_batch_reduce, dim3(b->nact), dim3(256), 0, b->stream, b->d_act,
                       b->d_pprefix, b->d_partials, b->d_div, b->d_cnt, b->d_mrel, b->p_out,
                       b->p_div, b->p_cnt, b->p_mrel);
    BHIP(b, hipGetLastError());
    return GABP_OK;
}

// Instance i diverged at iteration t of run r.  The launch that met it left its
// input whole, and no later launch wrote, so the state that single launches (full
// iterations) or couples of two-iteration launches (information-only ones) would
// have kept is made from it by single iterations, recording into the batch's error
// word, which is cleared before each of them.
gabp_status hold_batch(gabp_batch *b, int i, const BatchRun &r, int64_t t) {
    InstHost &H = b->h[i];
    const bool frozen = r.frozen[i] != 0;
    const int g = group_of(H, frozen), dt = b->dtype == GABP_F32 ? 0 : 1;
    if (t - r.t0[i] > r.iters[g]) return GABP_OK;   // in a single iteration
    const int64_t want = held_after_batch_run(r.t0[i], frozen, r.couples, t).iter;
    int j = 0;
    while (r.t0[i] + gabp::deep_part(r.iters[g], r.deeps[g], j + 1) < t) ++j;
    int64_t it = r.t0[i] + gabp::deep_part(r.iters[g], r.deeps[g], j);
    H.dbuf = (int)((r.t0[i] + j) & 1);
    char *base = b->ws + H.base;
    const void *bw = base + (b->dtype == GABP_F32 ? H.lay.b_w : H.lay.b64);
    const void *ad = base + (b->dtype == GABP_F32 ? H.lay.adiag_w : H.lay.adiag64);
    for (; it < want; ++it, H.dbuf ^= 1) {
        const void *in = base + H.lay.msg[H.dbuf];
        void *out = base + H.lay.msg[H.dbuf ^ 1];
        BHIP(b, gabp::launch_set_u32(b->d_err, 0u, b->stream));
        BHIP(b, frozen ? gabp::launch_iter_theta(dt, 1, H.L, in, out, base + H.lay.gain, bw,
                                                 r.eta, b->d_err, b->d_t, (uint32_t)(it + 1),
                                                 b->stream)
                       : gabp::launch_iter(dt, 1, H.L, in, out, ad, bw, r.eta, b->d_err,
                                           b->d_t, (uint32_t)(it + 1), b->stream));
    }
    H.iters = it;
    return GABP_OK;
}

}  // namespace

extern "C" {

const char *gabp_batch_last_error(const gabp_batch *b) {
    return b ? b->err.c_str() : g_batch_create_error.c_str();
}

void gabp_batch_destroy(gabp_batch *b) {
    if (!b) return;
    (void)hipSetDevice(b->device);
    if (b->stream) (void)hipStreamSynchronize(b->stream);
    if (b->own_ws && b->ws) (void)hipFree(b->ws);
    if (b->p_out) (void)hipHostFree(b->p_out);
    if (b->ev_in) (void)hipEventDestroy(b->ev_in);
    if (b->ev_out) (void)hipEventDestroy(b->ev_out);
    if (b->stream) (void)hipStreamDestroy(b->stream);
    delete b;
}

static gabp_status batch_layout(int32_t n, const gabp_instance *inst, int32_t dtype,
                                std::vector<InstHost> *hs, size_t *tables_off, size_t *total,
                                size_t *partial_cap, std::string &why) {
    if (n < 1 || !inst) return why = "need n >= 1 instances", GABP_E_INVALID;
    const size_t es = dtype == GABP_F32 ? 4 : 8;
    size_t off = 0, pc = 0;
    if (hs) hs->assign((size_t)n, InstHost());
    for (int i = 0; i < n; ++i) {
        std::string w;
        gabp_status st = check_grid_stencil(&inst[i].grid, &inst[i].stencil, dtype, w);
        if (st != GABP_OK) return why = "instance " + std::to_string(i) + ": " + w, st;
        const int deg = inst[i].stencil.alpha == 1 ? 4 : 12;
        Layout lay = make_layout(inst[i].grid.nx, inst[i].grid.ny, deg, es, dtype == GABP_F32);
        Lattice L = make_lattice(&inst[i].grid, &inst[i].stencil, lay);
        const int tc = L.tiles_x * ((L.ny + 3) / 4);
        pc += (size_t)tc;
        if (hs) {
            InstHost &H = (*hs)[(size_t)i];
            H.L = L;
            H.dtype = dtype;
            H.lay = lay;
            H.base = off;
            H.tiles_check = tc;
        }
        off = round_up(off + lay.total, kAlign);
    }
    *tables_off = off;
    // instance table, int lists, flag arrays (divergence, counter, error and
    // largest precision changes as uint32, then 64-bit change counts),
    // partials, and 2 n doubles more, as the documented sizes have it
    off = round_up(off + sizeof(BatchInst) * (size_t)n, kAlign);
    off = round_up(off + sizeof(int) * (size_t)lists_room(n), kAlign);
    off = round_up(off + flag_bytes(n), kAlign);
    off = round_up(off + sizeof(double) * 2 * pc, kAlign);
    off = round_up(off + sizeof(double) * 2 * (size_t)n, kAlign);
    *total = off;
    *partial_cap = pc;
    return GABP_OK;
}

gabp_status gabp_batch_workspace_size(int32_t n, const gabp_instance *inst, int32_t dtype,
                                      size_t *bytes) {
    std::string why;
    size_t toff = 0, total = 0, pc = 0;
    gabp_status st = batch_layout(n, inst, dtype, nullptr, &toff, &total, &pc, why);
    if (st != GABP_OK) return bfail(nullptr, st, why);
    if (!bytes) return bfail(nullptr, GABP_E_INVALID, "bytes is NULL");
    *bytes = total;
    return GABP_OK;
}

gabp_status gabp_batch_create(int32_t n, const gabp_instance *inst, const gabp_opts *opts,
                              gabp_batch **out) {
    if (!out) return bfail(nullptr, GABP_E_INVALID, "out is NULL");
    *out = nullptr;
    const int32_t dtype = opts ? opts->dtype : GABP_F32;
    if (opts && opts->prior_mean)
        return bfail(nullptr, GABP_E_INVALID, "batched instances take no prior mean");
    std::vector<InstHost> hs;
    std::string why;
    size_t toff = 0, total = 0, pc = 0;
    gabp_status st = batch_layout(n, inst, dtype, &hs, &toff, &total, &pc, why);
    if (st != GABP_OK) return bfail(nullptr, st, why);
    for (int i = 0; i < n; ++i) {
        const gabp_obs &o = inst[i].obs;
        const gabp_noise &nz = inst[i].noise;
        const int64_t N = inst[i].grid.nx * inst[i].grid.ny;
        if (!nz.var && (!(nz.sigma > 0) || !std::isfinite(nz.sigma)))
            return bfail(nullptr, GABP_E_INVALID, "instance " + std::to_string(i) + ": sigma must be positive");
        if (o.n < 0 || (o.n > 0 && (!o.cell || !o.y)))
            return bfail(nullptr, GABP_E_INVALID, "instance " + std::to_string(i) + ": bad observations");
        if (o.n > 0 && !o.on_device)
            for (int64_t k = 0; k < o.n; ++k)
                if (o.cell[k] < 0 || o.cell[k] >= N || !std::isfinite(o.y[k]) ||
                    (nz.var && !(nz.var[k] > 0)))
                    return bfail(nullptr, GABP_E_INVALID, "instance " + std::to_string(i) +
                                                              ": invalid observation " + std::to_string(k));
    }
    gabp_batch *b = new (std::nothrow) gabp_batch();
    if (!b) return bfail(nullptr, GABP_E_NOMEM, "host allocation failed");
    auto bail = [&](gabp_status s2) {
        g_batch_create_error = b->err;
        gabp_batch_destroy(b);
        return s2;
    };
    b->n = n;
    b->dtype = dtype;
    b->esize = dtype == GABP_F32 ? 4 : 8;
    b->h = hs;
    b->partial_cap = pc;
    if (hipGetDevice(&b->device) != hipSuccess) {
        b->err = "no HIP device";
        return bail(GABP_E_DEVICE);
    }
    if (hipDeviceGetAttribute(&b->cus, hipDeviceAttributeMultiprocessorCount, b->device) !=
        hipSuccess)
        b->cus = 256;
    b->ustream = opts ? (hipStream_t)opts->stream : nullptr;
    if (hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&b->ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&b->ev_out, hipEventDisableTiming) != hipSuccess) {
        b->err = "creating the batch stream or events failed";
        return bail(GABP_E_DEVICE);
    }
    // the internal stream starts after everything already queued on the
    // caller's stream (e.g. the observation arrays' uploads)
    if (hipEventRecord(b->ev_in, b->ustream) != hipSuccess ||
        hipStreamWaitEvent(b->stream, b->ev_in, 0) != hipSuccess) {
        b->err = "ordering the batch stream failed";
        return bail(GABP_E_DEVICE);
    }
    if (opts && opts->workspace) {
        if (opts->workspace_bytes < total) {
            b->err = "workspace too small: " + std::to_string(total) + " bytes needed";
            return bail(GABP_E_NOMEM);
        }
        if (((uintptr_t)opts->workspace) % kAlign != 0) {
            b->err = "workspace must be 256-byte aligned";
            return bail(GABP_E_INVALID);
        }
        b->ws = (char *)opts->workspace;
        b->ws_bytes = opts->workspace_bytes;
    } else {
        if (hipMalloc((void **)&b->ws, total) != hipSuccess) {
            b->ws = nullptr;
            b->err = "hipMalloc of the batch workspace failed";
            return bail(GABP_E_NOMEM);
        }
        b->own_ws = true;
        b->ws_bytes = total;
    }
    // device tables
    size_t off = toff;
    b->d_inst = (BatchInst *)(b->ws + off);
    off = round_up(off + sizeof(BatchInst) * (size_t)n, kAlign);
    b->d_act = (int *)(b->ws + off);
    b->d_pprefix = b->d_act + n;
    b->d_frozen = b->d_pprefix + n + 1;
    b->d_gact = b->d_frozen + n;
    b->d_gpre = b->d_gact + n;
    b->d_spre = b->d_gpre + n + 4;
    off = round_up(off + sizeof(int) * (size_t)lists_room(n), kAlign);
    b->d_div = (uint32_t *)(b->ws + off);
    b->d_t = b->d_div + n;
    b->d_err = b->d_t + 1;
    b->d_mrel = b->d_err + 1;
    b->d_cnt = (unsigned long long *)(b->ws + round_up(off + sizeof(uint32_t) * (size_t)(2 * n + 2), 8));
    off = round_up(off + flag_bytes(n), kAlign);
    b->d_partials = (double *)(b->ws + off);
    // pinned mirror: out[2n], cnt[n], div[n], mrel[n], t, lists
    const size_t pin_bytes = sizeof(double) * 2 * (size_t)n + sizeof(unsigned long long) * (size_t)n +
                             sizeof(uint32_t) * (2 * (size_t)n + 2) +
                             sizeof(int) * (size_t)lists_ints(n) * kStages + 64;
    if (hipHostMalloc((void **)&b->p_out, pin_bytes, hipHostMallocDefault) != hipSuccess) {
        b->p_out = nullptr;
        b->err = "pinned host allocation failed";
        return bail(GABP_E_NOMEM);
    }
    b->p_cnt = (unsigned long long *)(b->p_out + 2 * n);
    b->p_div = (uint32_t *)(b->p_cnt + n);
    b->p_mrel = b->p_div + n;
    b->p_t = b->p_mrel + n;
    b->p_lists = (int *)(b->p_t + 2);
    if (hipMemsetAsync(b->ws, 0, total, b->stream) != hipSuccess) {
        b->err = "hipMemsetAsync failed";
        return bail(GABP_E_DEVICE);
    }
    // instance records and per-instance set-up; an instance whose cells repeat out
    // of order raises its word of d_div and is set up again: where its observations
    // are staged here, at once (the staging waits for the stream in any case), else
    // when the words are looked at together
    std::vector<BatchInst> rec((size_t)n);
    for (int i = 0; i < n; ++i) {
        InstHost &H = b->h[i];
        char *base = b->ws + H.base;
        BatchInst &R = rec[(size_t)i];
        R.L = H.L;
        R.msg[0] = base + H.lay.msg[0];
        R.msg[1] = base + H.lay.msg[1];
        R.gain = base + H.lay.gain;
        R.adiag64 = (double *)(base + H.lay.adiag64);
        R.b64 = (double *)(base + H.lay.b64);
        R.mu64 = (double *)(base + H.lay.mu64);
        R.bel64 = (double *)(base + H.lay.bel64);
        R.adiag_w = dtype == GABP_F32 ? (const void *)(base + H.lay.adiag_w) : (const void *)R.adiag64;
        R.b_w = dtype == GABP_F32 ? (const void *)(base + H.lay.b_w) : (const void *)R.b64;
    }
    auto setup = [&](int i, uint32_t *repeated) -> gabp_status {
        InstHost &H = b->h[i];
        char *base = b->ws + H.base;
        BatchInst &R = rec[(size_t)i];
        const gabp_obs &o = inst[i].obs;
        const gabp_noise &nz = inst[i].noise;
        int64_t *tc = nullptr;
        double *ty = nullptr, *tv = nullptr;
        const int64_t *dc = o.cell;
        const double *dy = o.y, *dv = nz.var;
        if (o.n > 0 && !o.on_device) {
            bool ok = hipMalloc((void **)&tc, o.n * sizeof(int64_t)) == hipSuccess &&
                      hipMalloc((void **)&ty, o.n * sizeof(double)) == hipSuccess &&
                      (!nz.var || hipMalloc((void **)&tv, o.n * sizeof(double)) == hipSuccess) &&
                      hipMemcpyAsync(tc, o.cell, o.n * sizeof(int64_t), hipMemcpyHostToDevice, b->stream) == hipSuccess &&
                      hipMemcpyAsync(ty, o.y, o.n * sizeof(double), hipMemcpyHostToDevice, b->stream) == hipSuccess &&
                      (!nz.var || hipMemcpyAsync(tv, nz.var, o.n * sizeof(double), hipMemcpyHostToDevice, b->stream) == hipSuccess);
            if (!ok) {
                (void)hipStreamSynchronize(b->stream);
                (void)hipFree(tc);
                (void)hipFree(ty);
                (void)hipFree(tv);
                b->err = "staging observations failed";
                return GABP_E_NOMEM;
            }
            dc = tc;
            dy = ty;
            dv = tv;
        }
        auto terms = [&](uint32_t *rep) {
            return gabp::launch_setup(dtype == GABP_F32 ? 0 : 1, H.L, o.n, dc, dy, dv,
                                      nz.var ? 0.0 : nz.sigma * nz.sigma, R.adiag64, R.b64, nullptr,
                                      dtype == GABP_F32 ? base + H.lay.adiag_w : nullptr,
                                      dtype == GABP_F32 ? base + H.lay.b_w : nullptr, b->d_err, rep,
                                      R.mu64, H.lay.check_room(), b->stream);
        };
        hipError_t e = terms(repeated);
        if (e == hipSuccess && tc && repeated) {
            e = hipMemcpyAsync(b->p_div + i, repeated, sizeof(uint32_t), hipMemcpyDeviceToHost,
                               b->stream);
            const hipError_t es = hipStreamSynchronize(b->stream);
            if (e == hipSuccess) e = es;
            if (e == hipSuccess && b->p_div[i] != 0u) {
                e = terms(nullptr);
                if (e == hipSuccess) e = gabp::launch_set_u32(repeated, 0u, b->stream);
            }
        }
        if (tc || ty || tv) {
            (void)hipStreamSynchronize(b->stream);
            (void)hipFree(tc);
            (void)hipFree(ty);
            (void)hipFree(tv);
        }
        if (e != hipSuccess) {
            b->err = std::string("setup failed: ") + hipGetErrorString(e);
            return GABP_E_DEVICE;
        }
        return GABP_OK;
    };
    for (int i = 0; i < n; ++i) {
        const gabp_status s2 = setup(i, b->d_div + i);
        if (s2 != GABP_OK) return bail(s2);
    }
    if (hipMemcpyAsync(b->d_inst, rec.data(), sizeof(BatchInst) * (size_t)n, hipMemcpyHostToDevice,
                       b->stream) != hipSuccess ||
        hipMemcpyAsync(b->p_div, b->d_div, sizeof(uint32_t) * (size_t)n, hipMemcpyDeviceToHost,
                       b->stream) != hipSuccess ||
        hipMemcpyAsync(b->p_t, b->d_err, sizeof(uint32_t), hipMemcpyDeviceToHost, b->stream) != hipSuccess ||
        hipStreamSynchronize(b->stream) != hipSuccess) {
        b->err = "uploading the instance table failed";
        return bail(GABP_E_DEVICE);
    }
    bool again = false;
    for (int i = 0; i < n; ++i) {
        if (b->p_div[i] == 0u) continue;
        again = true;
        const gabp_status s2 = setup(i, nullptr);
        if (s2 != GABP_OK) return bail(s2);
    }
    if (again &&
        (hipMemsetAsync(b->d_div, 0, sizeof(uint32_t) * (size_t)n, b->stream) != hipSuccess ||
         hipMemcpyAsync(b->p_t, b->d_err, sizeof(uint32_t), hipMemcpyDeviceToHost, b->stream) != hipSuccess ||
         hipStreamSynchronize(b->stream) != hipSuccess)) {
        b->err = "setting an instance up again failed";
        return bail(GABP_E_DEVICE);
    }
    if (b->p_t[0] != 0u) {
        b->err = "invalid observation (cell out of range, non-finite value or non-positive variance)";
        return bail(GABP_E_INVALID);
    }
    if (upload_lists(b, 0) != GABP_OK) return bail(GABP_E_DEVICE);
    *out = b;
    return GABP_OK;   // create synchronised the internal stream
}

gabp_status gabp_batch_iterate(gabp_batch *b, int32_t n_iters, double damping) {
    if (!b) return GABP_E_INVALID;
    StreamJoin join(b);
    if (!join.ok) return bfail(b, GABP_E_DEVICE, "stream ordering failed");
    if (n_iters < 0 || !(damping > 0.0) || !(damping <= 1.0))
        return bfail(b, GABP_E_INVALID, "need n_iters >= 0 and damping in (0, 1]");
    return run_iters(b, n_iters, damping);
}

// Fold one check's report into the per-instance state.  `changed`: the running
// set (or a frozen flag) did.
static gabp_status fold_check(gabp_batch *b, double rel_tol, bool &changed) {
    changed = false;
    for (int i = 0; i < b->n; ++i) {
        InstHost &H = b->h[i];
        if (!H.running) continue;
        if (b->p_div[i] != 0u) {
            const int64_t t = (int64_t)b->p_div[i];
            H.running = false;
            H.status = GABP_E_DIVERGED;
            H.diverged_at = t;
            H.iters = t;
            H.dbuf = (int)(t & 1);
            // the kept messages are those of the launch that diverged
            for (const BatchRun &r : b->runs) {
                if (r.t0[i] < 0 || t <= r.t0[i] || t > r.t0[i] + r.k) continue;
                const gabp_status st = hold_batch(b, i, r, t);
                if (st != GABP_OK) return st;
                break;
            }
            changed = true;
            continue;
        }
        const double a = std::sqrt(b->p_out[2 * i]), bb = std::sqrt(b->p_out[2 * i + 1]);
        const double rel = bb > 0 ? a / bb : a;
        H.rel = rel;
        if (!std::isfinite(rel) || (H.first_rel > 0 && rel > 1e3 * H.first_rel)) {
            H.running = false;
            H.status = GABP_E_DIVERGED;
            changed = true;
            continue;
        }
        if (H.first_rel < 0) H.first_rel = rel;
        if (rel <= rel_tol) {
            H.running = false;
            H.status = GABP_OK;
            changed = true;
            continue;
        }
        if (!H.frozen && H.prev_valid && H.iters >= 2 &&
            freeze_now(b->p_cnt[i], b->p_mrel[i], b->freeze_slots, b->freeze_rel)) {
            H.frozen = true;
            H.frozen_at = H.iters;
            changed = true;
        }
    }
    return GABP_OK;
}

gabp_status gabp_batch_solve(gabp_batch *b, int64_t max_iters, double damping, double rel_tol,
                             int32_t check_every, int64_t *iters_done, double *rel_residual,
                             int32_t *status) {
    if (!b) return GABP_E_INVALID;
    StreamJoin join(b);
    if (!join.ok) return bfail(b, GABP_E_DEVICE, "stream ordering failed");
    if (max_iters < 0 || check_every == 0 || !(rel_tol >= 0) || !(damping > 0.0) ||
        !(damping <= 1.0))
        return bfail(b, GABP_E_INVALID, "need max_iters >= 0, check_every != 0, rel_tol >= 0, damping in (0, 1]");
    // check_every < 0: adaptive chunks, as gabp_solve's, on the slowest
    // running instance; powers of two times |check_every|, at most kMaxChunk,
    // as there
    constexpr int kMaxChunk = 1280;
    const bool adaptive = check_every < 0;
    const int kmin = adaptive ? -check_every : check_every;
    int next = kmin;
    int64_t run = 0;
    while (run < max_iters) {
        const int k = (int)std::min<int64_t>(next, max_iters - run);
        gabp_status st = upload_lists(b, k);
        if (st != GABP_OK) return st;
        if (b->nact == 0) break;
        st = run_iters(b, k, damping);
        if (st != GABP_OK) return st;
        run += k;
        st = launch_check(b);
        if (st != GABP_OK) return st;
        BHIP(b, hipStreamSynchronize(b->stream));
        b->staged = 0;
        bool changed;
        const bool testing = b->nu > 0;
        st = fold_check(b, rel_tol, changed);
        if (st != GABP_OK) return st;
        b->runs.clear();
        if (testing) {
            for (int i = 0; i < b->n; ++i) {
                InstHost &H = b->h[i];
                if (H.frozen && H.frozen_at == H.iters) {
                    char *base = b->ws + H.base;
                    BHIP(b, gabp::launch_gain(b->dtype == GABP_F32 ? 0 : 1, H.L,
                                              base + H.lay.msg[H.iters & 1],
                                              b->dtype == GABP_F32 ? (void *)(base + H.lay.adiag_w)
                                                                   : (void *)(base + H.lay.adiag64),
                                              base + H.lay.gain, b->stream));
                    // frozen within the tolerance: both buffers get the
                    // precision messages the gains come from
                    if (b->p_cnt[i] != 0u)
                        BHIP(b, hipMemcpyAsync(base + H.lay.msg[(H.iters - 1) & 1],
                                               base + H.lay.msg[H.iters & 1],
                                               (size_t)H.L.deg * (size_t)H.L.plane *
                                                   (b->dtype == GABP_F32 ? sizeof(float)
                                                                         : sizeof(double)),
                                               hipMemcpyDeviceToDevice, b->stream));
                }
            }
        }
        if (changed) b->lists_dirty = true;
        next = kmin;
        if (adaptive) {
            double want = (double)kMaxChunk;
            for (auto &H : b->h) {
                if (!H.running) continue;
                double ki = kmin;
                if (H.frozen && H.prev_rel > 0 && H.rel < H.prev_rel && H.rel > 0 &&
                    H.iters > H.prev_iters) {
                    const double rate = std::log(H.rel / H.prev_rel) / (double)(H.iters - H.prev_iters);
                    ki = 0.5 * std::log(rel_tol / H.rel) / rate;
                }
                want = std::min(want, ki);
            }
            while (next * 2 <= kMaxChunk && next * 2 <= want) next *= 2;
        }
        for (auto &H : b->h)
            if (H.running) {
                H.prev_rel = H.rel;
                H.prev_iters = H.iters;
            }
    }
    for (int i = 0; i < b->n; ++i) {
        const InstHost &H = b->h[i];
        if (iters_done) iters_done[i] = H.iters;
        if (rel_residual) rel_residual[i] = H.rel;
        if (status) status[i] = H.running ? GABP_E_NOT_CONVERGED : H.status;
    }
    bool all_ok = true;
    for (const auto &H : b->h) all_ok = all_ok && !H.running && H.status == GABP_OK;
    return all_ok ? GABP_OK : GABP_E_NOT_CONVERGED;
}

gabp_status gabp_batch_posterior(gabp_batch *b, int32_t i, double *mean, double *var) {
    if (!b || i < 0 || i >= b->n) return GABP_E_INVALID;
    StreamJoin join(b);
    if (!join.ok) return bfail(b, GABP_E_DEVICE, "stream ordering failed");
    const InstHost &H = b->h[i];
    char *base = b->ws + H.base;
    BHIP(b, gabp::launch_post(b->dtype == GABP_F32 ? 0 : 1, H.L, base + H.lay.msg[state_buf(H)],
                              (const double *)(base + H.lay.adiag64), (const double *)(base + H.lay.b64),
                              H.frozen ? (const double *)(base + H.lay.bel64) : nullptr, nullptr, mean,
                              var, nullptr, b->stream));
    return GABP_OK;
}

gabp_status gabp_batch_get_messages(gabp_batch *b, int32_t i, void *prec, void *info) {
    if (!b || i < 0 || i >= b->n) return GABP_E_INVALID;
    StreamJoin join(b);
    if (!join.ok) return bfail(b, GABP_E_DEVICE, "stream ordering failed");
    const InstHost &H = b->h[i];
    char *base = b->ws + H.base;
    BHIP(b, gabp::launch_msgs_get(b->dtype == GABP_F32 ? 0 : 1, H.L, base + H.lay.msg[state_buf(H)],
                                  prec, info, b->stream));
    return GABP_OK;
}

gabp_status gabp_batch_log_precisions(gabp_batch *b, int32_t i, float *lam, float *valid) {
    if (!b) return GABP_E_INVALID;
    if (i < 0 || i >= b->n || !lam) return bfail(b, GABP_E_INVALID, "need 0 <= i < n and lam");
    StreamJoin join(b);
    if (!join.ok) return bfail(b, GABP_E_DEVICE, "stream ordering failed");
    const InstHost &H = b->h[i];
    char *base = b->ws + H.base;
    BHIP(b, gabp::launch_log_prec(b->dtype == GABP_F32 ? 0 : 1, H.L, base + H.lay.msg[state_buf(H)],
                                  lam, valid, b->stream));
    return GABP_OK;
}

gabp_status gabp_batch_warm_init(gabp_batch *b, int32_t i, const float *pred,
                                 int32_t keep_precisions) {
    if (!b) return GABP_E_INVALID;
    if (i < 0 || i >= b->n || !pred) return bfail(b, GABP_E_INVALID, "need 0 <= i < n and a pred");
    StreamJoin join(b);
    if (!join.ok) return bfail(b, GABP_E_DEVICE, "stream ordering failed");
    InstHost &H = b->h[i];
    if (H.status == GABP_E_DIVERGED) return bfail(b, GABP_E_DIVERGED, "instance has diverged");
    char *base = b->ws + H.base;
    BHIP(b, gabp::launch_warm_init(b->dtype == GABP_F32 ? 0 : 1, H.L, pred, keep_precisions ? 1 : 0,
                                   base + H.lay.msg[state_buf(H)], b->stream));
    H.prev_valid = false;
    if (H.frozen) b->lists_dirty = true;
    H.frozen = false;
    H.frozen_at = -1;
    return GABP_OK;
}

gabp_status gabp_batch_upscale_precisions(gabp_batch *b, int32_t i, float *pred, int64_t nxf,
                                          int64_t nyf, double scale) {
    if (!b) return GABP_E_INVALID;
    if (i < 0 || i >= b->n || !pred) return bfail(b, GABP_E_INVALID, "need 0 <= i < n and a pred");
    const InstHost &H = b->h[i];
    if (nxf < 1 || nyf < 1 || (nxf + 1) / 2 != H.L.nx || (nyf + 1) / 2 != H.L.ny)
        return bfail(b, GABP_E_INVALID,
                     "upscale_precisions: need ceil(nxf / 2) = nx and ceil(nyf / 2) = ny of the instance");
    if (!(scale > 0.0) || !std::isfinite(scale))
        return bfail(b, GABP_E_INVALID, "upscale_precisions: scale must be finite and > 0");
    StreamJoin join(b);
    if (!join.ok) return bfail(b, GABP_E_DEVICE, "stream ordering failed");
    char *base = b->ws + H.base;
    BHIP(b, gabp::launch_upscale_prec(b->dtype == GABP_F32 ? 0 : 1, H.L,
                                      base + H.lay.msg[state_buf(H)], (float)scale, pred, (int)nxf,
                                      (int)nyf, b->stream));
    return GABP_OK;
}

gabp_status gabp_batch_set_freeze_tolerance(gabp_batch *b, int64_t max_slots, double max_rel) {
    if (!b) return GABP_E_INVALID;
    if (max_slots < 0 || !(max_rel >= 0.0) || !std::isfinite(max_rel))
        return bfail(b, GABP_E_INVALID, "need max_slots >= 0 and a finite max_rel >= 0");
    b->freeze_slots = max_slots;
    b->freeze_rel = max_rel;
    return GABP_OK;
}

gabp_status gabp_batch_autotune(gabp_batch *b, int32_t trials, double damping, int32_t *chosen) {
    if (!b || trials < 1) return GABP_E_INVALID;
    StreamJoin join(b);
    if (!join.ok) return bfail(b, GABP_E_DEVICE, "stream ordering failed");
    hipEvent_t e0, e1;
    BHIP(b, hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return bfail(b, GABP_E_DEVICE, "hipEventCreate failed");
    }
    float best = INFINITY;
    int best_r = b->rpt;
    gabp_status st = gabp_batch_iterate(b, 1, damping);
    for (int pass = 0; pass < 2 && st == GABP_OK; ++pass)
        for (int r : gabp::kRptChoices) {
            b->rpt = r;
            b->lists_dirty = true;   // work-item counts depend on the tile shape
            st = upload_lists(b, 1);
            if (st != GABP_OK) break;
            if (hipEventRecord(e0, b->stream) != hipSuccess) { st = GABP_E_DEVICE; break; }
            // one at a time: only single iterations of instances not frozen have
            // rows per thread
            for (int k = 0; k < trials && st == GABP_OK; ++k) st = run_iters(b, 1, damping);
            if (st != GABP_OK) break;
            float ms = 0.f;
            if (hipEventRecord(e1, b->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { st = GABP_E_DEVICE; break; }
            if (b->nu > 0 && ms < best) {
                best = ms;
                best_r = r;
            }
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    b->rpt = best_r;
    b->lists_dirty = true;
    if (st != GABP_OK) return st == GABP_E_DEVICE ? bfail(b, st, "autotune timing failed") : st;
    if (chosen) *chosen = best_r;
    return GABP_OK;
}

gabp_status gabp_batch_info(const gabp_batch *b, int32_t i, int64_t *iters, int64_t *frozen_at,
                            int32_t *running) {
    if (!b || i < 0 || i >= b->n) return GABP_E_INVALID;
    const InstHost &H = b->h[i];
    if (iters) *iters = H.iters;
    if (frozen_at) *frozen_at = H.frozen ? H.frozen_at : -1;
    if (running) *running = H.running ? 1 : 0;
    return GABP_OK;
}

}  // extern "C"
