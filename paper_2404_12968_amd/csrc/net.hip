// Learned warm start: the kernels of a small 3x3 convolutional network that
// predicts posterior means and message precisions from the observations,
// trained on solutions the solver itself produced, and the message
// initialisation that turns a prediction into a starting state.
//
// Tensors: activations NHWC in BF16 ([B][H][W][C], C in {16, 32}); weights
// [32][9*Cin] BF16 with k = tap * Cin + ci, tap = 3 * (dy + 1) + (dx + 1)
// (rows beyond the layer's output channels are zero); FP32 biases, FP32
// master weights and FP32 gradients.
//
// The convolutions are implicit GEMMs on the gfx950 matrix cores
// (v_mfma_f32_32x32x16_bf16: BF16 operands, FP32 accumulation).  Operand
// layout of that instruction (A: 32 x 16, B: 16 x 32, D: 32 x 32): lane l
// holds A[l % 32][8 (l / 32) + j] and B[8 (l / 32) + j][l % 32] for j < 8,
// and D[8 i + 4 (l / 32) + j][l % 32] in accumulator 4 i + j.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>
#include <string>

#include "gabp.h"
#include "internal.h"
#include "lattice.h"
#include "numerics.h"

namespace gabp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ bf16x8 zero_bf16x8() {
    bf16x8 z;
#pragma unroll
    for (int j = 0; j < 8; ++j) z[j] = (__bf16)0.0f;
    return z;
}

// A workgroup barrier that waits for the wave's LDS accesses but not for its
// loads from memory (which __syncthreads would), so that loads issued ahead
// stay in flight across it.  Orders LDS contents only.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A raw buffer resource over [base, base + bytes), bytes below 2^30: loads at an
// offset past its end (an invalid lane passes kOut) return zero and touch no
// memory.
constexpr int kOut = 1 << 30;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_of(const void *base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, bytes, 0x00020000);
}

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;

__device__ __forceinline__ bf16x8 load_bf16x8(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// A persistent grid's walk over row segments (n of them, spr to a row, H rows to
// an image), PER at a time (this one the sub-th): each XCD takes one
// contiguous run, which its workgroups walk side by side, so that the rows a
// segment shares with those above and below it are in that XCD's L2 from
// about the same time (k_conv_rows, 1024 x 1024 pixels: 34.8 us against 43.0 with a
// contiguous run per workgroup, which re-reads the other two tap rows from
// beyond L2).
template <int PER>
struct RowWalk {
    long t, t1, row;   // segment, end of the run, image row over the batch
    int sx, y;         // segment within the row, row within the image
    int nl, drow, dsx;
    __device__ __forceinline__ RowWalk(long n, int spr, int H, int sub) {
        const int nb = (int)gridDim.x, nx = min(8, nb);
        const int xcd = (int)blockIdx.x % nx, local = (int)blockIdx.x / nx;
        nl = (nb - xcd + nx - 1) / nx * PER;
        if (n < (1L << 30)) {   // 32-bit divisions: the 64-bit ones cost a small launch about 1 us
            const unsigned len = (unsigned)n / (unsigned)nx, more = (unsigned)n % (unsigned)nx;
            const unsigned t0 = len * (unsigned)xcd + min((unsigned)xcd, more);
            const unsigned at = t0 + (unsigned)(local * PER + sub), r = at / (unsigned)spr;
            t1 = t0 + len + ((unsigned)xcd < more ? 1u : 0u);
            t = at;
            row = r;
            sx = (int)(at - r * (unsigned)spr);
            y = (int)(r % (unsigned)H);
        } else {
            t = xcd * n / nx + local * PER + sub;
            t1 = (xcd + 1) * n / nx;
            row = t / spr;
            sx = (int)(t - row * spr);
            y = (int)(row % H);
        }
        drow = nl / spr;
        dsx = nl - drow * spr;
    }
    __device__ __forceinline__ void next(int spr, int H) {
        t += nl;
        int dr = drow;
        sx += dsx;
        if (sx >= spr) {
            sx -= spr;
            ++dr;
        }
        row += dr;
        y += dr;
        while (y >= H) y -= H;
    }
};

// Bias, activation and stores of one 32-pixel tile: this lane's pixel starts at
// element o, its accumulators hold channels 8 i + 4 kh + j (4 i + j).
template <int COUT>
__device__ __forceinline__ void conv_store(const f32x16 &acc, const float *bl, int relu, int kh,
                                           bool here, size_t o, __bf16 *__restrict__ yb,
                                           float *__restrict__ yf) {
    float v[COUT / 2];
#pragma unroll
    for (int i = 0; i < COUT / 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float q = acc[4 * i + j] + bl[8 * i + 4 * kh + j];
            if (relu) q = q > 0.0f ? q : 0.0f;
            v[4 * i + j] = q;              // channel 8 i + 4 kh + j
        }
    if (yf && here) {
#pragma unroll
        for (int i = 0; i < COUT / 8; ++i)
            *(float4 *)(yf + o + 8 * i + 4 * kh) =
                make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    }
    if (yb) {
        // groups i < COUT / 16 to lanes 0..31, the rest to lanes 32..63:
        // after the swap a lane holds channels 8 g .. 8 g + 7 of its pixel
        // for g = i + kh COUT / 16
        uint32_t q[COUT / 8][2];
#pragma unroll
        for (int i = 0; i < COUT / 8; ++i) {
            bf16x4 pk;
#pragma unroll
            for (int j = 0; j < 4; ++j) pk[j] = (__bf16)v[4 * i + j];
            __builtin_memcpy(q[i], &pk, 8);
        }
#pragma unroll
        for (int i = 0; i < COUT / 16; ++i) {
            const auto s0 = __builtin_amdgcn_permlane32_swap(q[i][0], q[i + COUT / 16][0],
                                                             false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(q[i][1], q[i + COUT / 16][1],
                                                             false, false);
            u32x4 out = {s0[0], s1[0], s0[1], s1[1]};
            if (here) *(u32x4 *)(yb + o + 8 * i + kh * (COUT / 2)) = out;
        }
    }
}

// --------------------------------------------------------------------------
// Convolution, forward: y[p][co] = act(bias[co] + sum_{tap, ci}
// w[co][tap][ci] x[p + dil * off(tap)][ci]), zero padding.  M = output
// channel (32 weight rows), N = 32 consecutive pixels of a row, K = 9 * CIN in
// steps of 16 in (tap, channel) order.  The same kernel with flipped,
// transposed weights computes the data gradient.
//
// Every input pixel is read for nine taps: a wave keeps all weight fragments in
// registers (no staging and no barrier per tile), issues the loads of all K
// steps of a tile before its products, and walks tiles in RowWalk's order (x
// shifts meet in L1, row shifts in L2).  Out-of-image taps are out-of-range
// buffer loads (zero), tested once per column shift.  Lanes l and l + 32 hold
// alternate groups of four channels of one pixel and trade them
// (v_permlane32_swap) for 16-byte stores.  A 32 -> 32 layer of 1024 x 1024 pixels
// takes 45.5 us (84 with the weights staged per 256 pixels, tiles in launch
// order and 8-byte stores; 27 us at the copy rate), bound by the vector memory
// path, whose loads take 32 of each pixel's 64 bytes at a time: k_conv_rows
// takes the large layers.  A 2 x 61 x 93 layer takes 5 us (11.7).
//   kConvWaves: the launch's resident workgroups per CU.
// --------------------------------------------------------------------------
constexpr int kConvWaves = 2;

template <int CIN, int COUT>
__global__ __launch_bounds__(256, kConvWaves) void k_conv_fwd(
    const __bf16 *__restrict__ x, const __bf16 *__restrict__ w, const float *__restrict__ bias,
    int H, int W, int dilx, int dily, int relu, long nseg, int spr, __bf16 *__restrict__ yb,
    float *__restrict__ yf) {
    constexpr int K = 9 * CIN, NS = K / 16, PB = CIN * 2;   // PB: bytes per pixel
    __shared__ float bl[32];
    if (threadIdx.x < 32)
        bl[threadIdx.x] = bias && (int)threadIdx.x < COUT ? bias[threadIdx.x] : 0.0f;
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63u);
    const int n = lane & 31, kh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    RowWalk<4> q(nseg, spr, H, wave);          // segments of one tile
    if (q.t >= q.t1) return;
    bf16x8 a[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
        a[s] = *(const bf16x8 *)(w + (size_t)n * K + s * 16 + kh * 8);
    const int lo = n * PB + kh * 16;
    for (; q.t < q.t1; q.next(spr, H)) {
        const unsigned x0 = (unsigned)q.sx * 32u;
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
        int off[3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            off[c] = x0 + (unsigned)n + (unsigned)((c - 1) * dilx) < (unsigned)W ? lo : kOut;
        bf16x8 bv[NS];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int yy = q.y + (r - 1) * dily;
            const int bytes = (unsigned)yy < (unsigned)H ? 32 * PB : 0;
            const char *src = (const char *)x +
                              ((q.row + (long)(r - 1) * dily) * W + (long)x0) * PB;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const __amdgpu_buffer_rsrc_t rs = buf_of(src + (long)(c - 1) * dilx * PB, bytes);
                if (CIN == 16) {
                    bv[3 * r + c] = load_bf16x8(rs, off[c]);
                } else {
                    const int s = 2 * (3 * r + c);
                    bv[s] = load_bf16x8(rs, off[c]);
                    bv[(s + 1) % NS] = load_bf16x8(rs, off[c] + 32);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);     // every load is on its way before the products
#pragma unroll
        for (int s = 0; s < NS; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], bv[s], acc, 0, 0, 0);
        conv_store<COUT>(acc, bl, relu, kh, x0 + (unsigned)n < (unsigned)W,
                         ((size_t)q.row * W + x0 + n) * COUT, yb, yf);
    }
}

// --------------------------------------------------------------------------
// The same convolution for dilations up to 32, with the input staged in LDS:
// bitwise what k_conv_fwd gives.  k_conv_fwd's nine reads of a pixel are bound
// by the vector memory path (its loads take 32 of each pixel's 64 bytes).
// Here a workgroup takes 128 pixels of a row, loads the three tap rows' runs
// of 128 + 2 dil pixels once, as they lie in memory (the next segment's while
// this one is computed), and its four waves read their 32-pixel tiles' taps
// from LDS.  1024 x 1024 pixels, 32 -> 32: 34.8 us at dilations 1 to 9 and 40.7 at 27
// (3.9 and 3.3 TB/s of activations read and written once; matrix products
// 8 us, LDS reads about 15), 41 and 52 us with FP32 output.  Three workgroups
// per CU (156 VGPRs): two take 41.8 us, and four spill.
// --------------------------------------------------------------------------
constexpr int kRowTile = 128, kRowSpan = kRowTile + 64, kRowsWaves = 3;

template <int CIN, int COUT>
__global__ __launch_bounds__(256, kRowsWaves) void k_conv_rows(
    const __bf16 *__restrict__ x, const __bf16 *__restrict__ w, const float *__restrict__ bias,
    int H, int W, int dil, int dily, int relu, long nseg, int spr, __bf16 *__restrict__ yb,
    float *__restrict__ yf) {
    constexpr int K = 9 * CIN, NS = K / 16, PB = CIN * 2;   // PB: bytes per pixel
    constexpr int QPP = CIN / 8, PPL = 64 / QPP;            // 16-byte parts per pixel, pixels per load
    constexpr int NL = (kRowSpan / PPL + 3) / 4;            // loads per wave and row
    __shared__ __align__(16) char xs[3 * kRowSpan * PB];
    __shared__ float bl[32];
    if (threadIdx.x < 32)
        bl[threadIdx.x] = bias && (int)threadIdx.x < COUT ? bias[threadIdx.x] : 0.0f;
    const int lane = (int)(threadIdx.x & 63u);
    const int n = lane & 31, kh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    RowWalk<1> q(nseg, spr, H, 0);
    bf16x8 a[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
        a[s] = *(const bf16x8 *)(w + (size_t)n * K + s * 16 + kh * 8);
    const int nstage = kRowTile + 2 * dil;
    // LDS position of the 16-byte part q of staged pixel p: parts are permuted
    // within a pixel so that eight neighbouring pixels' parts q lie in
    // different banks
    auto part_at = [](int p, int q) { return (p * QPP + (q ^ ((p * QPP >> 3) & (QPP - 1)))) * 16; };
    int rd[3];                                 // this lane's reads, one per column shift
#pragma unroll
    for (int c = 0; c < 3; ++c) rd[c] = part_at(32 * wave + n + c * dil, kh);
    bf16x8 st[3][NL];
    auto load_seg = [&]() {
        const int x0 = q.sx * kRowTile;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int yy = q.y + (r - 1) * dily;
            const int bytes = (unsigned)yy < (unsigned)H ? 1024 : 0;
            const char *src = (const char *)x + ((q.row + (long)(r - 1) * dily) * W + x0 - dil) * PB;
#pragma unroll
            for (int k = 0; k < NL; ++k) {
                const int p0 = (wave + 4 * k) * PPL;
                if (p0 >= nstage) continue;    // uniform
                const int xx = x0 - dil + p0 + lane / QPP;
                st[r][k] = load_bf16x8(buf_of(src + (long)p0 * PB, bytes),
                                       (unsigned)xx < (unsigned)W ? lane * 16 : kOut);
            }
        }
    };
    if (q.t < q.t1) load_seg();
    while (q.t < q.t1) {
        lds_barrier();                         // the segment before has been read
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < NL; ++k) {
                const int p0 = (wave + 4 * k) * PPL;
                if (p0 >= nstage) continue;
                *(bf16x8 *)(xs + r * kRowSpan * PB + part_at(p0 + lane / QPP, lane % QPP)) = st[r][k];
            }
        lds_barrier();
        const int x0 = q.sx * kRowTile + 32 * wave;
        const size_t o = ((size_t)q.row * W + x0 + n) * COUT;
        q.next(spr, H);
        if (q.t < q.t1) load_seg();
        if (x0 >= W) continue;                 // uniform: past the row's end
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int tap = s * 16 / CIN, odd = CIN == 32 ? s % 2 : 0;
            const bf16x8 bv = *(const bf16x8 *)(xs + (tap / 3) * kRowSpan * PB +
                                                (rd[tap % 3] ^ (odd * 32)));
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], bv, acc, 0, 0, 0);
        }
        conv_store<COUT>(acc, bl, relu, kh, x0 + n < W, o, yb, yf);
    }
}

// --------------------------------------------------------------------------
// Backward of one layer, y = act(conv(x, w) + bias).  With dZ = dY * relu'(y)
// (BF16):
//   data gradient    dX = conv(dZ, flipped w)          (k_conv_fwd)
//   weight gradient  dW[co][tap][ci] = sum_p dZ[p][co] x[p + dil off(tap)][ci]
//   bias gradient    db[co] = sum_p dZ[p][co]
//
// k_wgrad forms dZ (written out for the data gradient, NULL when that is not
// wanted), the weight and bias gradients' partial sums and, in the blocks
// past nchunks, the flipped weights.  The weight gradient is an implicit GEMM on
// the matrix cores with the pixels as the reduction dimension (M = 32 output
// channels, N = 32 input channels of one tap, K = 16 pixels), whose operand
// fragments are eight consecutive pixels of one channel.  A workgroup takes a
// chunk of 1024 consecutive pixels (numbered over the whole batch) in units of
// 64.  Its last wave forms the next unit's dZ while the three others, one per
// tap row, stage the current unit's input pixels in LDS as they lie in memory
// (64 bytes per pixel; the unit after it is loaded meanwhile) and read both
// through the transposing LDS load (ds_read_b64_tr_b16).  To that load a
// pixel is a row address of its own: a tap's shift is another row, and a tap
// that leaves the image, or a pixel past the batch, reads a row of zeros (one
// ballot per unit and tap says which).  So any width and dilation takes one
// path and nothing is transposed in memory.  k_sum_partials adds the chunks'
// partials; the order of every sum (16-pixel steps within a chunk, then 16
// runs of chunks) is fixed.
//
// Bound by HBM on large inputs (dY, y and x read, dZ written): 8 x 256 x 256 pixels
// of a 32 -> 32 layer take 41 us, 4.0 TB/s (34 us at the copy rate; transposed
// copies of dZ and x, then products and four sums, took 204), of a 32 -> 16 layer 27
// (40).  On small ones by the instructions of a chunk's 16 units, each wave alone on
// its SIMD: 20 us for 2 x 61 x 93 pixels, 36 with a loaded pixel's bounds worked out
// in 64 bits for each load, divisions for its column and row in each unit and the
// fragments' rows selected in every unit (544 with a per-pixel path for widths that
// are no multiple of 8).  The barrier between the dZ wave and the others waits for LDS
// only, so that loads stay in flight across it.
// --------------------------------------------------------------------------
constexpr int kUnit = 64;       // pixels per unit
constexpr int kChunk = 1024;    // pixels per workgroup and partial sum
constexpr int kSumRuns = 16;    // runs of chunks that k_sum_partials forms first

// Staged pixels per tap row, a template argument of k_wgrad so that its loads are
// straight-line code (with their number a variable the loads were waited for one
// by one): 64 + 2 dil in a row where that is at most 128, else 64 for each of the
// three taps.
inline int wgrad_span(int dil) { return dil <= 16 ? 96 : dil <= 32 ? 128 : 192; }

// Eight pixels of 32 channels, transposed: lane l gets pixels 8 (l / 32) + j
// (j < 8) of channel l % 32 from LDS rows of 64 bytes per pixel.  `at` and `at4`
// are the lane's parts of the rows it passes to the two loads, pixels
// 8 (l / 32) + (l % 16) / 4 and four on (tr_lane_offset past the fragment's pixel 0
// where the pixels lie in a row).
__device__ __forceinline__ int tr_lane_offset(int lane) {
    return (8 * (lane >> 5) + ((lane & 15) >> 2)) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
}
__device__ __forceinline__ bf16x8 tr_frag(const char *at, const char *at4) {
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    union {
        s16x4 h[2];
        bf16x8 v;
    } f;
    f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)at);
    f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)at4);
    return f.v;
}
// Orders a wave's LDS writes before its own later LDS reads of other lanes'
// data and the reverse (the LDS serves a wave's accesses in order, so only
// the compiler has to keep it).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Flipped, transposed weights for the data gradient:
// wt[ci][tap'][co] = w[co][8 - tap'][ci] (rows ci >= CIN are zero).
__device__ __forceinline__ void flip_weight(const __bf16 *__restrict__ w, int cin, int cout,
                                            int idx, __bf16 *__restrict__ wt) {
    const int K2 = 9 * cout;               // row length of wt
    if (idx >= 32 * K2) return;
    const int ci = idx / K2, r = idx % K2;
    const int tp = r / cout, co = r % cout;
    __bf16 v = (__bf16)0.0f;
    if (ci < cin) v = w[(size_t)co * (9 * cin) + (8 - tp) * cin + ci];
    wt[idx] = v;
}

template <int CIN, int COUT, int SPAN>
__global__ __launch_bounds__(256) void k_wgrad(
    const float *__restrict__ dy, const __bf16 *__restrict__ y, int relu,
    const __bf16 *__restrict__ x, int H, int W, int dilx, int dily, int P, int nchunks,
    __bf16 *__restrict__ dz, float *__restrict__ part, float *__restrict__ dbpart,
    const __bf16 *__restrict__ w, __bf16 *__restrict__ wt) {
    constexpr int NN = 9 * CIN;
    // three waves' staged pixels, each followed by a pixel of zeros; dZ, twice
    constexpr int XB = (SPAN + 1) * 64, ZB = kUnit * 64;
    __shared__ __align__(16) char lds[3 * XB + 2 * ZB];
    if ((int)blockIdx.x >= nchunks) {
        flip_weight(w, CIN, COUT, ((int)blockIdx.x - nchunks) * 256 + (int)threadIdx.x, wt);
        return;
    }
    // channels that the layer does not have, and the pixels of zeros, stay zero
    for (int e = (int)threadIdx.x; e < (3 * XB + 2 * ZB) / 16; e += 256)
        *(u32x4 *)(lds + e * 16) = u32x4{0, 0, 0, 0};
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63u);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    char *zs = lds + 3 * XB;
    const int g = xcd_remap((int)blockIdx.x, nchunks);
    const int c0 = g * kChunk, c1 = min(P, c0 + kChunk);
    const int nu = (c1 - c0 + kUnit - 1) / kUnit;
    if (wave == 3) {
        // dZ of each unit, eight channels per lane
        // (loaded one unit ahead)
        constexpr int LPP = COUT / 8, PPL = 64 / LPP, NC = kUnit / PPL;   // lanes per pixel, pixels per load
        float f[NC][8];
        bf16x8 yv[NC];
        // this lane's first element of the chunk's first unit
        const size_t e0 = (size_t)(c0 + lane / LPP) * COUT + (lane % LPP) * 8;
        auto load_dy = [&](int i) {
            const size_t e = e0 + (size_t)(i * kUnit) * COUT;
            if ((i + 1) * kUnit <= c1 - c0) {      // a whole unit (uniform)
#pragma unroll
                for (int c = 0; c < NC; ++c) __builtin_memcpy(f[c], dy + e + c * PPL * COUT, 32);
                if (!relu) return;
#pragma unroll
                for (int c = 0; c < NC; ++c) __builtin_memcpy(&yv[c], y + e + c * PPL * COUT, 16);
                return;
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
#pragma unroll
                for (int j = 0; j < 8; ++j) f[c][j] = 0.0f;
                yv[c] = zero_bf16x8();
                if (i * kUnit + c * PPL + lane / LPP < c1 - c0) {
                    __builtin_memcpy(f[c], dy + e + c * PPL * COUT, 32);
                    if (relu) __builtin_memcpy(&yv[c], y + e + c * PPL * COUT, 16);
                }
            }
        };
        load_dy(0);
        for (int i = 0; i < nu; ++i) {
            bf16x8 z[NC];
            if (relu) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        z[c][j] = (__bf16)((float)yv[c][j] > 0.0f ? f[c][j] : 0.0f);
            } else {
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int j = 0; j < 8; ++j) z[c][j] = (__bf16)f[c][j];
            }
            if (i + 1 < nu) load_dy(i + 1);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int pu = c * PPL + lane / LPP, p = c0 + i * kUnit + pu;
                *(bf16x8 *)(zs + (i & 1) * ZB + pu * 64 + (lane % LPP) * 16) = z[c];
                if (dz && p < c1) *(bf16x8 *)(dz + (size_t)p * COUT + (lane % LPP) * 8) = z[c];
            }
            lds_barrier();
        }
        return;
    }
    f32x16 acc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[k][v] = 0.0f;
    float bsum = 0.0f;
    char *xs = lds + wave * XB;
    const int oy = (wave - 1) * dily;
    constexpr bool span = SPAN <= 128;         // one staged run serves the three column shifts
    const int pitch = span ? dilx : kUnit;     // staged pixels between two column shifts
    constexpr int LPP = CIN / 8, PPL = 64 / LPP, NS = SPAN / PPL;
    bf16x8 st[NS];
    // loads of unit i: staged pixel p is pixel (unit's first) + oy W - dil + p, or
    // + oy W + (c - 1) dil + p % 64 for the run c = p / 64 of a column shift.  A
    // run's loads go through a buffer that starts at the chunk's first pixel of it (or
    // the batch's) and ends with the batch: a pixel past the end reads zeros, and
    // so does one before the start, at an offset that wraps.
    struct Run {
        __amdgpu_buffer_rsrc_t pixels;
        int off;
    } run[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        constexpr long kReach = kChunk + 2 * kUnit;   // staged pixels of a run, and past them
        const long q = (long)c0 + (long)oy * W + (long)(t - 1) * dilx, qb = max(q, 0L);
        const bool none = q <= -kReach;
        run[t].pixels = buf_of(x + min(qb, (long)P) * CIN,
                               none ? 0 : (int)min(max((long)P - qb, 0L), kReach) * CIN * 2);
        run[t].off = (none ? 0 : (int)(q - qb) * CIN * 2) + lane * 16;
    }
    auto load_unit = [&](int i) {
        const int u = i * kUnit * CIN * 2;
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            const Run &r = run[span ? 0 : c * PPL / kUnit];
            st[c] = load_bf16x8(r.pixels,
                                r.off + u + (span ? c * PPL : c * PPL % kUnit) * CIN * 2);
        }
    };
    const int lo = tr_lane_offset(lane);
    const int lp = lo >> 6;                    // this lane's pixel of a fragment's first read
    const char *xt[3];                         // of the three column shifts
#pragma unroll
    for (int c = 0; c < 3; ++c) xt[c] = xs + lo + c * pitch * 64;
    // this lane's pixel of the unit: column and image row, carried from unit to unit
    const unsigned w64 = (unsigned)kUnit / (unsigned)W, wrest = (unsigned)kUnit % (unsigned)W;
    const unsigned hstep = w64 % (unsigned)H;
    const unsigned p0 = (unsigned)c0 + (unsigned)lane;
    unsigned px = p0 % (unsigned)W, py = p0 / (unsigned)W % (unsigned)H;
    load_unit(0);
    for (int i = 0; i < nu; ++i) {
        wave_lds_order();                      // the reads of the unit before are done
#pragma unroll
        for (int c = 0; c < NS; ++c)
            *(bf16x8 *)(xs + (c * PPL + lane / LPP) * 64 + (lane % LPP) * 16) = st[c];
        if (i + 1 < nu) load_unit(i + 1);
        // which taps of the unit's pixels stay in the image
        const bool row_in = p0 + (unsigned)(i * kUnit) < (unsigned)P && py + (unsigned)oy < (unsigned)H;
        uint64_t in[3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            in[c] = __ballot(row_in && px + (unsigned)((c - 1) * dilx) < (unsigned)W);
        px += wrest;
        py += hstep;
        if (px >= (unsigned)W) {
            px -= (unsigned)W;
            ++py;
        }
        if (py >= (unsigned)H) py -= (unsigned)H;
        lds_barrier();                         // the unit's dZ is there
        bf16x8 af[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const char *at = zs + (i & 1) * ZB + lo + k * 16 * 64;
            af[k] = tr_frag(at, at + 4 * 64);
            if (wave == 0) {
#pragma unroll
                for (int j = 0; j < 8; ++j) bsum += (float)af[k][j];
            }
        }
        // reads and products of the whole unit as one block, the LDS rows of its
        // fragments constants but for the units with a tap outside the image
        auto products = [&](auto row) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                bf16x8 bf[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) bf[c] = tr_frag(row(c, k, 0), row(c, k, 1));
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[k], bf[c], acc[c], 0, 0, 0);
            }
        };
        if ((in[0] & in[1] & in[2]) == ~0ull) {   // uniform
            products([&](int c, int k, int q) { return xt[c] + (k * 16 + q * 4) * 64; });
        } else {
            const char *zero = xs + SPAN * 64 + (lo & 63);
            const char *o[3][4][2];
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t m = (uint32_t)(in[c] >> (32 * (k / 2))) >> (16 * (k % 2));
                    o[c][k][0] = (m >> lp) & 1u ? xt[c] + k * 16 * 64 : zero;
                    o[c][k][1] = (m >> (lp + 4)) & 1u ? xt[c] + (k * 16 + 4) * 64 : zero;
                }
            products([&](int c, int k, int q) { return o[c][k][q]; });
        }
    }
    // D[co][ci] with co = 8 i + 4 h + j in accumulator 4 i + j, ci = lane % 32
    const int r = lane & 31, h = lane >> 5;
    float *out = part + (size_t)g * 32 * NN;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (r < CIN)
                out[(size_t)(8 * (v / 4) + 4 * h + v % 4) * NN + (3 * wave + c) * CIN + r] = acc[c][v];
    bsum += __shfl_xor(bsum, 32, 64);          // lanes r and r + 32 hold the same channel
    if (wave == 0 && h == 0) dbpart[(size_t)g * 32 + r] = bsum;
}

// dW and db from the chunks' partials: 32 columns per block (dW's ndw
// columns, then db's 32), kSumRuns runs of rows summed in order, then the
// runs in order.  Bound by the latency of a run's chain of loads (32 rows on
// 512 chunks).
__global__ __launch_bounds__(32 * kSumRuns) void k_sum_partials(const float *__restrict__ part,
                                                                const float *__restrict__ dbpart,
                                                                int nrows, int ndw,
                                                                float *__restrict__ dw,
                                                                float *__restrict__ db) {
    __shared__ float sh[kSumRuns][32];
    const int c = (int)(threadIdx.x & 31u), run = (int)(threadIdx.x >> 5);
    const bool bias = (int)blockIdx.x * 32 >= ndw;
    const int i = bias ? c : (int)blockIdx.x * 32 + c, pitch = bias ? 32 : ndw;
    const float *in = bias ? dbpart : part;
    const int per = (nrows + kSumRuns - 1) / kSumRuns;
    const int r0 = run * per, r1 = min(nrows, r0 + per);
    float acc = 0.0f;
#pragma unroll 8
    for (int r = r0; r < r1; ++r) acc += in[(size_t)r * pitch + i];
    sh[run][c] = acc;
    __syncthreads();
    if (run != 0) return;
    float v = 0.0f;
#pragma unroll
    for (int k = 0; k < kSumRuns; ++k) v += sh[k][c];
    if (bias) db[i] = v;
    else dw[i] = v;
}

// Adam step on FP32 master weights (bias-corrected moments); refreshes the
// BF16 copy used by the matrix cores.  A tensor has 32 to 9216 elements, so a launch
// takes its 3 us whatever it does: workgroup row blockIdx.y takes one of up to 16
// tensors (a network's twelve, one launch each: 57 us of a training step, 5 now).
constexpr int kAdamTensors = 16;
struct AdamList {
    gabp_adam_tensor t[kAdamTensors];
};

__global__ __launch_bounds__(256) void k_adam(AdamList list, float lr, float b1, float b2,
                                              float eps, float c1, float c2) {
    const gabp_adam_tensor &t = list.t[blockIdx.y];
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= t.n) return;
    const float gi = t.g[i];
    const float mi = b1 * t.m[i] + (1.0f - b1) * gi;
    const float vi = b2 * t.v[i] + (1.0f - b2) * gi * gi;
    t.m[i] = mi;
    t.v[i] = vi;
    const float wi = t.w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    t.w[i] = wi;
    if (t.w_bf16) ((__bf16 *)t.w_bf16)[i] = (__bf16)wi;
}

// Loss and output gradient.  pred[p][16]: channel 0 the mean, channels 1..12
// log(-Lam) of the sender-indexed precision messages.  Mean term:
// (mu^ - mu*)^2 averaged over pixels; precision term: weight times the mean
// of (l^ - l*)^2 over existing edges (valid > 0).  Per-block partial loss
// sums in a fixed order.
__global__ __launch_bounds__(256) void k_warm_loss(const float *__restrict__ pred,
                                                   const float *__restrict__ mu_t,
                                                   const float *__restrict__ lam_t,
                                                   const float *__restrict__ valid, long P,
                                                   int ndir, float inv_np, float lam_w_inv_ne,
                                                   float *__restrict__ grad,
                                                   double *__restrict__ part) {
    __shared__ double sh[4];
    const long p = (long)blockIdx.x * 256 + threadIdx.x;
    double l = 0.0;
    if (p < P) {
        // the pixel's 16 prediction channels as four 16-byte rows
        const float4 *pr = (const float4 *)(pred + p * 16);
        float v[16], g[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 t = pr[q];
            v[4 * q] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
        }
        const float e = v[0] - mu_t[p];
        g[0] = 2.0f * e * inv_np;
        l += (double)e * e * inv_np;
#pragma unroll
        for (int d = 0; d < 15; ++d) {
            float ed = 0.0f;
            if (d < ndir) {
                const float ok = valid[(size_t)d * P + p];
                ed = ok > 0.0f ? v[1 + d] - lam_t[(size_t)d * P + p] : 0.0f;
            }
            g[1 + d] = 2.0f * ed * lam_w_inv_ne;
            l += (double)ed * ed * lam_w_inv_ne;
        }
        float4 *gr = (float4 *)(grad + p * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) gr[q] = make_float4(g[4 * q], g[4 * q + 1], g[4 * q + 2], g[4 * q + 3]);
    }
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) l += __shfl_xor(l, k, 64);
    if ((threadIdx.x & 63u) == 0u) sh[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Input features of a lattice problem, NHWC BF16 [ny][nx][16]: channel 0 the
// observation mask, 1 the mean observed value (0 where unobserved), 2 the
// log prior scale kappa (shifted), the rest zero.  cnt/sum are FP32 scratch
// planes of nx*ny.  Bound by writing the features, 32 bytes a cell in two 16-byte
// stores: every cell's are written as unobserved, together with zeros into the
// scratch of the observed cells, then the observations are added up there and
// those cells' two channels written over.  From one observation in 12 cells on the
// whole scratch is cleared and every cell's features are built from it instead:
// observations in no order reach the scratch and the features a cell at a time, each
// for a line of its own.  First way, second and the second with 2-byte stores, us:
// 1024^2 with 1 % observed 17.3, 17.9 and 24, 6 % in no order 21.7, 21.6 and 28 and by
// cell 18.4, 19.4 and 26, 15 % 39, 31 and 38 and by cell 22.0, 22.3 and 28, every cell 175,
// 115 and 122 and by cell 29, 23 and 30; 2048 x 1500 with 1 % 26, 32 and 53, every cell 514,
// 322 and 342.  ALIGNED: x is 16-byte aligned.
template <bool ALIGNED>
__device__ __forceinline__ void feat_store(__bf16 *__restrict__ o, float mask, float mean,
                                           float kfeat) {
    bf16x8 a = {}, b = {};
    a[0] = (__bf16)mask;
    a[1] = (__bf16)mean;
    a[2] = (__bf16)kfeat;
    if (ALIGNED) {
        ((bf16x8 *)o)[0] = a;
        ((bf16x8 *)o)[1] = b;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            o[k] = a[k];
            o[8 + k] = b[k];
        }
    }
}

template <bool ALIGNED>
__global__ __launch_bounds__(256) void k_feat_fill(long N, float kfeat, __bf16 *__restrict__ x,
                                                   long n, const int64_t *__restrict__ cell,
                                                   float *__restrict__ cnt,
                                                   float *__restrict__ sum) {
    const long p = (long)blockIdx.x * 256 + threadIdx.x;
    if (p < n) {
        const int64_t c = cell[p];
        if (c >= 0 && c < N) {
            cnt[c] = 0.0f;
            sum[c] = 0.0f;
        }
    }
    if (p < N) feat_store<ALIGNED>(x + p * 16, 0.0f, 0.0f, kfeat);
}

// p[0 .. n) = 0 (a kernel, not a memset, so that callers may capture it in a graph)
__global__ __launch_bounds__(256) void k_feat_zero(long n, float *__restrict__ p) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

template <bool ALIGNED>
__global__ __launch_bounds__(256) void k_feat_build(long N, const float *__restrict__ cnt,
                                                    const float *__restrict__ sum, float kfeat,
                                                    __bf16 *__restrict__ x) {
    const long p = (long)blockIdx.x * 256 + threadIdx.x;
    if (p >= N) return;
    const float c = cnt[p];
    feat_store<ALIGNED>(x + p * 16, c > 0.0f ? 1.0f : 0.0f, c > 0.0f ? sum[p] / c : 0.0f, kfeat);
}

__global__ __launch_bounds__(256) void k_feat_scatter(long n, const int64_t *__restrict__ cell,
                                                      const double *__restrict__ yv, long N,
                                                      float *__restrict__ cnt,
                                                      float *__restrict__ sum) {
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const int64_t c = cell[k];
    if (c < 0 || c >= N) return;
    atomicAdd(&cnt[c], 1.0f);
    atomicAdd(&sum[c], (float)yv[k]);
}

// Mask and mean observed value of the observed cells.
__global__ __launch_bounds__(256) void k_feat_observed(long n, const int64_t *__restrict__ cell,
                                                       long N, const float *__restrict__ cnt,
                                                       const float *__restrict__ sum,
                                                       __bf16 *__restrict__ x) {
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const int64_t c = cell[k];
    if (c < 0 || c >= N) return;
    x[c * 16] = (__bf16)1.0f;
    x[c * 16 + 1] = (__bf16)(sum[c] / cnt[c]);
}

// Warm start of the messages from a prediction (mean mu^ and log(-Lam^) per
// sender-indexed edge): Lam_{i->j} = -exp(l^), and the information message
// that makes every edge consistent with the predicted means,
// th_{i->j} = Lam_{i->j} mu^_j - (Q_ij / c) mu^_i.  With exact means and
// converged precisions this is the fixed point; in general the beliefs
// become mu_i = mu^_i + (b - A mu^)_i / Lam_i.  keep_prec keeps the current
// precision messages instead of the predicted ones.
template <typename T, int ALPHA>
__global__ __launch_bounds__(256) void k_warm_init(Lattice L, const float *__restrict__ pred,
                                                   int keep_prec, T *__restrict__ m) {
    constexpr int DEG = ALPHA == 1 ? 4 : 12;
    const int tile = (int)blockIdx.x;
    const int x = (tile % L.tiles_x) * 64 + (int)(threadIdx.x & 63u);
    const int y = (tile / L.tiles_x) * 4 + (int)(threadIdx.x >> 6);
    if (x >= L.nx || y >= L.ny) return;
    const uint32_t i = (uint32_t)(y * L.pitch + x);
    const size_t pi = (size_t)y * L.nx + x;
    const float mui = pred[pi * 16];
    const T li = ALPHA == 2 ? ell<T>(L, x, y) : (T)0;
#pragma unroll
    for (int d = 0; d < DEG; ++d) {
        int xn, yn;
        if (!neighbour(L, x, y, d, xn, yn)) continue;
        const float muj = pred[((size_t)yn * L.nx + xn) * 16];
        T lam;
        if (keep_prec) lam = (m + (size_t)d * L.plane)[i];
        else lam = -(T)expf(pred[pi * 16 + 1 + d]);
        const T q = q_over_c<T, ALPHA>(L, d, li, xn, yn);
        (m + (size_t)d * L.plane)[i] = lam;
        (m + (size_t)(DEG + d) * L.plane)[i] = lam * (T)muj - q * (T)mui;
    }
}

// Training targets of the precision outputs from a solver state:
// lam[d][y][x] = log(-Lam) of the message from (x, y) to its neighbour in
// direction d (the sender-indexed plane d of the message buffer m) and
// valid[d][y][x] = 1 where that neighbour exists; 0 in both elsewhere and
// for d >= deg (12 planes are always written).  -Lam is floored at 1e-30.
template <typename T, int ALPHA>
__global__ __launch_bounds__(256) void k_log_prec(Lattice L, const T *__restrict__ m,
                                                  float *__restrict__ lam,
                                                  float *__restrict__ valid) {
    constexpr int DEG = ALPHA == 1 ? 4 : 12;
    const int tile = (int)blockIdx.x;
    const int x = (tile % L.tiles_x) * 64 + (int)(threadIdx.x & 63u);
    const int y = (tile / L.tiles_x) * 4 + (int)(threadIdx.x >> 6);
    if (x >= L.nx || y >= L.ny) return;
    const uint32_t i = (uint32_t)(y * L.pitch + x);
    const size_t np = (size_t)L.nx * L.ny, pi = (size_t)y * L.nx + x;
#pragma unroll
    for (int d = 0; d < 12; ++d) {
        float l = 0.0f, v = 0.0f;
        int xn, yn;
        if (d < DEG && neighbour(L, x, y, d, xn, yn)) {
            const float neg = -(float)(m + (size_t)d * L.plane)[i];
            l = logf(neg > 1e-30f ? neg : 1e-30f);
            v = 1.0f;
        }
        lam[(size_t)d * np + pi] = l;
        if (valid) valid[(size_t)d * np + pi] = v;
    }
}

// --------------------------------------------------------------------------
// host launchers
// --------------------------------------------------------------------------
hipError_t launch_log_prec(int dtype, const Lattice &L, const void *m, float *lam, float *valid,
                           hipStream_t s) {
    dim3 grid(L.tiles_x * ((L.ny + 3) / 4)), block(256);
    if (dtype == 0) {
        if (L.alpha == 1)
            hipLaunchKernelGGL((k_log_prec<float, 1>), grid, block, 0, s, L, (const float *)m, lam, valid);
        else
            hipLaunchKernelGGL((k_log_prec<float, 2>), grid, block, 0, s, L, (const float *)m, lam, valid);
    } else {
        if (L.alpha == 1)
            hipLaunchKernelGGL((k_log_prec<double, 1>), grid, block, 0, s, L, (const double *)m, lam, valid);
        else
            hipLaunchKernelGGL((k_log_prec<double, 2>), grid, block, 0, s, L, (const double *)m, lam, valid);
    }
    return hipGetLastError();
}

hipError_t launch_warm_init(int dtype, const Lattice &L, const float *pred, int keep_prec,
                            void *m, hipStream_t s) {
    dim3 grid(L.tiles_x * ((L.ny + 3) / 4)), block(256);
    if (dtype == 0) {
        if (L.alpha == 1)
            hipLaunchKernelGGL((k_warm_init<float, 1>), grid, block, 0, s, L, pred, keep_prec, (float *)m);
        else
            hipLaunchKernelGGL((k_warm_init<float, 2>), grid, block, 0, s, L, pred, keep_prec, (float *)m);
    } else {
        if (L.alpha == 1)
            hipLaunchKernelGGL((k_warm_init<double, 1>), grid, block, 0, s, L, pred, keep_prec, (double *)m);
        else
            hipLaunchKernelGGL((k_warm_init<double, 2>), grid, block, 0, s, L, pred, keep_prec, (double *)m);
    }
    return hipGetLastError();
}

}  // namespace gabp

// ==========================================================================
// C ABI of the network primitives
// ==========================================================================
// Scratch of gabp_warm_features_noalloc: the two FP32 planes (observation
// counts and sums) of at most kFeatScratchCells cells, 16 MiB that each GPU
// the library runs on holds until the process ends.  Host code must not pass
// this name to a kernel (it is a host-side stand-in): the device address
// comes from hipGetSymbolAddress, once per device.
constexpr long kFeatScratchCells = 1L << 21;
static __device__ __align__(256) float scratch[2 * kFeatScratchCells];

namespace {
thread_local std::string g_net_error;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_dev[kMaxDevices] = {};   // device address of `scratch`, per device

// The current device's address of `scratch`, looked up on the device's first
// call (with that device current); allocates nothing.
hipError_t scratch_address(float **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_dev[dev] = (float *)p;
    }
    *out = g_scratch_dev[dev];
    return hipSuccess;
}

// Input features from observations with cnt/sum scratch planes of N cells (2 N
// floats, of which at least the observed cells' are cleared and used).
hipError_t features_into(int64_t nobs, const int64_t *cell, const double *y, long N,
                         double kappa, float *scr, void *x_bf16, hipStream_t s) {
    const float kf = (float)(std::log(kappa) + 2.5);
    const bool aligned = (uintptr_t)x_bf16 % 16 == 0, dense = nobs > N / 12;
    auto blocks = [](long n) { return dim3((unsigned)((n + 255) / 256)); };
    const dim3 obs = blocks((long)nobs), block(256);
    float *cnt = scr, *sum = scr + N;
    __bf16 *x = (__bf16 *)x_bf16;
    if (dense)
        hipLaunchKernelGGL(gabp::k_feat_zero, blocks(2 * N), block, 0, s, 2 * N, scr);
    else if (aligned)
        hipLaunchKernelGGL(gabp::k_feat_fill<true>, blocks(std::max(N, (long)nobs)), block, 0, s, N,
                           kf, x, (long)nobs, cell, cnt, sum);
    else
        hipLaunchKernelGGL(gabp::k_feat_fill<false>, blocks(std::max(N, (long)nobs)), block, 0, s, N,
                           kf, x, (long)nobs, cell, cnt, sum);
    if (nobs > 0)
        hipLaunchKernelGGL(gabp::k_feat_scatter, obs, block, 0, s, (long)nobs, cell, y, N, cnt, sum);
    if (dense && aligned)
        hipLaunchKernelGGL(gabp::k_feat_build<true>, blocks(N), block, 0, s, N, (const float *)cnt,
                           (const float *)sum, kf, x);
    else if (dense)
        hipLaunchKernelGGL(gabp::k_feat_build<false>, blocks(N), block, 0, s, N, (const float *)cnt,
                           (const float *)sum, kf, x);
    else if (nobs > 0)
        hipLaunchKernelGGL(gabp::k_feat_observed, obs, block, 0, s, (long)nobs, cell, N,
                           (const float *)cnt, (const float *)sum, x);
    return hipGetLastError();
}

gabp_status nfail(gabp_status st, const std::string &m) {
    g_net_error = m;
    return st;
}

bool chan_ok(int c) { return c == 16 || c == 32; }

#define NHIP(call)                                                                      \
    do {                                                                                \
        hipError_t e_ = (call);                                                         \
        if (e_ != hipSuccess)                                                           \
            return nfail(GABP_E_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

int cu_count() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
        return 256;
    return cus;
}

// A dilation beyond the image's side reaches nothing on that axis, whatever
// it is: clamped there so that a column's position plus it stays in 32 bits.
int clamp_dil(int dil, int side) { return dil < side ? dil : side; }

// Whether k_conv_rows takes a convolution: its staged runs hold dilations up
// to 32; below 65536 pixels its two barriers and staging cost more than the
// strided loads they save (128 x 256: 5.2 against 4.7 us, 2 x 128 x 256: 7.0 against
// 7.2, 8 x 256 x 256: 21.4 against 26.0, 1024 x 1024: 34.8 against 45.5), and so
// do segments less than three quarters full (8 x 600 x 64: 20.4 against 18.5).
bool conv_by_rows(int B, int H, int W, int dil) {
    const long seg = gabp::kRowTile, spr = (W + seg - 1) / seg;
    return dil <= 32 && (long)B * H * W >= 65536 && 4L * W >= 3 * seg * spr;
}

hipError_t conv_dispatch(const void *x, int B, int H, int W, int cin, const void *w,
                         const float *bias, int cout, int dil, int relu, void *yb, float *yf,
                         hipStream_t s) {
    const __bf16 *xx = (const __bf16 *)x, *ww = (const __bf16 *)w;
    __bf16 *ybb = (__bf16 *)yb;
    const int dx = clamp_dil(dil, W), dy = clamp_dil(dil, H);
    // one round of resident workgroups over segments of 128 pixels (one per
    // workgroup) or 32 (one per wave), so that weights are loaded once per wave
    // and there is no tail
    const bool rows = conv_by_rows(B, H, W, dil);
    const int seg = rows ? gabp::kRowTile : 32, per = rows ? 1 : 4;
    const int spr = W / seg + (W % seg != 0);
    const long segs = (long)B * H * spr, want = (segs + per - 1) / per;
    const long resident = (long)cu_count() * (rows ? gabp::kRowsWaves : gabp::kConvWaves);
    dim3 grid((unsigned)(want < resident ? want : resident)), block(256);
    if (rows) {
        if (cin == 16 && cout == 16)
            hipLaunchKernelGGL((gabp::k_conv_rows<16, 16>), grid, block, 0, s, xx, ww, bias, H, W, dx, dy, relu, segs, spr, ybb, yf);
        else if (cin == 16)
            hipLaunchKernelGGL((gabp::k_conv_rows<16, 32>), grid, block, 0, s, xx, ww, bias, H, W, dx, dy, relu, segs, spr, ybb, yf);
        else if (cout == 16)
            hipLaunchKernelGGL((gabp::k_conv_rows<32, 16>), grid, block, 0, s, xx, ww, bias, H, W, dx, dy, relu, segs, spr, ybb, yf);
        else
            hipLaunchKernelGGL((gabp::k_conv_rows<32, 32>), grid, block, 0, s, xx, ww, bias, H, W, dx, dy, relu, segs, spr, ybb, yf);
        return hipGetLastError();
    }
    if (cin == 16 && cout == 16)
        hipLaunchKernelGGL((gabp::k_conv_fwd<16, 16>), grid, block, 0, s, xx, ww, bias, H, W, dx, dy, relu, segs, spr, ybb, yf);
    else if (cin == 16)
        hipLaunchKernelGGL((gabp::k_conv_fwd<16, 32>), grid, block, 0, s, xx, ww, bias, H, W, dx, dy, relu, segs, spr, ybb, yf);
    else if (cout == 16)
        hipLaunchKernelGGL((gabp::k_conv_fwd<32, 16>), grid, block, 0, s, xx, ww, bias, H, W, dx, dy, relu, segs, spr, ybb, yf);
    else
        hipLaunchKernelGGL((gabp::k_conv_fwd<32, 32>), grid, block, 0, s, xx, ww, bias, H, W, dx, dy, relu, segs, spr, ybb, yf);
    return hipGetLastError();
}

hipError_t wgrad_dispatch(const float *dy, const void *y, int relu, const void *x, int H, int W,
                          int cin, int cout, int dil, int P, int nchunks, void *dz, float *part,
                          float *dbpart, const void *w, void *wt, hipStream_t s) {
    const int dx = clamp_dil(dil, W), dyl = clamp_dil(dil, H);
    const int nflip = dz ? (32 * 9 * cout + 255) / 256 : 0;
    dim3 grid((unsigned)(nchunks + nflip)), block(256);
    const __bf16 *yy = (const __bf16 *)y, *xx = (const __bf16 *)x, *ww = (const __bf16 *)w;
    __bf16 *z = (__bf16 *)dz, *t = (__bf16 *)wt;
#define WGRAD(CI, CO, SP)                                                                          \
    hipLaunchKernelGGL((gabp::k_wgrad<CI, CO, SP>), grid, block, 0, s, dy, yy, relu, xx, H, W, dx, \
                       dyl, P, nchunks, z, part, dbpart, ww, t)
#define WGRAD_SPAN(CI, CO)                                                                         \
    do {                                                                                           \
        if (span == 96) WGRAD(CI, CO, 96);                                                         \
        else if (span == 128) WGRAD(CI, CO, 128);                                                  \
        else WGRAD(CI, CO, 192);                                                                   \
    } while (0)
    const int span = gabp::wgrad_span(dx);
    if (cin == 16 && cout == 16) WGRAD_SPAN(16, 16);
    else if (cin == 16) WGRAD_SPAN(16, 32);
    else if (cout == 16) WGRAD_SPAN(32, 16);
    else WGRAD_SPAN(32, 32);
#undef WGRAD_SPAN
#undef WGRAD
    return hipGetLastError();
}

long wgrad_chunks(long P) { return (P + gabp::kChunk - 1) / gabp::kChunk; }
}  // namespace

extern "C" {

const char *gabp_net_last_error(void) { return g_net_error.c_str(); }

gabp_status gabp_conv3x3_fwd(const void *x, int32_t B, int32_t H, int32_t W, int32_t cin,
                             const void *w, const float *bias, int32_t cout, int32_t dil,
                             int32_t relu, void *y_bf16, float *y_f32, void *stream) {
    if (!x || !w || B < 1 || H < 1 || W < 1 || !chan_ok(cin) || !chan_ok(cout) || dil < 1 ||
        (!y_bf16 && !y_f32))
        return nfail(GABP_E_INVALID, "conv3x3_fwd: bad arguments (channels must be 16 or 32)");
    NHIP(conv_dispatch(x, B, H, W, cin, w, bias, cout, dil, relu, y_bf16, y_f32, (hipStream_t)stream));
    return GABP_OK;
}

size_t gabp_conv3x3_bwd_workspace(int32_t B, int32_t H, int32_t W, int32_t cin, int32_t cout) {
    const long P = (long)B * H * W;
    const long nchunks = wgrad_chunks(P);
    size_t bytes = 0;
    bytes += (size_t)32 * 9 * 32 * 2 + 256;                  // flipped weights
    bytes += (size_t)P * cout * 2 + 256;                     // dz (NHWC)
    bytes += (size_t)nchunks * 32 * 9 * cin * 4 + 256;       // the chunks' partials of dw
    bytes += (size_t)nchunks * 32 * 4 + 256;                 // and of db
    return bytes;
}

// Backward of one layer y = act(conv(x, w) + b): from dy (FP32 NHWC, cout
// channels) and the layer's input x and output y (BF16), the weight and bias
// gradients dw [32][9*cin], db [32] (FP32, rows >= cout zero) and, when dx is
// not NULL, the input gradient dx (FP32 NHWC, cin channels).  Deterministic.
gabp_status gabp_conv3x3_bwd(const void *x, const void *y, const float *dy, int32_t B, int32_t H,
                             int32_t W, int32_t cin, const void *w, int32_t cout, int32_t dil,
                             int32_t relu, float *dw, float *db, float *dx, void *workspace,
                             size_t workspace_bytes, void *stream) {
    if (!x || !y || !dy || !w || !dw || !db || B < 1 || H < 1 || W < 1 || !chan_ok(cin) ||
        !chan_ok(cout) || dil < 1 || !workspace)
        return nfail(GABP_E_INVALID, "conv3x3_bwd: bad arguments");
    if ((long)B * H * W >= (1L << 31) - 64)
        return nfail(GABP_E_INVALID, "conv3x3_bwd: more than 2^31 - 64 pixels");
    if (workspace_bytes < gabp_conv3x3_bwd_workspace(B, H, W, cin, cout))
        return nfail(GABP_E_NOMEM, "conv3x3_bwd: workspace too small");
    hipStream_t s = (hipStream_t)stream;
    const long P = (long)B * H * W;
    const int nchunks = (int)wgrad_chunks(P), ndw = 32 * 9 * cin;
    char *ws = (char *)workspace;
    auto take = [&](size_t bytes) {
        char *p = ws;
        ws += (bytes + 255) / 256 * 256;
        return p;
    };
    __bf16 *wt = (__bf16 *)take((size_t)32 * 9 * 32 * 2);
    __bf16 *dz = (__bf16 *)take((size_t)P * cout * 2);
    float *part = (float *)take((size_t)nchunks * ndw * 4);
    float *dbpart = (float *)take((size_t)nchunks * 32 * 4);
    NHIP(wgrad_dispatch(dy, y, relu, x, H, W, cin, cout, dil, (int)P, nchunks, dx ? dz : nullptr,
                        part, dbpart, w, wt, s));
    if (dx) NHIP(conv_dispatch(dz, B, H, W, cout, wt, nullptr, cin, dil, 0, nullptr, dx, s));
    hipLaunchKernelGGL(gabp::k_sum_partials, dim3((unsigned)(ndw / 32 + 1)),
                       dim3(32 * gabp::kSumRuns), 0, s, (const float *)part, (const float *)dbpart,
                       nchunks, ndw, dw, db);
    NHIP(hipGetLastError());
    return GABP_OK;
}

gabp_status gabp_adam_steps(int32_t n_tensors, const gabp_adam_tensor *t, double lr, double beta1,
                            double beta2, double eps, int32_t step, void *stream) {
    if (n_tensors < 0 || (n_tensors > 0 && !t) || step < 1)
        return nfail(GABP_E_INVALID, "adam_steps: bad arguments");
    for (int k = 0; k < n_tensors; ++k)
        if (!t[k].w || !t[k].g || !t[k].m || !t[k].v || t[k].n < 0)
            return nfail(GABP_E_INVALID, "adam_step: bad arguments");
    const float c1 = (float)(1.0 - std::pow(beta1, step)), c2 = (float)(1.0 - std::pow(beta2, step));
    for (int k = 0; k < n_tensors; k += gabp::kAdamTensors) {
        gabp::AdamList list{};
        const int n = std::min(gabp::kAdamTensors, n_tensors - k);
        int64_t most = 0;
        for (int q = 0; q < n; ++q) {
            list.t[q] = t[k + q];
            most = std::max(most, t[k + q].n);
        }
        hipLaunchKernelGGL(gabp::k_adam, dim3((unsigned)((most + 255) / 256), (unsigned)n), dim3(256),
                           0, (hipStream_t)stream, list, (float)lr, (float)beta1, (float)beta2,
                           (float)eps, c1, c2);
        NHIP(hipGetLastError());
    }
    return GABP_OK;
}

gabp_status gabp_adam_step(float *w, const float *g, float *m, float *v, void *w_bf16, int64_t n,
                           double lr, double beta1, double beta2, double eps, int32_t step,
                           void *stream) {
    const gabp_adam_tensor t{w, g, m, v, w_bf16, n};
    return gabp_adam_steps(1, &t, lr, beta1, beta2, eps, step, stream);
}

gabp_status gabp_warm_loss(const float *pred, const float *mu_t, const float *lam_t,
                           const float *valid, int64_t P, int32_t ndir, double lam_weight,
                           float *grad, double *partials, int32_t *nparts, void *stream) {
    if (!pred || !mu_t || !grad || !partials || !nparts || P < 1 || ndir < 0 || ndir > 12 ||
        (ndir > 0 && (!lam_t || !valid)))
        return nfail(GABP_E_INVALID, "warm_loss: bad arguments");
    const int nb = (int)((P + 255) / 256);
    *nparts = nb;
    const float inv_np = (float)(1.0 / (double)P);
    const float lw = (float)(lam_weight / ((double)P * (ndir > 0 ? ndir : 1)));
    hipLaunchKernelGGL(gabp::k_warm_loss, dim3(nb), dim3(256), 0, (hipStream_t)stream, pred, mu_t,
                       lam_t, valid, (long)P, ndir, inv_np, lw, grad, partials);
    NHIP(hipGetLastError());
    return GABP_OK;
}

gabp_status gabp_warm_features(int64_t nobs, const int64_t *cell, const double *y, int64_t nx,
                               int64_t ny, double kappa, float *work, void *x_bf16,
                               void *stream) {
    if (nx < 1 || ny < 1 || !work || !x_bf16 || nobs < 0 || (nobs > 0 && (!cell || !y)) ||
        !(kappa > 0))
        return nfail(GABP_E_INVALID, "warm_features: bad arguments");
    NHIP(features_into(nobs, cell, y, (long)nx * ny, kappa, work, x_bf16, (hipStream_t)stream));
    return GABP_OK;
}

gabp_status gabp_warm_features_noalloc(int64_t nobs, const int64_t *cell, const double *y,
                                       int64_t nx, int64_t ny, double kappa, void *x_bf16,
                                       void *stream) {
    if (nx < 1 || ny < 1 || !x_bf16 || nobs < 0 || (nobs > 0 && (!cell || !y)) ||
        !(kappa > 0))
        return nfail(GABP_E_INVALID, "warm_features_noalloc: bad arguments");
    if (nx > kFeatScratchCells || ny > kFeatScratchCells || nx * ny > kFeatScratchCells)
        return nfail(GABP_E_INVALID,
                     "warm_features_noalloc: nx * ny exceeds the static scratch of 2^21 cells");
    float *scr = nullptr;
    NHIP(scratch_address(&scr));
    NHIP(features_into(nobs, cell, y, (long)nx * ny, kappa, scr, x_bf16, (hipStream_t)stream));
    return GABP_OK;
}

}  // extern "C"
