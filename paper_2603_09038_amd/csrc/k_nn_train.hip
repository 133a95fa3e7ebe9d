// FP32 forward and backward of the learned preconditioner's network (training, and the FP32
// inference option): three 3x3x3 cross-correlations (zero padding 1, bias) on the (p+1)^3
// nodal tiles, 2 -> 16 -> 16 -> 1 channels with ReLU between, their input gradients, weight
// gradients and the gather/scatter around them.  All arithmetic is FP32, but for the
// weight gradients' sums (see there).
//
// Sixteen tiles form a group: the tiles of +r of eight consecutive elements and the tiles of
// -r of the same eight (tile t = 8 sign + element).  The 16-channel tensors are stored
// [group][point][tile][channel], the network's input and output [group][point][channel][tile],
// so that the 16 columns of an FP32 MFMA (v_mfma_f32_16x16x4_f32: lane l supplies A[l%16][l/16] and B[l/16][l%16], element v of
// its result is D[4(l/16)+v][l%16]) are the sixteen tiles at ONE point.  Every lane of an
// MFMA then has the same neighbours, so taps that leave the tile are skipped, not multiplied
// by zero: 13/15 of the taps remain per axis at p = 4, 65 % in all.  Operands come straight
// from global memory, and a result goes back there (a point's 16 x 16 block is 1 KB, four
// channels of a tile in each lane: one 16-byte load or store a point; with the tile index
// fastest, four 4-byte ones, the 16 -> 16 layer took 1.02 ms instead of 0.77), and a group is
// read from the L2 that its workgroup's XCD keeps: no barrier.
//
// The convolutions used to run on the vector ALU, one thread per point with its operands in
// LDS, at 41-48 TFLOP/s.  At 65,536 tiles of 5^3 points (32^3 elements, p = 4) the MFMA form
// is bound by the matrix pipe for the 16 -> 16 layers (8,788 MFMAs of 32 cycles a group,
// 0.47 ms at full rate) and by HBM for the others.  Times beside each kernel.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "k_nn.h"

namespace hexpa {

namespace {

typedef float f4_t __attribute__((ext_vector_type(4)));

constexpr int kTileGroup = 16;      // tiles of a group (MFMA columns)
constexpr int kGroupElems = 8;      // elements of a group (each with its +r and its -r tile)
constexpr int kConvWaves = 4;       // waves of a workgroup
constexpr int kGradBlocks = 768;    // weight gradients: three workgroups on each of 256 CUs

inline int64_t ngroups_of(int64_t nelem) { return (nelem + kGroupElems - 1) / kGroupElems; }
inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

__device__ __forceinline__ f4_t mfma4(float a, float b, f4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Work items are the N^2 point rows (j, k) of every group.  XCD x (workgroups b with
// b % 8 == x) owns a contiguous range of groups, and its waves take that range's rows
// round-robin, so the rows in flight on an XCD belong to a few groups, which its L2 holds.
// The grid is a multiple of eight workgroups.
template <int N>
struct RowWalk {
    int64_t it, end;
    int step;
    __device__ RowWalk(int64_t ngroups, int wave)
    {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        it = (ngroups * xcd >> 3) * (N * N) + slot * kConvWaves + wave;
        end = (ngroups * (xcd + 1) >> 3) * (N * N);
        step = (gridDim.x >> 3) * kConvWaves;
    }
    __device__ static void split(int64_t i, int64_t &g, int &j, int &k)
    {
        g = i / (N * N);
        const int r = (int)(i - g * (N * N));
        k = r / N;
        j = r - k * N;
    }
};

// grid of a row-walking kernel: on each XCD enough workgroups for the rows of its groups, at most
// `most` in all.  (The XCD with the most groups decides: with a grid for all rows divided by
// eight, one group, of eight elements, had one workgroup's four waves for its 25 rows at p = 4,
// and the FP32 network took 99 us there instead of 38; with four groups 50 instead of 40.)
inline unsigned conv_grid(int64_t ngroups, int n, int most)
{
    const int64_t want = ((ngroups + 7) / 8 * n * n + kConvWaves - 1) / kConvWaves;
    return (unsigned)std::min<int64_t>(most, 8 * want);
}

// ------------------------------------------------------------------ weight packing
// Lane-ordered A-operands.  Table 0: layer 2 forward, [tap][lane][s]: row o = l%16, k-step s = input
// channel 4(l/16) + s (one 16-byte read a tap).  1: layer 2 input gradient, row c = l%16, output
// channel 4(l/16) + s of the flipped tap.  2: layer 1 forward, step (row tap r = ty + 3 tz, half u): row o, k =
// (point, channel) = (h >> 1, h & 1), u = 0: taps tx = 0, 1; u = 1: only point 1, tx = 2.
// 3: layer 3 input gradient, step r: row c, k = tap tx = h (h = 3: zero) of the flipped tap.
// 4: layer 3 forward (vector ALU), [tap][lane][s]: channel 4(l/16) + s.
constexpr int kPackW2 = 27 * 4, kPackW1 = 9 * 2, kPackG3 = 9;
constexpr int kPackSteps32 = 2 * kPackW2 + kPackW1 + kPackG3 + kPackW2;
static_assert(kPackSteps32 * 64 <= kNetPack32, "packed weights fit the work array");
constexpr int kPackOff[5] = {0, kPackW2, 2 * kPackW2, 2 * kPackW2 + kPackW1, 2 * kPackW2 + kPackW1 + kPackG3};
static_assert(kPackW2 % 4 == 0 && kPackOff[4] * 64 % 4 == 0, "16-byte reads of the packed weights");

__global__ void k_pack32(const float *__restrict__ prm, float *__restrict__ wp)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kPackSteps32 * 64) return;
    int s = i / 64;
    const bool quad = s < kPackOff[2] || s >= kPackOff[4];  // [tap][lane][s] tables
    const int iq = s < kPackOff[2] ? i : i - 64 * kPackOff[4];  // table 1 starts at a multiple of 256
    const int l = quad ? (iq >> 2) & 63 : i & 63, m = l & 15, h = l >> 4, c4 = 4 * h + (i & 3);
    float v = 0.f;
    if (s < kPackW2) {
        v = prm[kNetOffW2 + (m * kNetCh + c4) * 27 + s / 4];
    } else if ((s -= kPackW2) < kPackW2) {
        v = prm[kNetOffW2 + (c4 * kNetCh + m) * 27 + 26 - s / 4];
    } else if ((s -= kPackW2) < kPackW1) {
        const int r = s / 2, u = s % 2, pt = h >> 1, c = h & 1;
        const int tx = u == 0 ? pt : 2;
        if (u == 0 || pt == 1) v = prm[kNetOffW1 + (m * kNetCin + c) * 27 + tx + 3 * r];
    } else if ((s -= kPackW1) < kPackG3) {
        if (h < 3) v = prm[kNetOffW3 + m * 27 + 26 - (h + 3 * s)];
    } else {
        v = prm[kNetOffW3 + c4 * 27 + (s - kPackG3) / 4];
    }
    wp[i] = v;
}

// ------------------------------------------------------------------ 16 -> 16 convolution
// Out row (j, k) of a group: N points' accumulators (16 channels x 16 tiles each).  The wave
// walks the row taps r = (ty, tz) that stay in the tile: the input row's points are loaded
// once (4 registers a point), each used by up to three taps and 4 k-steps (52 MFMAs a row at
// N = 5) while the next input row is in flight; the weights of its three taps come from LDS
// in three 16-byte reads.  (All 27 taps' weights in registers cost two of the four waves a
// SIMD now holds.)  The sum is taken in partial sums of 48 products, one an input row: a
// shorter chain rounds less than one over all 432, and with it fewer ReLU masks of the
// backward pass fall on the other side than in exact arithmetic.  BWD false: layer 2 forward,
// + bias, ReLU.  BWD true: the input gradient of layer 2, masked where the forward activation
// is not positive.
// 32^3 elements, p = 4: 2.35 -> 0.77 ms forward, 2.35 -> 0.78 ms input gradient.
constexpr int kConvBlocks = 1024;  // four workgroups on each CU

// The row taps of out row (j, k) of group g, then those of the wave's next item, ...
template <int N>
struct TapWalk {
    RowWalk<N> w;
    int64_t g;
    int j, k, ty, tz;
    bool live;  // an item is left
    __device__ TapWalk(int64_t ngroups, int wave) : w(ngroups, wave)
    {
        live = w.it < w.end;
        first();
    }
    __device__ void first()
    {
        w.split(live ? w.it : 0, g, j, k);
        ty = j > 0 ? 0 : 1;
        tz = k > 0 ? 0 : 1;
    }
    // to the next row tap; true when that is another item's first
    __device__ bool next()
    {
        if (++ty <= (j < N - 1 ? 2 : 1)) return false;
        ty = j > 0 ? 0 : 1;
        if (++tz <= (k < N - 1 ? 2 : 1)) return false;
        w.it += w.step;
        live = w.it < w.end;
        first();
        return true;
    }
    __device__ int row() const { return (k + tz - 1) * N + j + ty - 1; }
};

// a point's 16 channels x 16 tiles: lane (h, tile) holds channels 4h .. 4h + 3
template <int N>
__device__ __forceinline__ void load_row(f4_t (&b)[N], const float *__restrict__ in, const TapWalk<N> &t, int lane)
{
    const f4_t *p = reinterpret_cast<const f4_t *>(in + (t.g * (N * N) + t.row()) * (int64_t)(N * kNetCh * kTileGroup)) +
                    (lane & 15) * 4 + (lane >> 4);
#pragma unroll
    for (int i = 0; i < N; ++i) b[i] = p[i * (kNetCh * kTileGroup / 4)];
}
// stores such a point, rectified or masked by the forward activation
template <bool BWD>
__device__ __forceinline__ void store_point(float *__restrict__ out, const float *__restrict__ act, int64_t o, f4_t v)
{
    f4_t a = {0.f, 0.f, 0.f, 0.f}, r;
    if (BWD) a = *reinterpret_cast<const f4_t *>(act + o);
#pragma unroll
    for (int c = 0; c < 4; ++c) r[c] = BWD ? (a[c] > 0.f ? v[c] : 0.f) : fmaxf(v[c], 0.f);
    *reinterpret_cast<f4_t *>(out + o) = r;
}
template <int N>
__device__ __forceinline__ bool row_inside(int j, int k, int r)
{
    return (unsigned)(j + r % 3 - 1) < (unsigned)N && (unsigned)(k + r / 3 - 1) < (unsigned)N;
}

__device__ __forceinline__ void stage_weights(f4_t *sw, const float *__restrict__ wp)
{
    const f4_t *src = reinterpret_cast<const f4_t *>(wp);
    for (int i = threadIdx.x; i < 27 * 64; i += 256) sw[i] = src[i];
    __syncthreads();
}

template <int N, bool BWD>
__global__ __launch_bounds__(256, 4) void k_conv16(int64_t ngroups, const float *__restrict__ in,
                                                   const float *__restrict__ wp, const float *__restrict__ bias,
                                                   const float *__restrict__ act, float *__restrict__ out)
{
    __shared__ f4_t sw[27 * 64];
    const int lane = threadIdx.x & 63, h = lane >> 4, m = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    stage_weights(sw, wp);
    TapWalk<N> w(ngroups, wave);
    if (!w.live) return;
    f4_t b0 = {0.f, 0.f, 0.f, 0.f};
    if (!BWD)
#pragma unroll
        for (int v = 0; v < 4; ++v) b0[v] = bias[4 * h + v];
    f4_t cur[N], nxt[N], acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = b0;
    load_row<N>(cur, in, w, lane);
    for (;;) {
        const int r = 3 * w.tz + w.ty;
        const int64_t o0 = ((w.g * N + w.k) * N + w.j) * (int64_t)(N * kNetCh * kTileGroup) + kNetCh * m + 4 * h;
        const bool done = w.next();  // this was the item's last row tap
        load_row<N>(nxt, in, w, lane);  // past the last item: a valid row that is not used
        __builtin_amdgcn_sched_barrier(0);  // in flight during this row's MFMAs
        f4_t wt[3], part[N];
#pragma unroll
        for (int tx = 0; tx < 3; ++tx) wt[tx] = sw[(3 * r + tx) * 64 + lane];
#pragma unroll
        for (int i = 0; i < N; ++i) part[i] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int tx = 0; tx < 3; ++tx)
#pragma unroll
                for (int i = 0; i < N; ++i)
                    if (i + tx - 1 >= 0 && i + tx - 1 < N) part[i] = mfma4(wt[tx][s], cur[i + tx - 1][s], part[i]);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] += part[i];
        if (done) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                store_point<BWD>(out, act, o0 + i * (kNetCh * kTileGroup), acc[i]);
                acc[i] = b0;
            }
            if (!w.live) break;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) cur[i] = nxt[i];
    }
}

// ------------------------------------------------------------------ 2 -> 16 and 1 -> 16
// The same with few input channels: the four k of an MFMA are neighbouring points of a row.
// BWD false: layer 1 forward (two channels; k = two points x two channels; output i takes the
// pair (i-1, i) for tx = 0, 1 and the pair (i, i+1) for tx = 2).  BWD true: the input gradient
// of layer 3 (one channel; k = the points i-1, i, i+1).  Points outside the tile enter as zero.
// Bound by HBM (writes 16 channels a point, and reads as many for the mask).
// 32^3, p = 4: 0.257 -> 0.24 ms forward, 0.213 -> 0.24 ms input gradient.
template <int N, bool BWD>
__global__ __launch_bounds__(256, 4) void k_conv_in(int64_t ngroups, const float *__restrict__ in,
                                                    const float *__restrict__ wp, const float *__restrict__ bias,
                                                    const float *__restrict__ act, float *__restrict__ out)
{
    constexpr int C = BWD ? 1 : 2, NL = BWD ? N : N + 1, NWT = BWD ? 9 : 18;
    const int lane = threadIdx.x & 63, h = lane >> 4, m = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __shared__ float sw[NWT * 64];
    for (int i = threadIdx.x; i < NWT * 64; i += 256) sw[i] = wp[i];
    __syncthreads();
    RowWalk<N> w(ngroups, wave);
    f4_t b0 = {0.f, 0.f, 0.f, 0.f};
    if (!BWD)
#pragma unroll
        for (int v = 0; v < 4; ++v) b0[v] = bias[4 * h + v];
    const int dp = BWD ? h : h >> 1;  // this lane's point past the first of an operand
    const int lane_in = BWD ? 0 : (h & 1) * kTileGroup;
    for (; w.it < w.end; w.it += w.step) {
        int64_t g;
        int j, k;
        w.split(w.it, g, j, k);
        f4_t acc[N];
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = b0;
#pragma unroll 1
        for (int r = 0; r < 9; ++r) {
            if (!row_inside<N>(j, k, r)) continue;
            const float *p = in + ((g * N + k + r / 3 - 1) * N + j + r % 3 - 1) * (int64_t)(N * C * kTileGroup) + lane_in + m;
            float b[NL];
#pragma unroll
            for (int q = 0; q < NL; ++q) {
                const int pt = q - 1 + dp;
                const bool ok = pt >= 0 && pt < N && dp < 3;
                const float v = p[(ok ? pt : 0) * (C * kTileGroup)];
                b[q] = ok ? v : 0.f;
            }
            f4_t part[N];
            const float w0 = sw[(BWD ? r : 2 * r) * 64 + lane], w1 = BWD ? 0.f : sw[(2 * r + 1) * 64 + lane];
#pragma unroll
            for (int i = 0; i < N; ++i) part[i] = mfma4(w0, b[i], (f4_t){0.f, 0.f, 0.f, 0.f});
            if (!BWD)
#pragma unroll
                for (int i = 0; i < N; ++i) part[i] = mfma4(w1, b[i + (BWD ? 0 : 1)], part[i]);
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] += part[i];
        }
        const int64_t o0 = ((g * N + k) * N + j) * (int64_t)(N * kNetCh * kTileGroup) + kNetCh * m + 4 * h;
#pragma unroll
        for (int i = 0; i < N; ++i) store_point<BWD>(out, act, o0 + i * (kNetCh * kTileGroup), acc[i]);
    }
}

// ------------------------------------------------------------------ 16 -> 1 convolution
// Layer 3 forward: one output channel leaves 15 of 16 MFMA rows unused, so this one runs on
// the vector ALU in the same data flow: lane (h, tile) sums the channels 4s + h of its tile
// for the points of one output row, the four quarter sums are added at the end.  Bound by the
// reads of its input (16 channels a point).  32^3, p = 4: 0.444 -> 0.25 ms.
template <int N>
__global__ __launch_bounds__(256, 4) void k_conv_out(int64_t ngroups, const float *__restrict__ in,
                                                     const float *__restrict__ wp, const float *__restrict__ bias,
                                                     float *__restrict__ out)
{
    __shared__ f4_t sw[27 * 64];
    const int lane = threadIdx.x & 63, h = lane >> 4, m = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    stage_weights(sw, wp);
    TapWalk<N> w(ngroups, wave);
    if (!w.live) return;
    // the bias enters one lane's sum first: added to the finished sums its rounding would be
    // correlated with them and leave a systematic error in the odd part (1.5e-8 of z measured)
    const float b3 = h == 0 ? bias[0] : 0.f;
    f4_t cur[N], nxt[N];
    float acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = b3;
    load_row<N>(cur, in, w, lane);
    for (;;) {
        const int r = 3 * w.tz + w.ty;
        float *o = out + ((w.g * N + w.k) * N + w.j) * (int64_t)(N * kTileGroup) + m;
        const bool done = w.next();
        load_row<N>(nxt, in, w, lane);
        __builtin_amdgcn_sched_barrier(0);
        f4_t wt[3];
        float part[N];
#pragma unroll
        for (int tx = 0; tx < 3; ++tx) wt[tx] = sw[(3 * r + tx) * 64 + lane];
#pragma unroll
        for (int i = 0; i < N; ++i) part[i] = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int tx = 0; tx < 3; ++tx)
#pragma unroll
                for (int i = 0; i < N; ++i)
                    if (i + tx - 1 >= 0 && i + tx - 1 < N) part[i] = fmaf(wt[tx][s], cur[i + tx - 1][s], part[i]);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] += part[i];
        if (done) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float v = acc[i];
                v += __shfl_xor(v, 16);
                v += __shfl_xor(v, 32);
                if (h == 0) o[i * kTileGroup] = v;
                acc[i] = b3;
            }
            if (!w.live) break;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) cur[i] = nxt[i];
    }
}

// ------------------------------------------------------------------ weight gradients
// dW[o][c][tap] = sum over tiles and points of dout[o][pt] in[c][pt + off(tap)]: an MFMA
// takes four tiles as its k (lane l holds channel l%16) and adds a 16 x 16 block of one tap.
// The blocks of a wave's taps (layer 2: the nine of its tap plane) stay in registers over every row it takes; the
// waves of a workgroup are then added in FP64 in wave order through LDS and the workgroup writes one row of
// `partial` (weights, then biases), which the two reduction kernels add in FP64 in a fixed order.
// What is added in FP32 before that is short, since each addition rounds at the size of the
// sum so far: layer 2 takes 4 N products an MFMA chain, adds the four chains of a row in a tree
// and the rows one by one; layers 1 and 3 take eight products a chain and add a point's two
// chains in FP32, all else in FP64.  (One chain over all products of a wave, 10,400 at 32^3,
// left twice the rounding of the result, 5.4e-8 and at 48^3 9.2e-8; now 2.7e-8 and 2.9e-8, of
// which 2.5e-8 is the rounding of the result to FP32.)
// Layer 2, 32^3, p = 4: 2.46 -> 0.63 ms (the matrix pipe, as the convolutions).
// The rows come as 16-byte loads (a vector memory instruction occupies the CU's address unit
// for about 16 cycles whatever its width: with 4-byte loads in the layout the MFMA wants this
// kernel took 1.02-1.22 ms) and are turned through wave-private LDS, a point's block at
// [tile][channel] with tile pitch PITCH: lane (h, channel) reads tiles 4s + h (PITCH 16) or
// 4h + s (PITCH 20, which spreads the four h over the banks), s = 0..3.
template <int N>
__device__ __forceinline__ void load_raw(f4_t (&b)[N], const float *__restrict__ in, int64_t row, int lane)
{
    const f4_t *p = reinterpret_cast<const f4_t *>(in + row * (N * kNetCh * kTileGroup)) + lane;
#pragma unroll
    for (int i = 0; i < N; ++i) b[i] = p[i * 64];
}
template <int N, int PITCH>
__device__ __forceinline__ void turn_row(f4_t (&b)[N], const f4_t (&raw)[N], float *buf, int lane)
{
    constexpr int PT = kTileGroup * PITCH;
    // the wave's lanes run in lockstep and the LDS serves a wave in order: only the compiler has
    // to keep the reads behind the other lanes' writes, and those behind the row before
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    const float *p = buf + (lane & 15) + (lane >> 4) * (PITCH == 16 ? PITCH : 4 * PITCH);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        *reinterpret_cast<f4_t *>(buf + i * PT + (lane >> 2) * PITCH + (lane & 3) * 4) = raw[i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
#pragma unroll
        for (int s = 0; s < 4; ++s) b[i][s] = p[i * PT + s * (PITCH == 16 ? 4 * PITCH : PITCH)];
    }
}

template <int N>
__global__ __launch_bounds__(256, 2) void k_wgrad16(int64_t ngroups, const float *__restrict__ in,
                                                    const float *__restrict__ dout, float *__restrict__ partial)
{
    constexpr int NT = kNetW2 + kNetCh;
    constexpr int RED = 27 * 4 * 64, BUF = N * kTileGroup * 16;
    __shared__ double red[RED > kConvWaves * BUF / 2 ? RED : kConvWaves * BUF / 2];  // row buffers, then the sums
    __shared__ double redb[64];
    const int lane = threadIdx.x & 63, m = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *buf = reinterpret_cast<float *>(red) + wave * BUF;
    if (threadIdx.x < 64) redb[threadIdx.x] = 0.0;
    // This wave's tap plane tz: of each 3N - 2 consecutive waves of an XCD, N - 1, N and N - 1
    // take tz = 0, 1, 2, in proportion to the output planes a group has for it.  Its items are
    // those planes of the XCD's groups, round-robin over the waves of the same tz.
    constexpr int PER = 3 * N - 2;
    const int xcd = blockIdx.x & 7, W = (blockIdx.x >> 3) * kConvWaves + wave, TW = (gridDim.x >> 3) * kConvWaves;
    const int q = W / PER, r = W - q * PER;
    const int tz = r < N - 1 ? 0 : (r < 2 * N - 1 ? 1 : 2), base = tz == 0 ? 0 : (tz == 1 ? N - 1 : 2 * N - 1);
    const int cnt = tz == 1 ? N : N - 1, k0 = tz == 0 ? 1 : 0;  // output planes k0 .. k0 + cnt - 1
    const int nw = TW / PER * cnt + min(max(TW % PER - base, 0), cnt);
    const int64_t g0 = ngroups * xcd >> 3, end = ((ngroups * (xcd + 1) >> 3) - g0) * cnt;
    f4_t acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = (f4_t){0.f, 0.f, 0.f, 0.f};
    float bacc = 0.f;
    auto add = [](f4_t *c, const f4_t (&part)[3]) {
#pragma unroll
        for (int tx = 0; tx < 3; ++tx) {
            c[tx] += part[tx];
            asm volatile("" : "+v"(c[tx]));  // here: sunk to the next use, the parts would spill
        }
    };
    // one block of MFMAs: output row a, input row b, row tap ty, in four parts of 4 N products
    auto block = [&](const f4_t (&a)[N], const f4_t (&b)[N], f4_t *c) {
        f4_t part[4][3];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int tx = 0; tx < 3; ++tx) part[s][tx] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int tx = 0; tx < 3; ++tx)
                    if (i + tx - 1 >= 0 && i + tx - 1 < N) part[s][tx] = mfma4(a[i][s], b[i + tx - 1][s], part[s][tx]);
            if (s & 1) add(part[s - 1], part[s]);
        }
        add(part[0], part[2]);
        add(c, part[0]);
    };
    for (int64_t it = q * cnt + r - base; it < end; it += nw) {
        const int64_t g = g0 + it / cnt;
        const int k = k0 + (int)(it % cnt), kin = k + tz - 1;
        // input row jp meets the output rows jp + 1, jp, jp - 1 (ty = 0, 1, 2): three output
        // rows in a ring of slots, the input row double-buffered; the loads of the next rows
        // are in flight during this row's MFMAs
        f4_t a[3][N], b[N], ra[2][N], rb[2][N];
        const int64_t rin = (g * N + kin) * N, rout = (g * N + k) * N;
        load_raw<N>(rb[0], in, rin, lane);
        load_raw<N>(ra[0], dout, rout, lane);
        load_raw<N>(ra[1], dout, rout + 1, lane);
        load_raw<N>(rb[1], in, rin + 1, lane);
        turn_row<N, 16>(b, rb[0], buf, lane);
        turn_row<N, 16>(a[0], ra[0], buf, lane);
        load_raw<N>(ra[0], dout, rout + 2, lane);
        turn_row<N, 16>(a[1], ra[1], buf, lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jp = 0; jp < N; ++jp) {
            if (jp > 0) block(a[(jp + 2) % 3], b, acc + 6);
            block(a[jp % 3], b, acc + 3);
            if (jp + 1 < N) block(a[(jp + 1) % 3], b, acc);
            if (tz == 1) {
                float bpart = 0.f;
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const f4_t v = a[jp % 3][i];
                    bpart += (v[0] + v[1]) + (v[2] + v[3]);
                }
                bacc += bpart;
            }
            // the rows after the next: requested before the next ones are turned
            if (jp + 2 < N) load_raw<N>(rb[jp & 1], in, rin + jp + 2, lane);
            if (jp + 3 < N) load_raw<N>(ra[(jp + 1) & 1], dout, rout + jp + 3, lane);
            __builtin_amdgcn_sched_barrier(0);
            if (jp + 1 < N) turn_row<N, 16>(b, rb[(jp + 1) & 1], buf, lane);
            if (jp + 2 < N) turn_row<N, 16>(a[(jp + 2) % 3], ra[jp & 1], buf, lane);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < RED; i += 256) red[i] = 0.0;
    for (int p = 0; p < kConvWaves; ++p) {
        __syncthreads();
        if (wave == p) {
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[(4 * (9 * tz + t) + v) * 64 + lane] += acc[t][v];
            redb[lane] += bacc;
        }
    }
    __syncthreads();
    float *row = partial + (int64_t)blockIdx.x * NT;
    for (int i = threadIdx.x; i < 27 * 4 * 64; i += 256) {
        const int l = i & 63, v = (i >> 6) & 3, t = i >> 8;
        row[((4 * (l >> 4) + v) * kNetCh + (l & 15)) * 27 + t] = (float)red[i];
    }
    if (threadIdx.x < kNetCh)
        row[kNetW2 + m] = (float)((redb[m] + redb[m + 16]) + (redb[m + 32] + redb[m + 48]));
}

// Layers 1 and 3: one operand has 16 channels (`wide`: rows c = l%16), the other one or two
// (`thin`), whose (tap, channel) combinations are the MFMA columns: column 16 ct + l%16 is
// tap col / C, channel col % C, read at the point shifted by that tap (zero outside the
// tile).  Layer 1 (C = 2): wide = dout at pt, thin = in at pt + off.  Layer 3 (C = 1): wide =
// in at q, thin = dout at q - off; its bias is the column of the centre tap summed.
// Bound by the read of the wide operand.  32^3, p = 4: 0.491 -> 0.25 and 0.530 -> 0.17 ms.
template <int N, int C>
__global__ __launch_bounds__(256, 3) void k_wgrad_thin(int64_t ngroups, const float *__restrict__ wide,
                                                       const float *__restrict__ thin, float *__restrict__ partial)
{
    constexpr int NCT = (27 * C + 15) / 16, NW = 27 * C * kNetCh, NT = NW + (C == 2 ? kNetCh : 1);
    constexpr int RED = NCT * 4 * 64, BUF = N * kTileGroup * 20;
    __shared__ double red[RED > kConvWaves * BUF / 2 ? RED : kConvWaves * BUF / 2];  // row buffers, then the sums
    __shared__ double redb[64];
    const int lane = threadIdx.x & 63, h = lane >> 4, m = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *buf = reinterpret_cast<float *>(red) + wave * BUF;
    double acc[NCT][4];
    int off[NCT];               // shift of this lane's column, in floats of `thin`
    int mi[NCT], mj[NCT], mk[NCT];  // bit x: the shifted point of a point with that index is inside
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
        acc[t][0] = acc[t][1] = acc[t][2] = acc[t][3] = 0.0;
        const int col = 16 * t + m, tap = col / C;
        const bool has = tap < 27;
        const int sg = C == 2 ? 1 : -1;
        const int dx = has ? sg * (tap % 3 - 1) : 0, dy = has ? sg * ((tap / 3) % 3 - 1) : 0, dz = has ? sg * (tap / 9 - 1) : 0;
        off[t] = has ? ((dx + N * (dy + N * dz)) * C + col % C) * kTileGroup : 0;
        mi[t] = mj[t] = mk[t] = 0;
        for (int x = 0; x < N; ++x) {
            if (has && (unsigned)(x + dx) < (unsigned)N) mi[t] |= 1 << x;
            if (has && (unsigned)(x + dy) < (unsigned)N) mj[t] |= 1 << x;
            if (has && (unsigned)(x + dz) < (unsigned)N) mk[t] |= 1 << x;
        }
    }
    double bacc = 0.0;
    RowWalk<N> w(ngroups, wave);
    for (; w.it < w.end; w.it += w.step) {
        int64_t g;
        int j, k;
        w.split(w.it, g, j, k);
        f4_t a[N], raw[N];
        load_raw<N>(raw, wide, (g * N + k) * N + j, lane);
        turn_row<N, 20>(a, raw, buf, lane);
        float bpart = 0.f;
        const float *p = thin + ((g * N + k) * N + j) * (int64_t)(N * C * kTileGroup) + 4 * h;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            f4_t b[NCT];
#pragma unroll
            for (int t = 0; t < NCT; ++t) {
                const bool ok = (mi[t] >> i) & (mj[t] >> j) & (mk[t] >> k) & 1;
                const f4_t v = *reinterpret_cast<const f4_t *>(p + i * (C * kTileGroup) + (ok ? off[t] : 0));
                b[t] = ok ? v : (f4_t){0.f, 0.f, 0.f, 0.f};
            }
            // a point's sixteen products in two chains of eight
#pragma unroll
            for (int t = 0; t < NCT; ++t) {
                f4_t u = mfma4(a[i][0], b[t][0], (f4_t){0.f, 0.f, 0.f, 0.f});
                f4_t v = mfma4(a[i][1], b[t][1], (f4_t){0.f, 0.f, 0.f, 0.f});
                u = mfma4(a[i][2], b[t][2], u);
                v = mfma4(a[i][3], b[t][3], v);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    acc[t][x] += (double)(u[x] + v[x]);
                    asm volatile("" : "+v"(acc[t][x]));  // here: not sunk behind the other points' MFMAs
                }
            }
            if (C == 2) bpart += (a[i][0] + a[i][1]) + (a[i][2] + a[i][3]);
            else bpart += (b[0][0] + b[0][1]) + (b[0][2] + b[0][3]);  // column m = 13: the centre tap
        }
        bacc += (double)bpart;
    }
    __syncthreads();
    for (int q = 0; q < kConvWaves; ++q) {
        if (wave == q) {
#pragma unroll
            for (int t = 0; t < NCT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = (4 * t + v) * 64 + lane;
                    red[i] = q == 0 ? acc[t][v] : red[i] + acc[t][v];
                }
            redb[lane] = q == 0 ? bacc : redb[lane] + bacc;
        }
        __syncthreads();
    }
    float *row = partial + (int64_t)blockIdx.x * NT;
    for (int i = threadIdx.x; i < NCT * 4 * 64; i += 256) {
        const int l = i & 63, v = (i >> 6) & 3, col = 16 * (i >> 8) + (l & 15), ch = 4 * (l >> 4) + v;
        if (col < 27 * C) row[(ch * C + col % C) * 27 + col / C] = (float)red[i];
    }
    if (C == 2) {
        if (threadIdx.x < kNetCh) row[NW + m] = (float)((redb[m] + redb[m + 16]) + (redb[m + 32] + redb[m + 48]));
    } else if (threadIdx.x == 0) {
        row[NW] = (float)((redb[13] + redb[13 + 16]) + (redb[13 + 32] + redb[13 + 48]));
    }
}

// grad[w] += sum over rows of partial[row][w] in two passes, each in a fixed order (FP64
// accumulation, so the result is reproducible): the rows are cut into kReduceChunks chunks;
// a workgroup takes 64 columns of one chunk, its four waves summing every fourth row of it
// and their four sums added in wave order (part2[chunk][w], FP64); then one thread per
// column adds the chunks in order.  (One thread per column over all rows left most of the
// GPU idle: a layer has 433-6928 weights, so 2-28 workgroups.)
constexpr int kReduceChunks = 32;

__global__ __launch_bounds__(256) void k_reduce_chunks(const float *__restrict__ partial, int rows, int nt,
                                                       double *__restrict__ part2)
{
    __shared__ double red[4][64];
    const int l = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int w = blockIdx.x * 64 + l, chunk = blockIdx.y;
    const int r0 = (int)((int64_t)rows * chunk / kReduceChunks);
    const int r1 = (int)((int64_t)rows * (chunk + 1) / kReduceChunks);
    double a = 0.0;
    if (w < nt)
        for (int g = r0 + sl; g < r1; g += 4) a += partial[(int64_t)g * nt + w];
    red[sl][l] = a;
    __syncthreads();
    if (sl == 0 && w < nt) part2[(int64_t)chunk * nt + w] = ((red[0][l] + red[1][l]) + red[2][l]) + red[3][l];
}

__global__ void k_reduce_rows(const double *__restrict__ part2, int nt, float *__restrict__ grad)
{
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= nt) return;
    double a = 0.0;
    for (int c = 0; c < kReduceChunks; ++c) a += part2[(int64_t)c * nt + w];
    grad[w] += (float)a;
}

// ------------------------------------------------------------------ gather and scatter
// One workgroup per group: the eight elements' residual tiles through LDS, so that both the
// gather (element order) and the tile store ([point][channel][16]) are coalesced.  Elements
// past the mesh are zero tiles.  32 threads sum the squares of one element, in a fixed tree.
template <int N>
__global__ __launch_bounds__(256) void k_nn_input(int64_t nelem, const double *__restrict__ r,
                                                  const int32_t *__restrict__ emap, const float *__restrict__ logk,
                                                  float *__restrict__ x0, float *__restrict__ s_out)
{
    constexpr int P = N * N * N, PP = P | 1;  // odd row pitch
    __shared__ float sx[kGroupElems][PP], sl[kGroupElems][PP];
    const int64_t g = blockIdx.x;
    const int t = threadIdx.x, el = t >> 5, u = t & 31;
    const int64_t e = g * kGroupElems + el;
    constexpr int NS = (P + 31) / 32;
    double rv[NS], ss = 0.0;
    float lk[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const int pt = u + 32 * q;
        const bool ok = pt < P && e < nelem;
        rv[q] = ok ? r[emap[e * P + pt]] : 0.0;
        lk[q] = ok ? logk[e * P + pt] : 0.f;
        ss = fma(rv[q], rv[q], ss);
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    const double rms = sqrt(ss / P);
    const double sc = rms > 0.0 ? rms : 1.0;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const int pt = u + 32 * q;
        if (pt < P) {
            sx[el][pt] = (float)(rv[q] / sc);
            sl[el][pt] = lk[q];
        }
    }
    if (u == 0 && e < nelem) s_out[e] = (float)sc;
    __syncthreads();
    float *o = x0 + g * (int64_t)(P * 2 * kTileGroup);
    for (int i = t; i < P * 2 * kTileGroup; i += 256) {
        const int lane = i & 15, c = (i >> 4) & 1, pt = i >> 5;
        const float v = c ? sl[lane & 7][pt] : sx[lane & 7][pt];
        o[i] = (c == 0 && lane >= kGroupElems) ? -v : v;
    }
}

// z[g] += s_e (out(+r)_e - out(-r)_e) / 2 * inv_mult[g]: the odd part of the network,
// averaged over the elements sharing g.
template <int N>
__global__ __launch_bounds__(256) void k_nn_output(int64_t nelem, const float *__restrict__ out,
                                                   const float *__restrict__ s, const int32_t *__restrict__ emap,
                                                   const double *__restrict__ inv_mult, double scale,
                                                   double *__restrict__ z)
{
    constexpr int P = N * N * N;
    __shared__ float so[P * (kTileGroup + 1)];
    const int64_t grp = blockIdx.x, e0 = grp * kGroupElems;
    for (int i = threadIdx.x; i < P * kTileGroup; i += 256)
        so[(i >> 4) * (kTileGroup + 1) + (i & 15)] = out[grp * (int64_t)(P * kTileGroup) + i];
    __syncthreads();
    const int ne = (int)min((int64_t)kGroupElems, nelem - e0);
    for (int i = threadIdx.x; i < ne * P; i += 256) {
        const int el = i / P, pt = i - el * P;
        const int gi = emap[e0 * P + i];
        const float *o = so + pt * (kTileGroup + 1) + el;
        const double odd = 0.5 * scale * ((double)o[0] - (double)o[kGroupElems]);
        unsafeAtomicAdd(z + gi, odd * (double)s[e0 + el] * inv_mult[gi]);
    }
}

// adjoint: d/d out(+r) = s_e gz inv_mult / 2, d/d out(-r) = its negative; zero for the tiles
// past the mesh, which keeps them out of every weight gradient
template <int N>
__global__ __launch_bounds__(256) void k_nn_output_grad(int64_t nelem, const double *__restrict__ gz,
                                                        const float *__restrict__ s,
                                                        const int32_t *__restrict__ emap,
                                                        const double *__restrict__ inv_mult, float *__restrict__ gout)
{
    constexpr int P = N * N * N;
    __shared__ float so[kGroupElems][P | 1];
    const int64_t grp = blockIdx.x, e0 = grp * kGroupElems;
    for (int i = threadIdx.x; i < kGroupElems * P; i += 256) {
        const int el = i / P, pt = i - el * P;
        float v = 0.f;
        if (e0 + el < nelem) {
            const int gi = emap[e0 * P + i];
            v = (float)(0.5 * gz[gi] * inv_mult[gi] * (double)s[e0 + el]);
        }
        so[el][pt] = v;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < P * kTileGroup; i += 256) {
        const int lane = i & 15, pt = i >> 4;
        const float v = so[lane & 7][pt];
        gout[grp * (int64_t)(P * kTileGroup) + i] = lane >= kGroupElems ? -v : v;
    }
}

// floats of the largest block of partial rows (even, so the FP64 chunk sums behind it are
// 8-byte aligned)
constexpr int64_t kPartialRows = ((int64_t)kGradBlocks * (kNetW2 + kNetCh) + 1) & ~(int64_t)1;

void reduce_layer(unsigned rows, int nt, const float *partial, float *grad_w, hipStream_t s)
{
    double *part2 = reinterpret_cast<double *>(const_cast<float *>(partial) + kPartialRows);
    hipLaunchKernelGGL(k_reduce_chunks, dim3((nt + 63) / 64, kReduceChunks), dim3(256), 0, s, partial, (int)rows, nt,
                       part2);
    hipLaunchKernelGGL(k_reduce_rows, dim3(nblk(nt)), dim3(256), 0, s, part2, nt, grad_w);
}

template <int N>
hipError_t forward_t(int64_t ng, const float *params, float *wt, const float *x0, float *a1, float *a2, float *out,
                     hipStream_t s)
{
    const dim3 wide(conv_grid(ng, N, kConvBlocks)), b(256);
    hipLaunchKernelGGL(k_pack32, dim3(nblk(kPackSteps32 * 64)), dim3(256), 0, s, params, wt);
    hipLaunchKernelGGL((k_conv_in<N, false>), wide, b, 0, s, ng,
                       x0, wt + 64 * kPackOff[2], params + kNetOffB1, nullptr, a1);
    hipLaunchKernelGGL((k_conv16<N, false>), wide, b, 0, s, ng, a1, wt + 64 * kPackOff[0], params + kNetOffB2, nullptr, a2);
    hipLaunchKernelGGL((k_conv_out<N>), wide, b, 0, s, ng, a2, wt + 64 * kPackOff[4], params + kNetOffB3, out);
    return hipGetLastError();
}

// wt holds the packed weights the forward pass of the same parameters left there; a
// partial row (a layer's weights, then its biases) has the order of the gradient vector
template <int N>
hipError_t backward_t(int64_t ng, const float *wt, const float *x0, const float *a1, const float *a2,
                      const float *gout, float *ga2, float *ga1, float *grads, float *partial, hipStream_t s)
{
    // (k_wgrad16 needs 3N - 2 waves on every XCD: four workgroups)
    const dim3 nb(conv_grid(ng, N, kGradBlocks)), nb2(std::max(32u, conv_grid(ng, N, 512))), wide(conv_grid(ng, N, kConvBlocks)), b(256);
    hipLaunchKernelGGL((k_wgrad_thin<N, 1>), nb, b, 0, s, ng, a2, gout, partial);
    reduce_layer(nb.x, kNetW3 + 1, partial, grads + kNetOffW3, s);
    hipLaunchKernelGGL((k_conv_in<N, true>), wide, b, 0, s, ng,
                       gout, wt + 64 * kPackOff[3], nullptr, a2, ga2);
    hipLaunchKernelGGL((k_wgrad16<N>), nb2, b, 0, s, ng, a1, ga2, partial);
    reduce_layer(nb2.x, kNetW2 + kNetCh, partial, grads + kNetOffW2, s);
    hipLaunchKernelGGL((k_conv16<N, true>), wide, b, 0, s, ng, ga2, wt + 64 * kPackOff[1], nullptr, a1, ga1);
    // layer 1 (the input needs no gradient)
    hipLaunchKernelGGL((k_wgrad_thin<N, 2>), nb, b, 0, s, ng, ga1, x0, partial);
    reduce_layer(nb.x, kNetW1 + kNetCh, partial, grads + kNetOffW1, s);
    return hipGetLastError();
}

}  // namespace

int64_t nn_tiles(int64_t nelem) { return ngroups_of(nelem) * kTileGroup; }

int64_t nn_partial_floats()
{
    // partial rows, then the FP64 chunk sums (two floats each)
    return kPartialRows + 2 * (int64_t)kReduceChunks * (kNetW2 + kNetCh);
}

hipError_t nn_forward(int n, int64_t nelem, const float *params, float *wt, const float *x0, float *a1, float *a2,
                      float *out, hipStream_t s)
{
    const int64_t ng = ngroups_of(nelem);
    if (ng <= 0) return hipSuccess;
    if (n == 3) return forward_t<3>(ng, params, wt, x0, a1, a2, out, s);
    if (n == 4) return forward_t<4>(ng, params, wt, x0, a1, a2, out, s);
    if (n == 5) return forward_t<5>(ng, params, wt, x0, a1, a2, out, s);
    return hipErrorInvalidValue;
}

hipError_t nn_backward(int n, int64_t nelem, const float *wt, const float *x0, const float *a1, const float *a2,
                       const float *gout, float *ga2, float *ga1, float *grads, float *partial, hipStream_t s)
{
    const int64_t ng = ngroups_of(nelem);
    if (ng <= 0) return hipSuccess;
    if (n == 3) return backward_t<3>(ng, wt, x0, a1, a2, gout, ga2, ga1, grads, partial, s);
    if (n == 4) return backward_t<4>(ng, wt, x0, a1, a2, gout, ga2, ga1, grads, partial, s);
    if (n == 5) return backward_t<5>(ng, wt, x0, a1, a2, gout, ga2, ga1, grads, partial, s);
    return hipErrorInvalidValue;
}

hipError_t nn_input(int n, int64_t nelem, const double *r, const int32_t *emap, const float *logk, float *x0,
                    float *s, hipStream_t st)
{
    const dim3 nb((unsigned)ngroups_of(nelem));
    if (nb.x == 0) return hipSuccess;
    if (n == 3) hipLaunchKernelGGL(k_nn_input<3>, nb, dim3(256), 0, st, nelem, r, emap, logk, x0, s);
    else if (n == 4) hipLaunchKernelGGL(k_nn_input<4>, nb, dim3(256), 0, st, nelem, r, emap, logk, x0, s);
    else if (n == 5) hipLaunchKernelGGL(k_nn_input<5>, nb, dim3(256), 0, st, nelem, r, emap, logk, x0, s);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t nn_output(int n, int64_t nelem, const float *out, const float *s, const int32_t *emap,
                     const double *inv_mult, double scale, double *z, hipStream_t st)
{
    const dim3 nb((unsigned)ngroups_of(nelem));
    if (nb.x == 0) return hipSuccess;
    if (n == 3) hipLaunchKernelGGL(k_nn_output<3>, nb, dim3(256), 0, st, nelem, out, s, emap, inv_mult, scale, z);
    else if (n == 4) hipLaunchKernelGGL(k_nn_output<4>, nb, dim3(256), 0, st, nelem, out, s, emap, inv_mult, scale, z);
    else if (n == 5) hipLaunchKernelGGL(k_nn_output<5>, nb, dim3(256), 0, st, nelem, out, s, emap, inv_mult, scale, z);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t nn_output_grad(int n, int64_t nelem, const double *gz, const float *s, const int32_t *emap,
                          const double *inv_mult, float *gout, hipStream_t st)
{
    const dim3 nb((unsigned)ngroups_of(nelem));
    if (nb.x == 0) return hipSuccess;
    if (n == 3) hipLaunchKernelGGL(k_nn_output_grad<3>, nb, dim3(256), 0, st, nelem, gz, s, emap, inv_mult, gout);
    else if (n == 4) hipLaunchKernelGGL(k_nn_output_grad<4>, nb, dim3(256), 0, st, nelem, gz, s, emap, inv_mult, gout);
    else if (n == 5) hipLaunchKernelGGL(k_nn_output_grad<5>, nb, dim3(256), 0, st, nelem, gz, s, emap, inv_mult, gout);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace hexpa
