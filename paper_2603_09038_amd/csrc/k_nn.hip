// Kernels of the learned preconditioner: the FP16 inference of its per-element 3-layer
// convolutional network on the (p+1)^3 nodal tile (3x3x3 cross-correlation, zero padding 1,
// bias, ReLU between layers; the FP32 forward and backward are in k_nn_train.hip), Adam, and
// the p=1 coarse level of the two-level preconditioner.  Tile points are i + N j + N^2 k (the
// operator's local node order); weights are [c_out][c_in][tap], tap = tx + 3 ty + 9 tz
// reading the neighbour (i + tx - 1, j + ty - 1, k + tz - 1).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "k_nn.h"

namespace hexpa {

namespace {

inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

__global__ void k_count(int64_t total, const int32_t *__restrict__ emap, double *__restrict__ cnt)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < total) unsafeAtomicAdd(cnt + emap[idx], 1.0);
}
__global__ void k_recip_or_zero(int64_t n, double *__restrict__ v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = v[i] > 0.0 ? 1.0 / v[i] : 0.0;
}
__global__ void k_fill_f32(float *y, float v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) y[i] = v;
}

__global__ void k_adam(float *__restrict__ p, float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                       int n, float lr, float bc1, float bc2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    g[i] = 0.0f;
}

__global__ void k_sub(double *y, const double *a, const double *b, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = a[i] - b[i];
}
__global__ void k_mul(double *y, const double *a, const double *b, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = a[i] * b[i];
}

__global__ void k_loss_scale(double *g, int64_t n, double *sc)
{
    const double den = sc[1];
    const double f = den > 0.0 ? 2.0 / den : 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        g[i] *= f;
    if (blockIdx.x == 0 && threadIdx.x == 0) sc[2] = den > 0.0 ? sc[0] / den : 0.0;
}

// ---------------------------------------------------------------- coarse level
// uf = P1 u1, plus m1 * m2 where given.  Bound by memory; 32-bit indexes (a lattice has
// fewer than 2^31 points) since 64-bit divisions by run-time sizes cost more than the traffic:
// 129^3 points, with the product 18.4 us; the product 9.4 and the sum 16.9 before.
__global__ void k_prolong(BoxDims b, const double *__restrict__ gll, const double *__restrict__ u1,
                          double *__restrict__ uf, const double *__restrict__ m1, const double *__restrict__ m2)
{
    const uint32_t p = b.p, Mx = b.nx * p + 1, My = b.ny * p + 1, Mz = b.nz * p + 1;
    const uint32_t Cx = b.nx + 1, Cy = b.ny + 1;
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= Mx * My * Mz) return;
    const double base = m1 ? m1[g] * m2[g] : 0.0;
    const uint32_t K = g / (Mx * My), R = g - K * (Mx * My), J = R / Mx, I = R - J * Mx;
    const uint32_t ex = min(I / p, (uint32_t)b.nx - 1), ey = min(J / p, (uint32_t)b.ny - 1),
                   ez = min(K / p, (uint32_t)b.nz - 1);
    const double x = gll[I - ex * p], y = gll[J - ey * p], z = gll[K - ez * p];
    double v = 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int ca = c & 1, cb = (c >> 1) & 1, cc = c >> 2;
        const double w = (ca ? x : 1.0 - x) * (cb ? y : 1.0 - y) * (cc ? z : 1.0 - z);
        v += w * u1[(ex + ca) + Cx * ((ey + cb) + Cy * (ez + cc))];
    }
    uf[g] = m1 ? base + v : v;
}

// Restriction r1 = P1^T rf, separable: the weight of fine node (I,J,K) at coarse vertex
// (a,b,c) is w(I,a) w(J,b) w(K,c), so three 1-D passes (x, then y, then z), each summing
// the at most 2p + 1 fine lattice points whose 1-D weight for a coarse index is nonzero,
// in a fixed order (no atomics).  Pass `axis` maps in[nz'][ny'][nx'] to out with that
// axis shortened from M = n p + 1 to n + 1.
// The 1-D weight: a fine node in element ex at GLL coordinate xi weighs 1 - xi at vertex ex and
// xi at ex + 1.  All loads of a point are in flight together.  129^3 to
// 33^3 points: 8.3 -> 7.4 us an axis.
__global__ void k_restrict_axis(int axis, uint32_t n, uint32_t p, uint32_t nx_in, uint32_t ny_in, uint32_t nz_in,
                                const double *__restrict__ gll, const double *__restrict__ in,
                                double *__restrict__ out)
{
    const uint32_t C = n + 1, M = n * p + 1;
    const uint32_t ox = axis == 0 ? C : nx_in, oy = axis == 1 ? C : ny_in, oz = axis == 2 ? C : nz_in;
    const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= ox * oy * oz) return;
    const uint32_t k = idx / (ox * oy), rem = idx - k * (ox * oy), j = rem / ox, i = rem - j * ox;
    const uint32_t a = axis == 0 ? i : (axis == 1 ? j : k);  // coarse index along the axis
    const uint32_t stride = axis == 0 ? 1 : (axis == 1 ? nx_in : nx_in * ny_in);
    const uint32_t base = (axis == 0 ? 0 : i) + nx_in * ((axis == 1 ? 0 : j) + ny_in * (axis == 2 ? 0 : k));
    const uint32_t I0 = a > 0 ? (a - 1) * p : 0, I1 = min(M - 1, (a + 1) * p);
    double acc = 0.0;
#pragma unroll 4
    for (uint32_t I = I0; I <= I1; ++I) {  // the weight of vertex a at I; the last node has no element to its right
        const double w = I < a * p ? gll[I - (a - 1) * p] : a < n ? 1.0 - gll[I - a * p] : gll[p];
        const double v = in[base + I * stride];
        acc = w != 0.0 ? fma(w, v, acc) : acc;
    }
    out[idx] = acc;
}

__global__ void k_probe_vec(BoxDims b, int cls, double *__restrict__ v)
{
    const int64_t Cx = b.nx + 1, Cy = b.ny + 1, Cz = b.nz + 1;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= Cx * Cy * Cz) return;
    const int64_t I = i % Cx, J = (i / Cx) % Cy, K = i / (Cx * Cy);
    v[i] = (I % 3 == cls % 3 && J % 3 == (cls / 3) % 3 && K % 3 == cls / 9) ? 1.0 : 0.0;
}

// Within the 3x3x3 neighbourhood of vertex i exactly one vertex has class cls; the entry
// of A v_cls at i is therefore A[i][j] for that neighbour j (0 if j is off the lattice).
// S is stored [slot][i], slot = (dx+1) + 3 (dy+1) + 9 (dz+1).  Constrained rows and
// columns (ess) become those of the identity.
__global__ void k_probe_gather(BoxDims b, int cls, const double *__restrict__ y, const uint8_t *__restrict__ ess,
                               double *__restrict__ S)
{
    const int64_t Cx = b.nx + 1, Cy = b.ny + 1, Cz = b.nz + 1, n1 = Cx * Cy * Cz;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n1) return;
    const int64_t I = i % Cx, J = (i / Cx) % Cy, K = i / (Cx * Cy);
    auto delta = [](int64_t X, int want) {
        const int d = (int)(((want - X) % 3 + 3) % 3);
        return d == 2 ? -1 : d;
    };
    const int dx = delta(I, cls % 3), dy = delta(J, (cls / 3) % 3), dz = delta(K, cls / 9);
    const int slot = (dx + 1) + 3 * (dy + 1) + 9 * (dz + 1);
    const int64_t In = I + dx, Jn = J + dy, Kn = K + dz;
    double v = 0.0;
    if (In >= 0 && In < Cx && Jn >= 0 && Jn < Cy && Kn >= 0 && Kn < Cz) {
        const int64_t j = In + Cx * (Jn + Cy * Kn);
        v = y[i];
        if (ess && (ess[i] || ess[j])) v = (j == i && ess[i]) ? 1.0 : 0.0;
    }
    S[slot * n1 + i] = v;
}

__global__ void k_dinv_center(int64_t n1, const double *__restrict__ S, double *__restrict__ dinv)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n1) dinv[i] = 1.0 / S[13 * n1 + i];
}

// Coarse PCG.  Every kernel leaves one partial sum per block, and each block of the next one
// adds them all in the same fixed order: no counter, no last block and, above all, no device
// fence, which writes the L2 of every XCD back.  The grid is capped so that this stays a few
// loads a thread.  33^3 unknowns: init / a / b 7.4 / 15.2 / 8.0 ->
// 4.8 / 8.7 / 4.8 us.  What is left of them is launch, one pass of latency and the sums.
constexpr int kCoarseThreads = 256, kCoarseBlocks = kCoarsePartials / 2;
// block-wide sum in a fixed order (a shuffle tree in each wave, then the wave sums); every
// thread gets it.  sh: 4 doubles, not used again before a barrier.
__device__ inline double coarse_sum(double v, double *sh)
{
    const int t = threadIdx.x;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((t & 63) == 0) sh[t >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}
__device__ inline double coarse_total(const double *__restrict__ partial, double *sh)
{
    double v = 0.0;
    for (int i = threadIdx.x; i < (int)gridDim.x; i += kCoarseThreads) v += partial[i];
    return coarse_sum(v, sh);
}

// u = 0, z = dinv r, p0 = 0; partial sums of r.z
__global__ __launch_bounds__(kCoarseThreads) void k_cpcg_init(int64_t n1, const double *__restrict__ dinv,
                                                   const double *__restrict__ r, double *__restrict__ u,
                                                   double *__restrict__ z, double *__restrict__ p0,
                                                   double *__restrict__ prz)
{
    __shared__ double sh[4];
    double v = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kCoarseThreads + threadIdx.x; i < n1; i += (int64_t)gridDim.x * kCoarseThreads) {
        const double zi = dinv[i] * r[i];
        z[i] = zi;
        u[i] = 0.0;
        p0[i] = 0.0;
        v = fma(r[i], zi, v);
    }
    v = coarse_sum(v, sh);
    if (threadIdx.x == 0) prz[blockIdx.x] = v;
}

// beta = r.z / (the r.z before it), 0 in iteration 0; p1 = z + beta p0; Ap = S (z + beta p0);
// partial sums of p1 . Ap.  A neighbour outside the box is read as the point itself and counted
// as zero, so that all loads of a point are in flight together.
__global__ __launch_bounds__(kCoarseThreads) void k_cpcg_a(BoxDims b, int it, const double *__restrict__ S,
                                                const double *__restrict__ z, const double *__restrict__ p0,
                                                double *__restrict__ p1, double *__restrict__ Ap,
                                                const double *__restrict__ prz, double *__restrict__ ppAp,
                                                CoarseScalars *sc)
{
    __shared__ double sh[4], sh2[4];
    const int Cx = b.nx + 1, Cy = b.ny + 1, Cz = b.nz + 1;
    const int64_t n1 = (int64_t)Cx * Cy * Cz;
    const double rz = coarse_total(prz, sh), old = it > 0 ? sc->rz[(it - 1) & 1] : 0.0;
    const double beta = old > 0.0 ? rz / old : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->rz[it & 1] = rz;
    double v = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kCoarseThreads + threadIdx.x; i < n1; i += (int64_t)gridDim.x * kCoarseThreads) {
        const uint32_t i32 = (uint32_t)i, K = i32 / (uint32_t)(Cx * Cy), R = i32 - K * (uint32_t)(Cx * Cy);
        const int J = R / (uint32_t)Cx, I = R - J * (uint32_t)Cx;
        double acc = 0.0;
#pragma unroll
        for (int s = 0; s < 27; ++s) {
            const int dx = s % 3 - 1, dy = (s / 3) % 3 - 1, dz = s / 9 - 1;
            const bool in = (unsigned)(I + dx) < (unsigned)Cx && (unsigned)(J + dy) < (unsigned)Cy &&
                            (unsigned)((int)K + dz) < (unsigned)Cz;
            const int64_t j = in ? i + dx + (int64_t)Cx * (dy + Cy * dz) : i;
            const double w = z[j] + beta * p0[j];
            acc = fma(S[s * n1 + i], in ? w : 0.0, acc);
        }
        const double pi = z[i] + beta * p0[i];
        p1[i] = pi;
        Ap[i] = acc;
        v = fma(pi, acc, v);
    }
    v = coarse_sum(v, sh2);
    if (threadIdx.x == 0) ppAp[blockIdx.x] = v;
}

// alpha = rz / (p1 . Ap); u += alpha p1; r -= alpha Ap; z = dinv r; partial sums of r.z
__global__ __launch_bounds__(kCoarseThreads) void k_cpcg_b(int64_t n1, int it, const double *__restrict__ dinv,
                                                const double *__restrict__ p1, const double *__restrict__ Ap,
                                                double *__restrict__ u, double *__restrict__ r,
                                                double *__restrict__ z, const double *__restrict__ ppAp,
                                                double *__restrict__ prz, const CoarseScalars *__restrict__ sc)
{
    __shared__ double sh[4], sh2[4];
    const double pAp = coarse_total(ppAp, sh);
    const double alpha = pAp > 0.0 ? sc->rz[it & 1] / pAp : 0.0;
    double v = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kCoarseThreads + threadIdx.x; i < n1; i += (int64_t)gridDim.x * kCoarseThreads) {
        u[i] = fma(alpha, p1[i], u[i]);
        const double ri = fma(-alpha, Ap[i], r[i]);
        r[i] = ri;
        const double zi = dinv[i] * ri;
        z[i] = zi;
        v = fma(ri, zi, v);
    }
    v = coarse_sum(v, sh2);
    if (threadIdx.x == 0) prz[blockIdx.x] = v;
}

// ---------------------------------------------------------------- FP16 MFMA inference
// The whole network part z += W G^T (s_e NN(G_e r / s_e, log kappa_e)) for one element per
// workgroup: gather and RMS-normalise the residual tile, three convolutions as implicit
// GEMMs on v_mfma_f32_16x16x16f16 (FP16 operands, FP32 accumulation), and the averaged
// scatter.  Layers 1 and 2 compute Y^T = W^T X^T: GEMM rows are the 16 output channels,
// columns 16 tile points (one row tile of the tile), and one k-step of 16 is one tap's 16
// input channels (layer 1: four taps of the two input channels padded to four).  Lane
// layout (pinned by the 16-bit lane-layout test): A lane l holds A[l%16][4(l/16)+t], B
// lane l holds B[4(l/16)+t][l%16], result lane l element v is D[4(l/16)+v][l%16], so a
// lane reads and writes four consecutive channels of one point.  Activations live in LDS
// as [padded point][channel] FP16 on the (N+2)^3 grid with a zero halo, so every shifted
// operand read is one 8-byte load.  Layer 3 (16 -> 1) is Y[pt][tap] = sum_c a2[pt][c]
// W3[c][tap] on MFMA followed by out[pt] = b3 + sum_tap Y[pt + off(tap)][tap] over the taps
// that stay in the tile.
typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
constexpr int kPackL1 = 7, kPackL2 = 27, kPackL3 = 2, kPackSteps = kPackL1 + kPackL2 + kPackL3;

// Weight tables in lane order: step s, lane l -> 4 halves, entry (k = 4(l/16)+t, output
// channel l%16): the A-operand of layers 1-2 (row = output channel) and the B-operand of
// layer 3 (column = tap).
__global__ void k_pack16(const float *__restrict__ prm, h4_t *__restrict__ wp)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kPackSteps * 64) return;
    const int s = i / 64, l = i % 64, g = l >> 4, col = l & 15;
    h4_t w;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float v = 0.f;
        if (s < kPackL1) {  // rows = (tap 4s+g, channel t): W1[o][t][tap], channels 2, 3 zero
            const int tap = 4 * s + g;
            if (t < kNetCin && tap < 27) v = prm[kNetOffW1 + (col * kNetCin + t) * 27 + tap];
        } else if (s < kPackL1 + kPackL2) {  // rows = channel 4g+t of tap s-7: W2[o][c][tap]
            const int tap = s - kPackL1, c = 4 * g + t;
            v = prm[kNetOffW2 + (col * kNetCh + c) * 27 + tap];
        } else {  // rows = channel 4g+t, columns = taps 16 ct + col: W3[0][c][tap]
            const int ct = s - kPackL1 - kPackL2, c = 4 * g + t, tap = 16 * ct + col;
            if (tap < 27) v = prm[kNetOffW3 + c * 27 + tap];
        }
        w[t] = (_Float16)v;
    }
    wp[i] = w;
}

template <int N>
struct Pad {
    static constexpr int P = N * N * N, NP = N + 2, NP3 = NP * NP * NP, RT = (P + 15) / 16;
    __host__ __device__ static constexpr int off(int tap)
    {
        return (tap % 3 - 1) + NP * ((tap / 3) % 3 - 1) + NP * NP * (tap / 9 - 1);
    }
    // the same neighbour in the unpadded tile
    __host__ __device__ static constexpr int toff(int tap)
    {
        return (tap % 3 - 1) + N * ((tap / 3) % 3 - 1) + N * N * (tap / 9 - 1);
    }
    __device__ static int pad(int pt)
    {
        const int i = pt % N, j = (pt / N) % N, k = pt / (N * N);
        return (i + 1) + NP * ((j + 1) + NP * (k + 1));
    }
    __device__ static bool halo(int q)
    {
        const int i = q % NP, j = (q / NP) % NP, k = q / (NP * NP);
        return i == 0 || j == 0 || k == 0 || i == NP - 1 || j == NP - 1 || k == NP - 1;
    }
};

template <int N>
__global__ __launch_bounds__(256, 2) void k_net16(int64_t nelem, const double *__restrict__ r,
                                                  const int32_t *__restrict__ emap, const float *__restrict__ logk,
                                                  const h4_t *__restrict__ wp, const float *__restrict__ prm,
                                                  const double *__restrict__ inv_mult, double scale,
                                                  double *__restrict__ z)
{
    // One element per workgroup of four waves: wave w owns GEMM row tiles w, w + 4, ...
    // (16 tile points each), so each wave keeps few operands in flight and several
    // workgroups share a CU.  Every tile point belongs to one thread in the gather,
    // normalisation, layer-3 tap sum and scatter (P <= 256).  The layer-3 table is stored
    // tap-major with an odd row pitch (in 4-byte words), so the 27 shifted reads of a wave
    // hit distinct LDS banks.
    using T = Pad<N>;
    constexpr int P = T::P, NP3 = T::NP3, RT = T::RT;
    constexpr int YP = 16 * RT + 2;  // row pitch of the layer-3 table (halves; odd in words)
    static_assert(P <= 256, "one tile point per thread");
    __shared__ h4_t x0b[NP3];      // [point] (r/s, log kappa, 0, 0)
    __shared__ h4_t a1b[NP3 * 4];  // [point][channel group of 4]
    __shared__ h4_t a2b[NP3 * 4];
    __shared__ _Float16 yb[32 * YP];  // layer-3 table [tap][row]
    __shared__ double red[4];
    const int tid = threadIdx.x, l = tid & 63, g = l >> 4, col = l & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const h4_t zero4 = {0, 0, 0, 0};
    for (int i = tid; i < NP3; i += 256) {
        x0b[i] = zero4;
#pragma unroll
        for (int k = 0; k < 4; ++k) a1b[i * 4 + k] = a2b[i * 4 + k] = zero4;
    }
    h4_t w1[kPackL1], w2[kPackL2], w3[kPackL3];
#pragma unroll
    for (int s = 0; s < kPackL1; ++s) w1[s] = wp[s * 64 + l];
#pragma unroll
    for (int s = 0; s < kPackL2; ++s) w2[s] = wp[(kPackL1 + s) * 64 + l];
#pragma unroll
    for (int s = 0; s < kPackL3; ++s) w3[s] = wp[(kPackL1 + kPackL2 + s) * 64 + l];
    // Layers 1 and 2 run transposed (D^T = W^T X^T: the packed weights as the A-operand, the
    // activations as the B-operand), so each lane ends with four consecutive output
    // channels 4g..4g+3 of one tile point and stores them with one 8-byte write.
    float bias1[4], bias2[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        bias1[v] = prm[kNetOffB1 + 4 * g + v];
        bias2[v] = prm[kNetOffB2 + 4 * g + v];
    }
    const float bias3 = prm[kNetOffB3];
    constexpr int MT = (RT + 3) / 4;  // row tiles per wave (the last ones may be absent)
    // A wave's tiles past RT (only when RT is not a multiple of 4) compute on clamped rows
    // and store nothing: the MFMA loops carry no per-tile branches.
    int rb[MT];                        // padded index of this lane's A-operand row (dummy rows repeat the last point)
    int op[MT];                        // padded index of the point whose channels this lane stores, -1 past the tile
    bool tv[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int rt = wave + 4 * m;
        tv[m] = rt < RT;
        rb[m] = T::pad(min(16 * rt + col, P - 1));
        op[m] = (tv[m] && 16 * rt + col < P) ? rb[m] : -1;
    }
    int o1[kPackL1];  // layer-1 tap offset of this lane's k-group in every k-step (taps past 26: zero weights)
#pragma unroll
    for (int s = 0; s < kPackL1; ++s) o1[s] = 4 * s + g < 27 ? T::off(4 * s + g) : 0;
    const bool own = tid < P;  // this thread's tile point
    const int pp = own ? T::pad(tid) : 0;
    uint32_t inmask = 0;  // bit tap: the neighbour (tap) of this thread's point lies in the tile
    {
        const int pi = tid % N, pj = (tid / N) % N, pk = tid / (N * N);
#pragma unroll
        for (int tap = 0; tap < 27; ++tap) {
            const int dx = tap % 3 - 1, dy = (tap / 3) % 3 - 1, dz = tap / 9 - 1;
            if ((unsigned)(pi + dx) < (unsigned)N && (unsigned)(pj + dy) < (unsigned)N && (unsigned)(pk + dz) < (unsigned)N)
                inmask |= 1u << tap;
        }
    }
    __syncthreads();

    for (int64_t e = blockIdx.x; e < nelem; e += gridDim.x) {
        // gather r, element RMS
        int32_t gi = 0;
        double rv = 0.0;
        float lk = 0.f;
        if (own) {
            gi = emap[e * P + tid];
            rv = r[gi];
            lk = logk[e * P + tid];
        }
        double ss = rv * rv;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m);
        if (l == 0) red[wave] = ss;
        __syncthreads();
        ss = (red[0] + red[1]) + (red[2] + red[3]);
        const double rms = sqrt(ss / P);
        const double sc = rms > 0.0 ? rms : 1.0;

        // the network on +r and on -r; the preconditioner takes the odd part
        float odd = 0.f;
#pragma unroll 1
        for (int sgn = 0; sgn < 2; ++sgn) {
            if (own) {
                const h4_t v = {(_Float16)(float)((sgn ? -rv : rv) / sc), (_Float16)lk, (_Float16)0.f, (_Float16)0.f};
                x0b[pp] = v;
            }
            __syncthreads();
            f4_t acc[MT];
            // layer 1: 2 (padded to 4) -> 16 channels, ReLU
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < kPackL1; ++s)
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x16f16(w1[s], x0b[rb[m] + o1[s]], acc[m], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < MT; ++m)
                if (op[m] >= 0) {
                    h4_t h;
#pragma unroll
                    for (int v = 0; v < 4; ++v) h[v] = (_Float16)fmaxf(acc[m][v] + bias1[v], 0.f);
                    a1b[op[m] * 4 + g] = h;
                }
            __syncthreads();
            // layer 2: 16 -> 16, one tap per k-step, ReLU; a compiler barrier before each tap
            // keeps the compiler from hoisting all 27 taps' operand loads (registers): measured
            // faster than chunks of 3, 9 or 27 taps
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s0 = 0; s0 < 27; s0 += 1) {
                asm volatile("" ::: "memory");
#pragma unroll
                for (int s = s0; s < s0 + 1; ++s)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f32_16x16x16f16(w2[s], a1b[(rb[m] + T::off(s)) * 4 + g],
                                                                       acc[m], 0, 0, 0);
            }
#pragma unroll
            for (int m = 0; m < MT; ++m)
                if (op[m] >= 0) {
                    h4_t h;
#pragma unroll
                    for (int v = 0; v < 4; ++v) h[v] = (_Float16)fmaxf(acc[m][v] + bias2[v], 0.f);
                    a2b[op[m] * 4 + g] = h;
                }
            __syncthreads();
            // layer 3, part 1: Y[pt][tap] for every tile point and tap (rows past the tile unused)
#pragma unroll
            for (int ct = 0; ct < kPackL3; ++ct)
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const f4_t y = __builtin_amdgcn_mfma_f32_16x16x16f16(a2b[rb[m] * 4 + g], w3[ct],
                                                                         (f4_t){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    if (tv[m])
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            yb[(16 * ct + col) * YP + 16 * (wave + 4 * m) + 4 * g + v] = (_Float16)y[v];
                }
            __syncthreads();
            // layer 3, part 2: shifted sum over taps (the bias cancels in the odd part)
            if (own) {
                float o = bias3;
#pragma unroll
                for (int tap = 0; tap < 27; ++tap) {
                    const bool in = (inmask >> tap) & 1u;
                    const float yv = (float)yb[tap * YP + (in ? tid + T::toff(tap) : tid)];
                    o = in ? o + yv : o;
                }
                odd += sgn ? -0.5f * o : 0.5f * o;
            }
            // the next writes of x0b, a1 and yb come after the barrier at the top of the
            // next evaluation (x0b) or after further barriers (a1, yb)
        }
        // averaged scatter
        if (own) unsafeAtomicAdd(z + gi, (double)odd * sc * scale * inv_mult[gi]);
    }
}

}  // namespace

int64_t nn_pack16_bytes() { return (int64_t)kPackSteps * 64 * sizeof(h4_t); }

hipError_t nn_infer16(int n, int64_t nelem, const float *params, void *wpack, const double *r, const int32_t *emap,
                      const float *logk, const double *inv_mult, double scale, double *z, hipStream_t s)
{
    if (nelem <= 0) return hipSuccess;
    h4_t *wp = static_cast<h4_t *>(wpack);
    hipLaunchKernelGGL(k_pack16, dim3((kPackSteps * 64 + 255) / 256), dim3(256), 0, s, params, wp);
    // persistent workgroups (one element at a time each): enough to fill every CU several times over
    const unsigned nb = (unsigned)std::min<int64_t>(nelem, 256 * 8);
    if (n == 3) hipLaunchKernelGGL(k_net16<3>, dim3(nb), dim3(256), 0, s, nelem, r, emap, logk, wp, params, inv_mult, scale, z);
    else if (n == 4) hipLaunchKernelGGL(k_net16<4>, dim3(nb), dim3(256), 0, s, nelem, r, emap, logk, wp, params, inv_mult, scale, z);
    else if (n == 5) hipLaunchKernelGGL(k_net16<5>, dim3(nb), dim3(256), 0, s, nelem, r, emap, logk, wp, params, inv_mult, scale, z);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t nn_inv_mult(int n, int64_t nelem, int64_t ndof, const int32_t *emap, double *inv_mult, hipStream_t s)
{
    const int64_t tot = nelem * n * n * n;
    hipError_t e = vec_fill(inv_mult, 0.0, ndof, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_count, dim3(nblk(tot)), dim3(256), 0, s, tot, emap, inv_mult);
    hipLaunchKernelGGL(k_recip_or_zero, dim3(nblk(ndof)), dim3(256), 0, s, ndof, inv_mult);
    return hipGetLastError();
}

hipError_t nn_adam(float *p, float *g, float *m, float *v, int n, double lr, int step, hipStream_t s)
{
    const double bc1 = 1.0 - std::pow(0.9, step), bc2 = 1.0 - std::pow(0.999, step);
    hipLaunchKernelGGL(k_adam, dim3(nblk(n)), dim3(256), 0, s, p, g, m, v, n, (float)lr, (float)bc1, (float)bc2);
    return hipGetLastError();
}

hipError_t vec_fill_f32(float *y, float v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)std::min<int64_t>(nblk(n), 8192)), dim3(256), 0, s, y, v, n);
    return hipGetLastError();
}

hipError_t vec_sub(double *y, const double *a, const double *b, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_sub, dim3((unsigned)std::min<int64_t>(nblk(n), 8192)), dim3(256), 0, s, y, a, b, n);
    return hipGetLastError();
}
hipError_t vec_mul(double *y, const double *a, const double *b, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mul, dim3((unsigned)std::min<int64_t>(nblk(n), 8192)), dim3(256), 0, s, y, a, b, n);
    return hipGetLastError();
}

hipError_t vec_loss_scale(double *g, int64_t n, double *sc, hipStream_t s)
{
    hipLaunchKernelGGL(k_loss_scale, dim3((unsigned)std::min<int64_t>(nblk(n), 8192)), dim3(256), 0, s, g, n, sc);
    return hipGetLastError();
}

hipError_t coarse_prolong(const BoxDims &b, const double *gll, const double *u1, double *uf, const double *m1,
                          const double *m2, hipStream_t s)
{
    const int64_t nf = ((int64_t)b.nx * b.p + 1) * ((int64_t)b.ny * b.p + 1) * ((int64_t)b.nz * b.p + 1);
    hipLaunchKernelGGL(k_prolong, dim3(nblk(nf)), dim3(256), 0, s, b, gll, u1, uf, m1, m2);
    return hipGetLastError();
}

hipError_t coarse_restrict(const BoxDims &b, const double *gll, const double *rf, double *r1, double *t1, double *t2,
                           hipStream_t s)
{
    const int64_t Mx = (int64_t)b.nx * b.p + 1, My = (int64_t)b.ny * b.p + 1, Mz = (int64_t)b.nz * b.p + 1;
    const int64_t Cx = b.nx + 1, Cy = b.ny + 1, Cz = b.nz + 1;
    hipLaunchKernelGGL(k_restrict_axis, dim3(nblk(Cx * My * Mz)), dim3(256), 0, s, 0, b.nx, b.p, Mx, My, Mz, gll, rf, t1);
    hipLaunchKernelGGL(k_restrict_axis, dim3(nblk(Cx * Cy * Mz)), dim3(256), 0, s, 1, b.ny, b.p, Cx, My, Mz, gll, t1, t2);
    hipLaunchKernelGGL(k_restrict_axis, dim3(nblk(Cx * Cy * Cz)), dim3(256), 0, s, 2, b.nz, b.p, Cx, Cy, Mz, gll, t2, r1);
    return hipGetLastError();
}

hipError_t coarse_probe_vec(const BoxDims &b, int cls, double *v, hipStream_t s)
{
    const int64_t n1 = (int64_t)(b.nx + 1) * (b.ny + 1) * (b.nz + 1);
    hipLaunchKernelGGL(k_probe_vec, dim3(nblk(n1)), dim3(256), 0, s, b, cls, v);
    return hipGetLastError();
}

hipError_t coarse_probe_gather(const BoxDims &b, int cls, const double *y, const uint8_t *ess1, double *S,
                               hipStream_t s)
{
    const int64_t n1 = (int64_t)(b.nx + 1) * (b.ny + 1) * (b.nz + 1);
    hipLaunchKernelGGL(k_probe_gather, dim3(nblk(n1)), dim3(256), 0, s, b, cls, y, ess1, S);
    return hipGetLastError();
}

hipError_t coarse_dinv(int64_t n1, const double *S, double *dinv, hipStream_t s)
{
    hipLaunchKernelGGL(k_dinv_center, dim3(nblk(n1)), dim3(256), 0, s, n1, S, dinv);
    return hipGetLastError();
}

hipError_t coarse_pcg(const BoxDims &b, const double *S, const double *dinv, double *r1, double *u, double *z,
                      double *p0, double *p1, double *Ap, double *partial, CoarseScalars *sc, int iters,
                      hipStream_t s)
{
    const int64_t n1 = (int64_t)(b.nx + 1) * (b.ny + 1) * (b.nz + 1);
    const unsigned nb = (unsigned)std::min<int64_t>((n1 + kCoarseThreads - 1) / kCoarseThreads, kCoarseBlocks);
    double *prz = partial, *ppAp = partial + kCoarseBlocks;
    hipLaunchKernelGGL(k_cpcg_init, dim3(nb), dim3(kCoarseThreads), 0, s, n1, dinv, r1, u, z, p0, prz);
    for (int k = 0; k < iters; ++k) {
        double *pin = (k & 1) ? p1 : p0, *pout = (k & 1) ? p0 : p1;
        hipLaunchKernelGGL(k_cpcg_a, dim3(nb), dim3(kCoarseThreads), 0, s, b, k, S, z, pin, pout, Ap, prz, ppAp, sc);
        hipLaunchKernelGGL(k_cpcg_b, dim3(nb), dim3(kCoarseThreads), 0, s, n1, k, dinv, pout, Ap, u, r1, z, ppAp, prz, sc);
    }
    return hipGetLastError();
}

}  // namespace hexpa
