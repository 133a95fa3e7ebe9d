// Fused FP64 apply on the vector ALU with the z contractions in registers (orders p <= 4).
//
// A thread owns one z-pencil (a, b) of an element: it reads the D values of each tensor that
// the x and y contractions left there, forms the gradient (and value) at the pencil's Q
// quadrature points, multiplies by D, which it holds for the pencil's points, contracts back
// along z and writes the D results where it read.  The quadrature-point tensor, the largest
// one (3 Q^3 values an element), never reaches LDS, nor do two passes and two barriers of the
// pass-by-pass kernel; the transposed y and x contractions read the result at a stride.
// At p = 4 an element moves 2.3x fewer LDS bytes.
//
// D of the pencil is loaded for the next group of elements right after it has been used, so a
// whole group of D per workgroup is in flight from one D-step to the next.  sched_barriers keep
// the z stage's LDS reads beside their use (241 -> 161 registers at p = 4, Q = 6).
//
// Pass by pass -> this kernel, us, at about 20 M DOFs: mass p = 2 / 3 / 4 with Q = p + 1
// 396 / 375 / 263 -> 343 / 291 / 254, with Q = p + 2 471 / 869 / 316 -> 405 / 357 / 283;
// diffusion p = 3, Q = 4 771 -> 615, p = 4, Q = 5 622 -> 528; both p = 2, Q = 4 1718 -> 1600.
// What bounds it now: memory.  Diffusion at p = 4, Q = 5, 78^3 takes 901 us, 730 without the
// scatter's atomics; at p = 2, Q = 4, 155^3 2490 and 1842 (6.1 TB/s, the rate of a plain read).
// A wave of its own for the scatter, whose atomics no load then waits behind, changed nothing
// (2445), nor did longer runs of elements a workgroup (4 to 24: 2490 - 2530).
#pragma once
#include "apply_passes.h"

namespace hexpa {

template <int D, int Q, int OPS>
struct PencilShape {
    static constexpr bool kMass = (OPS & 1) != 0, kDiff = (OPS & 2) != 0;
    static constexpr int NC = kDiff ? (kMass ? 7 : 6) : 1;  // stored D values per point
    static constexpr int NCH = kDiff ? 3 : 1;  // tensors: B_y B_x, G_y B_x, B_y G_x (mass alone: the first)
    static constexpr int Q2 = Q * Q, Q3 = Q2 * Q, D2 = D * D, D3 = D2 * D;
    // Workgroup: one pencil a thread.  Mass alone has little arithmetic and registers to spare:
    // long runs of elements, whose inner faces are added before the scatter (p = 3, Q = 4 with
    // 64 and 256 threads 362 and 291 us).  Else as few waves at a barrier as leave few idle
    // (diffusion p = 4, Q = 5 with 128 and 256: 528 and 557).
    static constexpr int NT = !kDiff ? 256 : Q2 <= 16 ? 64 : 128;
    static constexpr int E = NT / Q2;
    static constexpr int DP = pad_stride(D);
    static constexpr int SR = DP * Q;  // stride of the slow index (b, then j) of the tensors
    static constexpr int SZ_A = cmax(D2 * DP, NCH * Q * SR) | 1;
    static constexpr int SZ_B = cmax((kDiff ? 2 * Q : Q) * D * DP, (kDiff ? 2 : 1) * D * SR) | 1;
    static constexpr int NM = (E * D3 + NT - 1) / NT;  // nodes per thread
    // waves per SIMD the registers are limited for; the sixth and seventh D value spill at p = 4
    static constexpr int MINW = NC == 7 && D == 5 ? 2 : 3;
    // (mass at p = 4, Q = 6: 469 us with non-temporal loads, 483 without)
    static constexpr bool WHOLE_LINES = !kDiff || Q2 % 16 == 0;
    // Where it is the faster one.  With Q = p + 2 a thread of diffusion holds 6 (p + 2) D values
    // for its pencil against 6 (p + 2)^3 E / NT in the pass-by-pass kernel, which then keeps more
    // waves resident (p = 1 / 2 / 3 / 4: 2430 / 1381 / 1126 / 725 there, 2748 / 1390 / 1175 / 763
    // here), and so at p <= 2 with Q = p + 1 (805 / 801 and 1055 / 879); with the mass term the
    // pass-by-pass kernel has a fourth tensor and loses at p = 2, Q = 4, too.  Mass at p = 1 with
    // Q = 3 is even (577 and 595).  So is diffusion at p = 2, Q = 4 on smaller meshes, there and
    // here: 24^3 12.0 and 13.1, 32^3 24.6 and 25.8, 50^3 85.0 and 81.5, 100^3 640 and 625, 155^3
    // 2468 and 2534.
    static constexpr bool ok =
        D <= 5 && (kDiff ? (Q == D && D >= 4) || (kMass && D == 3 && Q == 4) : D >= 3 || Q == D);
};

template <int D, int Q, int OPS>
__global__ __launch_bounds__((PencilShape<D, Q, OPS>::NT), (PencilShape<D, Q, OPS>::MINW)) void k_apply_pencil(
    int nelem, int ngroups, const int32_t *__restrict__ emap, const double *__restrict__ qd,
    const DevTables *__restrict__ tables, const double *__restrict__ x, double *__restrict__ y)
{
    using S = PencilShape<D, Q, OPS>;
    constexpr bool M = S::kMass, DF = S::kDiff;
    constexpr int E = S::E, NT = S::NT, NC = S::NC, NM = S::NM, DP = S::DP, SR = S::SR;
    constexpr int D2 = S::D2, D3 = S::D3, Q2 = S::Q2, Q3 = S::Q3, CH = Q * SR, PT = D * SR;
    __shared__ double bufA[E * S::SZ_A], bufB[E * S::SZ_B];
    __shared__ int32_t lmap[E * D3];
    const int tid = threadIdx.x;
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };  // LDS traffic only

    // The basis is read from the constant cache by each stage; kept across stages it would
    // not fit the scalar registers.
    auto tables_here = [&] {
        int o = 0;
        asm volatile("" : "+s"(o));
        return tables + o;
    };

    int g = blockIdx.x;
    if (g >= ngroups) return;
    // this thread's pencil
    const int pe = min(tid / Q2, E - 1), pn = tid - pe * Q2;
    const bool pencil = tid < E * Q2;
    double *pen = bufA + pe * S::SZ_A + (pencil ? pn : 0) * DP;
    double dq[NC][Q];
    auto load_d = [&](int gg) {
        const int64_t e = min(gg * E + pe, nelem - 1);
        const double *p = qd + e * (NC * Q3) + (pencil ? pn : 0);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int z = 0; z < Q; ++z) dq[c][z] = load_once<S::WHOLE_LINES>(p + c * Q3 + z * Q2);
    };
    // maps and x in row order (node row, element, i): consecutive DOFs of a group's neighbours
    auto load_map = [&](int32_t (&m)[NM], int gg) {
        const int e0 = gg * E, nv = gg < ngroups ? min(E, nelem - e0) : 0;
#pragma unroll
        for (int s = 0; s < NM; ++s) {
            const int L = tid + s * NT;
            int e, I;
            row_node<D, E>(L, e, I);
            m[s] = L < E * D3 && e < nv ? emap[(int64_t)(e0 + e) * D3 + I] : -1;
        }
    };
    auto load_x = [&](double (&v)[NM], const int32_t (&m)[NM]) {
#pragma unroll
        for (int s = 0; s < NM; ++s) v[s] = m[s] >= 0 ? x[m[s]] : 0.0;
    };
    int32_t mcur[NM], mnext[NM];
    double xv[NM];
    load_d(g);
    load_map(mcur, g);
    load_x(xv, mcur);

    for (;;) {
        const int gn = g + gridDim.x;
        const bool more = gn < ngroups;
#pragma unroll
        for (int s = 0; s < NM; ++s) {
            const int L = tid + s * NT;
            if (L < E * D3) {
                int e, I;
                row_node<D, E>(L, e, I);
                lmap[e * D3 + I] = mcur[s];
                bufA[e * S::SZ_A + I + (DP - D) * (I / D)] = xv[s];
            }
        }
        load_map(mnext, more ? gn : ngroups);
        barrier();

        // x and y axes
        const DevTables *tab = tables_here();
        if constexpr (DF) {
            valu_pass<DF1<D, Q, M>, E, NT>(bufA, S::SZ_A, tab, LdsOut<double>{bufB, S::SZ_B}, tid);
            barrier();
            tab = tables_here();
            valu_pass<DF2a<D, Q, M>, E, NT>(bufB, S::SZ_B, tab, LdsOut<double>{bufA, S::SZ_A}, tid);
            valu_pass<DF2b<D, Q, M>, E, NT>(bufB, S::SZ_B, tab, LdsOut<double>{bufA, S::SZ_A}, tid);
        } else {
            valu_pass<MF1<D, Q>, E, NT>(bufA, S::SZ_A, tab, LdsOut<double>{bufB, S::SZ_B}, tid);
            barrier();
            tab = tables_here();
            valu_pass<MF2<D, Q>, E, NT>(bufB, S::SZ_B, tab, LdsOut<double>{bufA, S::SZ_A}, tid);
        }
        load_x(xv, mnext);  // the next group's map has had the passes to arrive
        barrier();

        // z axis, D, transposed z axis
        tab = tables_here();
        {
            double vx[DF ? Q : 1], vy[DF ? Q : 1], vz[DF ? Q : 1], vu[M ? Q : 1];
#pragma unroll
            for (int z = 0; z < Q; ++z) {
                if constexpr (DF) vx[z] = vy[z] = vz[z] = 0.0;
                if constexpr (M) vu[z] = 0.0;
            }
#pragma unroll
            for (int k = 0; k < D; ++k) {
                const double c0 = pen[k];
                double c1 = 0.0, c2 = 0.0;
                if constexpr (DF) {
                    c1 = pen[CH + k];
                    c2 = pen[2 * CH + k];
                }
#pragma unroll
                for (int z = 0; z < Q; ++z) {
                    const double b = tB(tab, z, k, D);
                    if constexpr (DF) {
                        vz[z] = fma(tG(tab, z, k, D), c0, vz[z]);
                        vy[z] = fma(b, c1, vy[z]);
                        vx[z] = fma(b, c2, vx[z]);
                    }
                    if constexpr (M) vu[z] = fma(b, c0, vu[z]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int z = 0; z < Q; ++z) {
                if constexpr (DF) {
                    const double g0 = vx[z], g1 = vy[z], g2 = vz[z];
                    vx[z] = dq[0][z] * g0 + dq[1][z] * g1 + dq[2][z] * g2;
                    vy[z] = dq[1][z] * g0 + dq[3][z] * g1 + dq[4][z] * g2;
                    vz[z] = dq[2][z] * g0 + dq[4][z] * g1 + dq[5][z] * g2;
                }
                if constexpr (M) vu[z] *= dq[NC - 1][z];
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);
            load_d(more ? gn : g);
            __builtin_amdgcn_sched_barrier(0);
            tab = tables_here();
#pragma unroll
            for (int k = 0; k < D; ++k) {
                double w0 = 0.0, w1 = 0.0, w2 = 0.0;
#pragma unroll
                for (int z = 0; z < Q; ++z) {
                    const double b = tB(tab, z, k, D);
                    if constexpr (DF) {
                        w0 = fma(tG(tab, z, k, D), vz[z], w0);
                        w1 = fma(b, vy[z], w1);
                        w2 = fma(b, vx[z], w2);
                    }
                    if constexpr (M) w0 = fma(b, vu[z], w0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (pencil) {
                    pen[k] = w0;
                    if constexpr (DF) {
                        pen[CH + k] = w1;
                        pen[2 * CH + k] = w2;
                    }
                }
            }
        }
        barrier();

        tab = tables_here();
        // transposed y axis, columns (k, a): p1 = B^T W0 + G^T W1, p0 = B^T W2
        for (int c = tid; c < E * Q * D; c += NT) {
            const int e = c / (Q * D), q = c - e * (Q * D), a = q / D, k = q - a * D;
            const double *w = bufA + e * S::SZ_A + a * DP + k;
            double p1[D], p0[DF ? D : 1];
#pragma unroll
            for (int j = 0; j < D; ++j) {
                p1[j] = 0.0;
                if constexpr (DF) p0[j] = 0.0;
            }
#pragma unroll
            for (int b = 0; b < Q; ++b) {
                const double w0 = w[b * SR];
                double w1 = 0.0, w2 = 0.0;
                if constexpr (DF) {
                    w1 = w[CH + b * SR];
                    w2 = w[2 * CH + b * SR];
                }
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    p1[j] = fma(tB(tab, b, j, D), w0, p1[j]);
                    if constexpr (DF) {
                        p1[j] = fma(tG(tab, b, j, D), w1, p1[j]);
                        p0[j] = fma(tB(tab, b, j, D), w2, p0[j]);
                    }
                }
            }
            double *o = bufB + e * S::SZ_B + a * DP + k;
#pragma unroll
            for (int j = 0; j < D; ++j) {
                o[j * SR] = p1[j];
                if constexpr (DF) o[PT + j * SR] = p0[j];
            }
        }
        barrier();

        tab = tables_here();
        // transposed x axis, columns (k, j): y = B^T p1 + G^T p0, in node order
        for (int c = tid; c < E * D2; c += NT) {
            const int e = c / D2, q = c - e * D2, j = q / D, k = q - j * D;
            const double *p = bufB + e * S::SZ_B + j * SR + k;
            double o[D];
#pragma unroll
            for (int i = 0; i < D; ++i) o[i] = 0.0;
#pragma unroll
            for (int a = 0; a < Q; ++a) {
                const double p1 = p[a * DP];
                double p0 = 0.0;
                if constexpr (DF) p0 = p[PT + a * DP];
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    o[i] = fma(tB(tab, a, i, D), p1, o[i]);
                    if constexpr (DF) o[i] = fma(tG(tab, a, i, D), p0, o[i]);
                }
            }
            double *yo = bufA + e * S::SZ_A + D * j + D2 * k;
#pragma unroll
            for (int i = 0; i < D; ++i) yo[i] = o[i];
        }
        barrier();
        scatter_group<D, E, NT, S::SZ_A, true>(bufA, lmap, y, tid);
        if (!more) break;
        barrier();  // x and the map are rewritten by the next group
        g = gn;
#pragma unroll
        for (int s = 0; s < NM; ++s) mcur[s] = mnext[s];
    }
}

}  // namespace hexpa
