// Fused FP64 apply with chained MFMA contractions (orders p >= 5): one element per workgroup.
//
// The contractions of an element form a chain in which the result of one MFMA is an operand of
// the next without leaving its registers.  v_mfma_f64_4x4x4f64 (four independent 4x4x4
// products; block beta = (l >> 2) & 3, r = l & 3, h = l >> 4) takes A_beta[r][h] and
// B_beta[h][r] from lane l and returns D_beta[h][r]: the row of a result sits where an operand
// has its contracted index.  With the data as the A-operand the untouched row index moves to h;
// with the data as the B-operand the new index does.  So, for four z-planes at a time (block =
// plane),
//     X[j = r][i = h] as A, basis B[i = h][a = r]   ->  P[j = h][a = r]     (x axis)
//     basis A[b = r][j = h], P as B                 ->  U[b = h][a = r]     (y axis)
// is one chain, for sixteen columns n = (a, b)
//     basis A[c = r][k = h], U[k = h][n] as B       ->  g[c = h][n]         (z axis)
//     v = D g at the quadrature points, lane by lane
//     basis A[k = r][c = h], v as B                 ->  W[k = h][n]         (z^T)
// is another, and for four planes again
//     W[b = r][a = h] as A, basis B[a = h][i = r]   ->  R[b = h][i = r]     (x^T)
//     basis A[j = r][b = h], R as B                 ->  Y[j = h][i = r]     (y^T)
// is the third.  Only U and W, D Q^2 values per channel, pass through LDS (W in the place of
// U), against every intermediate of the pass-by-pass kernel, and three barriers an element are
// left of its eight.  All six contractions take their basis operand as B[4 tq + r][4 td + h]
// (forward) or B[4 tq + h][4 td + r] (transposed), or the same of G.
//
// The waves share an element evenly: a wave takes one 4-wide strip of a (forward) or i
// (transposed) of a plane group, and one 16-column tile of the z chain, whose D values (one
// tile: 12-18 doubles a lane) it loads for the next element as soon as it has used this one's,
// so that a whole element of D per workgroup is in flight from one D-step to the next.  When
// one plane is left over (D = 9), its blocks are the strips instead of planes and one wave
// takes it whole: at p = 8, 6 + 1 units of 45 MFMAs and 7 column tiles are seven waves' work.
//
// The pass-by-pass kernel with its operands through LDS (k_apply_dma) spent 80 % of a group's
// time in its chain of passes and 2-3 % waiting for memory.  At about 30 M DOFs (Q = p + 2;
// p = 5 / 6 / 7 / 8, kernel alone): diffusion 1556 / 1073 / 1193 / 1186 -> 1227 / 918 / 1161 /
// 1122 us, mass (MFMA) 746 / 508 / 544 / 566 -> 452 / 390 / 461 / 457, both 1744 / 1237 / 1552 /
// 1752 -> 1418 / 1027 / 1353 / 1272; with plain loads of D where its rows are not whole lines
// diffusion at p = 5 / 7 / 8 1022 / 1035 / 1057 (all orders timed with both load kinds at
// load_once).  What bounds it now: at p = 6 memory (4.6 TB/s; without
// the scatter's atomics, which are carried out beyond the L2 request by request, 674 us, the
// rate of a plain read), at p = 8 the chains (MFMA 41 %, LDS 45 % busy).
#pragma once
#include "apply_common.h"

namespace hexpa {

__device__ __forceinline__ double mfma_f64(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

template <int D, int Q, int OPS>
struct ChainShape {
    static constexpr bool kMass = (OPS & 1) != 0, kDiff = (OPS & 2) != 0;
    static constexpr int NC = kDiff ? (kMass ? 7 : 6) : 1;  // stored D values per point
    static constexpr int NCH = kDiff ? 3 : 1;  // tensors U: B_y B_x, G_y B_x, B_y G_x (mass alone: the first)
    static constexpr int TD = (D + 3) / 4, TQ = (Q + 3) / 4;  // 4-blocks of the 1-D sizes
    static constexpr int Q2 = Q * Q, Q3 = Q2 * Q, D2 = D * D, D3 = D2 * D;
    static constexpr int TN = (Q2 + 15) / 16;    // column tiles of the z chain
    static constexpr bool LAST = D % 4 == 1;     // one plane left over: its blocks are strips
    static constexpr int NG = LAST ? D / 4 : TD; // plane groups whose blocks are planes
    static constexpr int UF = NG * TQ + LAST, UT = NG * TD + LAST;  // units of the first and last chain
    static constexpr int NW = cmax3(UF, UT, TN), NT = 64 * NW;
    // LDS strides.  The sixteen lanes of one access differ by 4 beta mod 16 between planes and by
    // an odd row pitch between rows: all on different banks.
    static constexpr int odd(int v) { return v | 1; }
    static constexpr int s4(int v) { return v + (20 - v % 16) % 16; }  // next value = 4 mod 16
    static constexpr int PB = odd(Q), SK = s4(Q * PB);  // U, W: [channel][k][b][a]
    static constexpr int PD = odd(D), SX = s4(D * PD);  // x: [k][j][i]
    static constexpr int PT = 4 * TD;                   // basis tables [q][d], zero padded
    static constexpr int NS = (D3 + NT - 1) / NT;       // nodes per thread
    // the basis operands stay in registers where that leaves room for two workgroups' waves
    static constexpr bool WHOLE = TD * TQ <= 4;
    static constexpr int MINW = WHOLE ? 3 : 4;          // waves per SIMD the registers are limited for
    // Elements a workgroup takes one after the other before it scatters their outputs together:
    // a run's node rows are contiguous and its inner faces are added first, so there are fewer
    // atomic requests (p = 6: 12.7 -> 7.5 M at four elements).  Diffusion / mass at p = 6 with 1,
    // 2, 4, 6, 8: 977/585, 945/433, 919/392, 907/388, 904/422 us; at p = 8 with 2, 4, 6:
    // 1153/467, 1133/451, 1268/467 (LDS for a workgroup less).
    static constexpr int RUN = D >= 8 ? 4 : 6;
    // The run length for `each` elements a resident workgroup.  Runs save atomics but leave
    // workgroups without work where there are few, and their LDS costs residency; a run of one
    // is the kernel without them.  us with 1 / 2 / 3 / RUN elements (each in brackets):
    //   mass, p = 6, Q = 7: 14^3 (2) 15.2 / 15.4 / 16.4 / 19.6, 16^3 (3) 20.2 / 17.3 / 18.2 / 22.4,
    //   25^3 (12) 66.4 / 55.9 / 49.5 / 46.8, p = 5, Q = 6: 20^3 (5) 25.6 / 21.3 / 21.0 / 22.3 (19.8
    //   with four);
    //   diffusion, p = 7, Q = 8: 14^3 (3) 22.8 / 23.0 / 22.4 / 24.5, 15^3 (4) 28.1 / 25.3 / 26.1 /
    //   27.4, 21^3 (12) 64.3 / 61.6 / 59.5 / 59.9;
    //   where the basis operands come from LDS (not WHOLE) the halved LDS of the kernel without
    //   runs counts more.  Mass, p = 7, Q = 9: 13^3 (2) 15.8 / 19.6 / 18.4 / 21.3, 19^3 (6) 41.3 /
    //   48.1 / 45.0 / 37.1; diffusion, p = 8, Q = 10: 18^3 (11) 96.5 / 109 / 106 / 107, 22^3 (20)
    //   178 / 187 / 185 / 184, 27^3 (38) 343 / - / 338 / 337, p = 7, Q = 9, 45^3 (177) 1066 / - /
    //   1044 / 1025; both, p = 8, Q = 9: 22^3 178 / 194 / 191 / 192, 40^3 (125) 1030 / - / - / 998,
    //   Q = 10, whose runs spill registers: 22^3 202 / 226 / 227 / 227, 40^3 1189 / - / - / 1209.
    static constexpr int run_of(int each)
    {
        if (!WHOLE) return (kDiff ? each < 32 || (kMass && Q == 10) : each < 5) ? 1 : RUN;
        const int r = kDiff ? each / 2 : each < 5 ? (each < 3 ? each : 3) : cmax(each / 2, 4);
        return r < 1 ? 1 : r < RUN ? r : RUN;
    }
    static constexpr bool WHOLE_LINES = !kDiff || Q2 % 16 == 0;  // (mass: no difference)
    static constexpr bool ok = D >= 6;
};

// RUNS: runs of up to S::RUN elements (atomic scatter); else of one.
template <int D, int Q, int OPS, bool ATOMIC, bool RUNS>
__global__ __launch_bounds__((ChainShape<D, Q, OPS>::NT), (ChainShape<D, Q, OPS>::MINW)) void k_apply_chain(
    int n, int run, const int32_t *__restrict__ elist, const int32_t *__restrict__ emap, const double *__restrict__ qd,
    const DevTables *__restrict__ tab, const double *__restrict__ x, double *__restrict__ y)
{
    using S = ChainShape<D, Q, OPS>;
    constexpr bool M = S::kMass, DF = S::kDiff, EL = !ATOMIC;
    constexpr int TD = S::TD, TQ = S::TQ, SK = S::SK, SX = S::SX, PB = S::PB, PD = S::PD, PT = S::PT, NC = S::NC;
    constexpr int D2 = S::D2, D3 = S::D3, Q2 = S::Q2, Q3 = S::Q3, NT = S::NT, NS = S::NS, NG = S::NG;
    constexpr int CH = D * SK;  // channel stride
    // U/W, x, y and the basis tables (zero past Q and D).  A lane past the end of an index reads
    // on, into the next row or plane of the same element or into the zero tail, and its basis
    // operand is zero: everything there is finite when the element's values are, since all of
    // LDS is cleared once and the padding never written.
    constexpr int NT_ = S::NCH * CH + 4 * PB, NX = D * SX + 4 * PD;
    // Without runs (few elements a workgroup, and all coloured launches: elements of one colour
    // share no DOFs) there is nothing to merge: each thread adds its own nodes to y, coloured
    // with a load of y asked for when the element began.  (Through the runs' scatter most threads
    // idled while the others walked the rows, coloured with a load of y to wait for in each.
    // Coloured, all eight launches, us: mass p = 7, Q = 9, 25^3 202 -> 129, diffusion p = 8,
    // Q = 10, 22^3 349 -> 288, p = 7, Q = 9, 25^3 321 -> 262; pass by pass 142, 313, 281.)
    static_assert(ATOMIC || !RUNS, "runs merge by atomics");
    constexpr int RUN = RUNS ? S::RUN : 1;
    __shared__ double T[NT_], X[NX], Y[RUN * D3], tb[4 * TQ * PT], tg[DF ? 4 * TQ * PT : 1];
    __shared__ int32_t lmap[RUNS ? RUN * D3 : 1];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 4, r = lane & 3, beta = (lane >> 2) & 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };  // LDS traffic only

    // Runs of `run` <= RUN consecutive elements.  XCD x (workgroups b with b % 8 == x) owns a
    // contiguous range of runs, whose shared DOFs then meet in one L2; its workgroups take them
    // round-robin.  cur, its successor and the one after that are element numbers (g: the run).
    const int nb = gridDim.x, nruns = (n + run - 1) / run;
    int g, gend, nbx;
    if (nb >= 8) {
        const int xcd = blockIdx.x & 7;
        nbx = (nb >> 3) + (xcd < (nb & 7) ? 1 : 0);
        gend = (int)(((int64_t)nruns * (xcd + 1)) >> 3);
        g = (int)(((int64_t)nruns * xcd) >> 3) + (blockIdx.x >> 3);
    } else {
        nbx = nb;
        gend = nruns;
        g = blockIdx.x;
    }
    if (g >= gend) return;
    // the element after e in this workgroup's order, in the run gg (-1: there is none)
    auto next = [&](int e, int &gg) {
        if (e < 0) return -1;
        if (++e < min((gg + 1) * run, n)) return e;
        gg += nbx;
        return gg < gend ? gg * run : -1;
    };

    for (int i = tid; i < NT_; i += NT) T[i] = 0.0;
    for (int i = tid; i < NX; i += NT) X[i] = 0.0;
    for (int i = tid; i < 4 * TQ * PT; i += NT) {
        const int q = i / PT, d = i - q * PT;
        const bool in = q < Q && d < D;
        tb[i] = in ? tab->B[q * D + d] : 0.0;
        if constexpr (DF) tg[i] = in ? tab->G[q * D + d] : 0.0;
    }
    // this wave's unit of the first chain: planes pf (a block each), strip of a; of the last
    // chain: planes pt, strip of i; a left-over plane has its strips in the blocks
    const bool fl = S::LAST && wave == NG * TQ, tl = S::LAST && wave == NG * TD;
    const bool fwd = wave < S::UF, trn = wave < S::UT, tile = wave < S::TN;
    const int pf = fl ? D - 1 : 4 * (wave / TQ) + beta, sa = 4 * (fl ? beta : wave % TQ) + r;
    const int pt = tl ? D - 1 : 4 * (wave / TD) + beta, si = 4 * (tl ? beta : wave % TD) + r;
    const int pfc = min(pf, D - 1), ptc = min(pt, D - 1), sac = min(sa, 4 * TQ - 1), sic = min(si, 4 * TD - 1);
    const bool fin = pf < D && sa < Q, tin = pt < D && si < D;
    // column of the z chain
    const int nn = min(16 * wave + (lane & 15), Q2 - 1);
    const bool nin = 16 * wave + (lane & 15) < Q2;
    const int nT = (nn / Q) * PB + nn % Q;
    const int hT = h * SK + nT, hTl = min(4 * (TD - 1) + h, D - 1) * SK + nT;  // plane 4 tk + h; of the last block

    // basis operands: in registers for the whole kernel where they fit, else read from the
    // tables where they are used
    const double *tbf = tb + r * PT + h, *tgf = tg + r * PT + h, *tbt = tb + h * PT + r, *tgt = tg + h * PT + r;
    constexpr int WD = S::WHOLE ? TD : 1, WQ = S::WHOLE ? TQ : 1;
    double rbf[WQ][WD], rgf[WQ][WD], rbt[WD][WQ], rgt[WD][WQ], rbx[WD], rgx[WD], rbxt[WQ], rgxt[WQ];
    auto bf = [&](int tq, int td) { return S::WHOLE ? rbf[tq][td] : tbf[4 * tq * PT + 4 * td]; };
    auto gf = [&](int tq, int td) { return S::WHOLE ? rgf[tq][td] : tgf[4 * tq * PT + 4 * td]; };
    auto bt = [&](int td, int tq) { return S::WHOLE ? rbt[td][tq] : tbt[4 * tq * PT + 4 * td]; };
    auto gt = [&](int td, int tq) { return S::WHOLE ? rgt[td][tq] : tgt[4 * tq * PT + 4 * td]; };
    auto bx = [&](int td) { return S::WHOLE ? rbx[td] : tb[sac * PT + 4 * td + h]; };
    auto gx = [&](int td) { return S::WHOLE ? rgx[td] : tg[sac * PT + 4 * td + h]; };
    auto bxt = [&](int tq) { return S::WHOLE ? rbxt[tq] : tb[(4 * tq + h) * PT + sic]; };
    auto gxt = [&](int tq) { return S::WHOLE ? rgxt[tq] : tg[(4 * tq + h) * PT + sic]; };

    auto elem = [&](int gg) { return (int64_t)(EL ? elist[gg] : gg); };
    auto load_map = [&](int32_t (&m)[NS], int gg) {
        const int32_t *p = emap + elem(max(gg, 0)) * D3;
#pragma unroll
        for (int s = 0; s < NS; ++s) m[s] = p[min(tid + NT * s, D3 - 1)];
    };
    auto gather = [&](double (&v)[NS], const int32_t (&m)[NS]) {
#pragma unroll
        for (int s = 0; s < NS; ++s) v[s] = x[m[s]];
    };
    auto node = [&](int s) {  // place of node tid + NT s in X
        const int I = tid + NT * s, k = I / D2, q = I - k * D2, j = q / D;
        return k * SX + j * PD + q - j * D;
    };
    auto stage = [&](const double (&v)[NS]) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (tid + NT * s < D3) X[node(s)] = v[s];
    };
    double dq[NC][TQ];  // D of this wave's column tile: points c = 4 tc + h
    auto load_d = [&](int gg) {
        const double *p = qd + elem(max(gg, 0)) * (NC * Q3) + nn;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int tc = 0; tc < TQ; ++tc)
                dq[c][tc] = load_once<S::WHOLE_LINES>(p + c * Q3 + min(4 * tc + h, Q - 1) * Q2);
    };
    // Scatter-add of a run's outputs.  A thread keeps its element and place i in the node row of
    // the run and walks the rows (j, k): a wave's atomics cover whole rows of the run, and each
    // address is an addition away from the last.  Where the right face of an element and the
    // left face of the next hold the same DOF (read from the maps, so any element order stays
    // exact) their contributions are added first.
    auto scatter = [&] {
        constexpr int ROW = RUN * D, NGR = NT / ROW;
        const int row = tid / ROW, e = (tid - row * ROW) / D, i = tid - row * ROW - e * D;
        if (row >= NGR) return;
        int L = e * D3 + i + D * row;
        for (int jk = row; jk < D2; jk += NGR, L += D * NGR) {
            const int32_t gi = lmap[L];
            if (gi < 0) continue;
            if (i == 0 && e > 0 && lmap[L - D3 + (D - 1)] == gi) continue;  // added by the left neighbour
            double v = Y[L];
            if (i == D - 1 && e + 1 < RUN && lmap[L + D3 - (D - 1)] == gi) v += Y[L + D3 - (D - 1)];
            unsafeAtomicAdd(y + gi, v);
        }
    };
    // maps of this element, the next and the one after it; past the last one a workgroup loads
    // element 0 and drops it
    int32_t m0[NS], m1[NS];
    double xv[NS];
    int gc = g, cur = g * run, at = 0, g1 = g, nxt = next(cur, g1), g2 = g1, nx2;
    bool full = false;  // a run's outputs wait in Y
    load_map(m0, cur);
    load_map(m1, nxt);
    load_d(cur);
    gather(xv, m0);
    if constexpr (RUNS)
        for (int i = tid; i < RUN * D3; i += NT) lmap[i] = -1;
    barrier();  // basis tables
    if constexpr (S::WHOLE) {
#pragma unroll
        for (int td = 0; td < TD; ++td) {
#pragma unroll
            for (int tq = 0; tq < TQ; ++tq) {
                rbf[tq][td] = tbf[4 * tq * PT + 4 * td];
                rbt[td][tq] = tbt[4 * tq * PT + 4 * td];
                if constexpr (DF) {
                    rgf[tq][td] = tgf[4 * tq * PT + 4 * td];
                    rgt[td][tq] = tgt[4 * tq * PT + 4 * td];
                }
            }
            rbx[td] = tb[sac * PT + 4 * td + h];
            if constexpr (DF) rgx[td] = tg[sac * PT + 4 * td + h];
        }
#pragma unroll
        for (int tq = 0; tq < TQ; ++tq) {
            rbxt[tq] = tb[(4 * tq + h) * PT + sic];
            if constexpr (DF) rgxt[tq] = tg[(4 * tq + h) * PT + sic];
        }
    }
    stage(xv);
    barrier();

    for (;;) {
        // x and y axes of this element; the next one's x and the map after it are requested,
        // and the previous run's outputs go out
        nx2 = next(nxt, g2);
        gather(xv, m1);
        int32_t m2[NS];
        load_map(m2, nx2);
        double yv[NS];
        if constexpr (!ATOMIC)
#pragma unroll
            for (int s = 0; s < NS; ++s) yv[s] = y[m0[s]];
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (RUNS)
            if (full) scatter();
        if (fwd) {
            double pb[TD], pg[DF ? TD : 1];
            const double *Xp = X + pfc * SX + r * PD + h;
#pragma unroll
            for (int tj = 0; tj < TD; ++tj) {
                pb[tj] = 0.0;
                if constexpr (DF) pg[tj] = 0.0;
#pragma unroll
                for (int ti = 0; ti < TD; ++ti) {
                    const double xa = Xp[4 * tj * PD + 4 * ti];
                    pb[tj] = mfma_f64(xa, bx(ti), pb[tj]);
                    if constexpr (DF) pg[tj] = mfma_f64(xa, gx(ti), pg[tj]);
                }
            }
            double *U = T + pfc * SK + h * PB + sa;
#pragma unroll
            for (int tq = 0; tq < TQ; ++tq) {
                double u0 = 0.0, u1 = 0.0, u2 = 0.0;
#pragma unroll
                for (int tj = 0; tj < TD; ++tj) {
                    u0 = mfma_f64(bf(tq, tj), pb[tj], u0);
                    if constexpr (DF) {
                        u1 = mfma_f64(gf(tq, tj), pb[tj], u1);
                        u2 = mfma_f64(bf(tq, tj), pg[tj], u2);
                    }
                }
                if (fin && 4 * tq + h < Q) {
                    U[4 * tq * PB] = u0;
                    if constexpr (DF) {
                        U[4 * tq * PB + CH] = u1;
                        U[4 * tq * PB + 2 * CH] = u2;
                    }
                }
            }
        }
        barrier();
        // the scatter has read the map of the run before
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (RUNS && tid + NT * s < D3) {
                lmap[at * D3 + tid + NT * s] = m0[s];
                if (full)
                    for (int e = 1; e < RUN; ++e) lmap[e * D3 + tid + NT * s] = -1;
            }

        // z axis, D, transposed z axis, in place on this wave's columns
        if (tile) {
            double vx[DF ? TQ : 1], vy[DF ? TQ : 1], vz[DF ? TQ : 1], vu[M ? TQ : 1];
#pragma unroll
            for (int tc = 0; tc < TQ; ++tc) {
                if constexpr (DF) vx[tc] = vy[tc] = vz[tc] = 0.0;
                if constexpr (M) vu[tc] = 0.0;
            }
#pragma unroll
            for (int tk = 0; tk < TD; ++tk) {
                const double *p = T + (4 * tk + 3 < D ? 4 * tk * SK + hT : hTl);
                const double c0 = p[0];
                double c1 = 0.0, c2 = 0.0;
                if constexpr (DF) {
                    c1 = p[CH];
                    c2 = p[2 * CH];
                }
#pragma unroll
                for (int tc = 0; tc < TQ; ++tc) {
                    if constexpr (DF) {
                        vz[tc] = mfma_f64(gf(tc, tk), c0, vz[tc]);
                        vy[tc] = mfma_f64(bf(tc, tk), c1, vy[tc]);
                        vx[tc] = mfma_f64(bf(tc, tk), c2, vx[tc]);
                    }
                    if constexpr (M) vu[tc] = mfma_f64(bf(tc, tk), c0, vu[tc]);
                }
            }
#pragma unroll
            for (int tc = 0; tc < TQ; ++tc) {
                if constexpr (DF) {
                    const double g0 = vx[tc], g1 = vy[tc], g2 = vz[tc];
                    vx[tc] = dq[0][tc] * g0 + dq[1][tc] * g1 + dq[2][tc] * g2;
                    vy[tc] = dq[1][tc] * g0 + dq[3][tc] * g1 + dq[4][tc] * g2;
                    vz[tc] = dq[2][tc] * g0 + dq[4][tc] * g1 + dq[5][tc] * g2;
                }
                if constexpr (M) vu[tc] *= dq[NC - 1][tc];
            }
            __builtin_amdgcn_sched_barrier(0);
            load_d(nxt);  // the next element's, in flight until its D-step
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int tk = 0; tk < TD; ++tk) {
                double w0 = 0.0, w1 = 0.0, w2 = 0.0;
#pragma unroll
                for (int tc = 0; tc < TQ; ++tc) {
                    if constexpr (DF) {
                        w0 = mfma_f64(gt(tk, tc), vz[tc], w0);
                        w1 = mfma_f64(bt(tk, tc), vy[tc], w1);
                        w2 = mfma_f64(bt(tk, tc), vx[tc], w2);
                    }
                    if constexpr (M) w0 = mfma_f64(bt(tk, tc), vu[tc], w0);
                }
                if (nin && 4 * tk + h < D) {
                    double *p = T + 4 * tk * SK + hT;
                    p[0] = w0;
                    if constexpr (DF) {
                        p[CH] = w1;
                        p[2 * CH] = w2;
                    }
                }
            }
        }
        barrier();

        // transposed x and y axes; the next element's x takes its place
        if (trn) {
            const double *W = T + ptc * SK + r * PB + h;
            double yo[TD];
#pragma unroll
            for (int tj = 0; tj < TD; ++tj) yo[tj] = 0.0;
#pragma unroll
            for (int tq = 0; tq < TQ; ++tq) {
                double q0 = 0.0, q1 = 0.0;
#pragma unroll
                for (int ta = 0; ta < TQ; ++ta) {
                    const double *p = W + 4 * tq * PB + 4 * ta;
                    q0 = mfma_f64(p[0], bxt(ta), q0);
                    if constexpr (DF) {
                        q1 = mfma_f64(p[CH], bxt(ta), q1);
                        q0 = mfma_f64(p[2 * CH], gxt(ta), q0);
                    }
                }
#pragma unroll
                for (int tj = 0; tj < TD; ++tj) {
                    yo[tj] = mfma_f64(bt(tj, tq), q0, yo[tj]);
                    if constexpr (DF) yo[tj] = mfma_f64(gt(tj, tq), q1, yo[tj]);
                }
            }
#pragma unroll
            for (int tj = 0; tj < TD; ++tj)
                if (tin && 4 * tj + h < D) Y[at * D3 + ptc * D2 + (4 * tj + h) * D + si] = yo[tj];
        }
        stage(xv);
        barrier();
        if constexpr (!RUNS)
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (tid + NT * s < D3) {
                    const double v = Y[tid + NT * s];
                    if constexpr (ATOMIC) unsafeAtomicAdd(y + m0[s], v);
                    else y[m0[s]] = yv[s] + v;
                }
        full = g1 != gc || nxt < 0;  // the run ends here
        if (nxt < 0) break;
        at = full ? 0 : at + 1;
        cur = nxt;
        gc = g1;
        nxt = nx2;
        g1 = g2;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            m0[s] = m1[s];
            m1[s] = m2[s];
        }
    }
    if constexpr (RUNS) scatter();
}

}  // namespace hexpa
