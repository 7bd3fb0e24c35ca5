// Block sweeps of libhelm (gfx950): multi-right-hand-side forward and back
// substitution with the stored Schur-complement inverses G_j,
//     forward   w_j = G_j y_j,          y_{j+dir} = b_{j+dir} - E w_j,
//     backward  x_j = w_j - G_j z_j,    z_{j-dir} = E x_j,
// run from both ends of the grid at once (the two fronts of the twisted
// factorisation meet at row k, where w_k = x_k), one launch per step, every
// front of the batch in the same launch.
// A workgroup computes a 16-row x 16-column tile of the block product on
// the matrix cores (four waves split the contraction and are summed in a
// fixed order) and, for the same rows, the coupling vector the next step
// needs, so each step reads one operand vector instead of two.
#include "helm_device.h"
#include "helm_launch.h"

#include <algorithm>

namespace helm {

constexpr int SW_WAVES = 4;
constexpr int SW_CTG = 1;     // 16-column tiles per workgroup (the waves split them, then K)
constexpr int SW_GDEPTH = 2;  // 16-wide K chunks of the factor block in flight per wave
constexpr int SW_YDEPTH = 2;  // and of the coupling vector
// chunks per straight-line block of the contraction: a template parameter,
// chosen per launch as the smallest even count that covers one wave's
// chunks (at most 8), so a wave does not refill chunks it never uses

int sweep_row_tiles(int np) { return np / 16; }
int sweep_col_tiles(int S) { return ((S + 15) / 16 + SW_CTG - 1) / SW_CTG; }
int sweep_grid(int groups, int cgroups) { return 8 * ((groups * cgroups + 7) / 8); }

// coupling-vector layout of the precision (b_tiled4 for complex64)
template <typename T>
__device__ __forceinline__ size_t bt(int row, int col, int np) {
    return sizeof(T) == 4 ? b_tiled4(row, col, np) : b_tiled(row, col, np);
}

template <typename C>
__device__ __forceinline__ C conj_if(C v, bool c) {
    if (c) v.y = -v.y;
    return v;
}

// y = b_{row0} into Y0 (B-operand layout; rows >= nx and columns >= S zero)
template <typename T, bool CONJB>
__global__ __launch_bounds__(256) void k_sweep_init(const SweepTab* __restrict__ tab, int n) {
    using C = typename CT<T>::c;
    const int ci = find_chain(tab->c, n, blockIdx.x, [](const SweepInfo& c) { return c.itile0; });
    const SweepInfo d = load_entry(tab->c, ci);
    const int s16 = (d.S + 15) & ~15;
    const int64_t e = (int64_t)(blockIdx.x - d.itile0) * 256 + threadIdx.x;
    if (e >= (int64_t)d.np * s16) return;
    const int s = (int)(e / d.np), k = (int)(e % d.np);
    C v = mk<C>(0.0, 0.0);
    if (k < d.nx && s < d.S)
        v = conj_if(gld((const C*)d.B + (size_t)s * d.ldb + (size_t)d.row0 * d.nx + k), CONJB);
    gst((C*)d.Y0 + bt<T>(k, s, d.np), v);
}

// One workgroup per 16-row tile of a front's block row and group of SW_CTG
// 16-column tiles of the right-hand sides: the product G_j(rows) Y(columns)
// on the matrix cores, three real products per complex one (Gauss's form:
// Gr Yr, Gi Yi and (Gr + Gi)(Yr + Yi), in separate accumulators).  The waves share out the column tiles and split the
// contraction; the parts are summed in a fixed order through LDS.  Each wave
// streams its operands with SW_DEPTH chunks of 16 in flight, and several
// workgroups per compute unit hide the rest of the latency.
template <typename T, bool FWD, bool CONJB, int SW_UNROLL>
__global__ __launch_bounds__(64 * SW_WAVES) void k_sweep(int n, int tstep, int groups, int cgroups, int uni,
                                                        const SweepTab* __restrict__ tab) {
    using C = typename CT<T>::c;
    using V = typename CT<T>::v4;
    __shared__ T red[SW_WAVES][2][4][64];
    // XCD x (workgroup b runs on XCD b % 8) takes one contiguous range of the
    // (row tile, column tile) pairs, row tile by row tile and front by front:
    // the column tiles of a row tile share its factor rows, and the row tiles
    // of a front its coupling vectors, in one or two L2s.
    const int total = groups * cgroups, per = (total + 7) >> 3;
    const int q = (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);
    if (q >= total) return;
    const int g = q / cgroups, cgi = q - g * cgroups;
    // uni > 0: every front of the launch has uni row tiles
    const int ci = uni > 0 ? (int)((unsigned)g / (unsigned)uni)
                           : find_chain(tab->c, n, g, [](const SweepInfo& c) { return c.tile0; });
    const SweepInfo d = load_entry(tab->c, ci);
    if (tstep >= (FWD ? d.nfwd : d.nbwd)) return;
    const int nct = (d.S + 15) >> 4, ct0 = SW_CTG * cgi;
    if (ct0 >= nct) return;
    const int nctg = min(SW_CTG, nct - ct0);
    const int P = 4 / nctg;                       // contraction parts per column tile
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int lr = l & 15, lg = l >> 4;
    const int myct = w % nctg, part = w / nctg;
    const bool active = part < P;
    const int j = FWD ? d.row0 + d.dir * tstep : d.brow0 - d.dir * tstep;
    const int i0 = 16 * (g - d.tile0);
    const int np = d.np, nx = d.nx;
    // operand streams: this row tile of G_j and this column tile of Y, each
    // 64 consecutive elements per MFMA step (the tiled layouts)
    const C* Gt = (const C*)d.G + (size_t)j * np * np + (size_t)(i0 >> 4) * (np >> 2) * 64 + l;
    const C* Gt4 = Gt - l + 4 * l;   // complex64 layout: a lane's four values of a chunk adjacent
    // steps of one front alternate the coupling buffers: forward step t is
    // step t, backward step t is step nfwd + t of the front
    const int u = FWD ? tstep : d.nfwd + tstep;
    const C* Yin = (const C*)((u & 1) ? d.Y1 : d.Y0);
    C* Yout = (C*)((u & 1) ? d.Y0 : d.Y1);
    const int s = 16 * (ct0 + myct) + lr;
    const bool scol = s < d.S;
    const C* Yt = Yin + (size_t)(ct0 + myct) * (np >> 2) * 64 + l;
    const C* Yt4 = Yt - l + 4 * l;   // complex64 layout

    // epilogue operands (next block's right-hand side, or this block's
    // forward result), fetched before the contraction.  Forward: `more` -
    // the front continues; else a bottom front hands its vector to the top
    // front (Mout), and the top front's last step is x_k.
    const C* Bv = (const C*)d.B;
    C* X = (C*)d.X;
    const bool more = FWD && tstep + 1 < d.nfwd;
    const bool merge_in = more && d.Bm && tstep + 2 == d.nfwd;
    const bool hand_over = FWD && !more && d.Mout;
    const bool lead = active && part == 0;
    // loaded unconditionally at clamped addresses (so no load waits on
    // another), then zeroed where unused
    C pre[4];
    const bool want = lead && (FWD ? (merge_in || more || hand_over) : true);
    if (lead) {
        const int sc = min(s, d.S - 1);
        const int jr = (FWD && (more || hand_over)) ? j + d.dir : j;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int ic = min(i0 + acc_row<T>(lg, e), nx - 1);
            const C* src = !FWD      ? X + (size_t)sc * d.ldx + (size_t)j * nx + ic
                           : merge_in ? (const C*)d.Bm + bt<T>(ic, sc, np)
                                      : Bv + (size_t)sc * d.ldb + (size_t)jr * nx + ic;
            pre[e] = gld(src);
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    V p1, p2, p3;
#pragma unroll
    for (int e = 0; e < 4; ++e) { p1[e] = 0; p2[e] = 0; p3[e] = 0; }
    // this wave's chunks of 16 in the contraction; in MFMA step q lane group
    // lg carries k = 16 ch + 4 q + lg.  Chunk indices are clamped, so every
    // load is in range.
    const int nch = np >> 4;
    const int c_beg = active ? part * nch / P : 0, c_end = active ? (part + 1) * nch / P : 0;
    C ga[SW_GDEPTH][4], ya[SW_YDEPTH][4];
    auto gload = [&](C (&gq)[4], int c) {
        const int cc = min(c, c_end - 1);
        if constexpr (sizeof(T) == 4) {
            // complex64 blocks (a_tiled4): a lane's four values of the chunk
            // are adjacent, two 16-byte loads
            typedef float gv4f __attribute__((ext_vector_type(4)));
            const HELM_GLOBAL gv4f* p = (const HELM_GLOBAL gv4f*)(Gt4 + (size_t)cc * 256);
            const gv4f a = p[0], b = p[1];
            gq[0] = mk<C>(a.x, a.y);
            gq[1] = mk<C>(a.z, a.w);
            gq[2] = mk<C>(b.x, b.y);
            gq[3] = mk<C>(b.z, b.w);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) gq[q] = gld(Gt + (size_t)(4 * cc + q) * 64);
        }
    };
    auto yload = [&](C (&yq)[4], int c) {
        const int cc = min(c, c_end - 1);
        if constexpr (sizeof(T) == 4) {
            // complex64 coupling vectors (b_tiled4): two 16-byte loads
            typedef float gv4f __attribute__((ext_vector_type(4)));
            const HELM_GLOBAL gv4f* p = (const HELM_GLOBAL gv4f*)(Yt4 + (size_t)cc * 256);
            const gv4f a = p[0], b = p[1];
            yq[0] = mk<C>(a.x, a.y);
            yq[1] = mk<C>(a.z, a.w);
            yq[2] = mk<C>(b.x, b.y);
            yq[3] = mk<C>(b.z, b.w);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) yq[q] = gld(Yt + (size_t)(4 * cc + q) * 64);
        }
    };
    // The chunks run in straight-line blocks of SW_UNROLL, each starting
    // with empty queues: the products of a chunk past the end are skipped (a
    // wave-uniform branch) while the refills stay unconditional, so the
    // outstanding loads are the same on every path and each wait covers
    // exactly the chunk about to be used.  The factor block (from HBM) is
    // fetched SW_GDEPTH chunks ahead, the coupling vector (from L2)
    // SW_YDEPTH chunks ahead.
    for (int c0 = c_beg; c0 < c_end; c0 += SW_UNROLL) {
#pragma unroll
        for (int v = 0; v < SW_GDEPTH; ++v) {
            gload(ga[v], c0 + v);
            if (v < SW_YDEPTH) yload(ya[v], c0 + v);
        }
#pragma unroll
        for (int u = 0; u < SW_UNROLL; ++u) {
            const int vg = u % SW_GDEPTH, vy = u % SW_YDEPTH;
            if (c0 + u < c_end) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const T yr = ya[vy][q].x, yi = ya[vy][q].y;
                    const T gr = ga[vg][q].x, gi = ga[vg][q].y;
                    p1 = mfma16(gr, yr, p1);
                    p2 = mfma16(gi, yi, p2);
                    p3 = mfma16(gr + gi, yr + yi, p3);
                }
            }
            if (u + SW_GDEPTH < SW_UNROLL) gload(ga[vg], c0 + u + SW_GDEPTH);
            if (u + SW_YDEPTH < SW_UNROLL) yload(ya[vy], c0 + u + SW_YDEPTH);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = i0 + acc_row<T>(lg, e);
        if (!(want && scol && i < nx)) pre[e] = mk<C>(0.0, 0.0);
        else if (FWD && !merge_in) pre[e] = conj_if(pre[e], CONJB);
    }
    T sre[4], sim[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sre[e] = p1[e] - p2[e];
        sim[e] = p3[e] - p1[e] - p2[e];
    }
    if (P > 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { red[w][0][e][l] = sre[e]; red[w][1][e][l] = sim[e]; }
        __syncthreads();
        if (!lead) return;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sre[e] = red[myct][0][e][l];
            sim[e] = red[myct][1][e][l];
            for (int q = 1; q < P; ++q) {
                sre[e] += red[myct + nctg * q][0][e][l];
                sim[e] += red[myct + nctg * q][1][e][l];
            }
        }
    }
    if (!lead || !scol) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = i0 + acc_row<T>(lg, e);
        const T sr = sre[e], si = sim[e];
        const T ei = (T)(i >= nx ? 0.0 : ((i == 0 || i == nx - 1) ? -0.5 * d.cz : -d.cz));
        C nxt = mk<C>(0.0, 0.0);
        if (FWD) {
            // w_j; the next step's y_{j+dir} = b_{j+dir} - E w_j; at the end
            // of a bottom front that vector goes to the top front, and at the
            // end of a top front (w_j = x_j) both backward sweeps start with E x_j
            if (i < nx) gst(X + (size_t)s * d.ldx + (size_t)j * nx + i, mk<C>(sr, si));
            if (more || hand_over) {
                if (i < nx) nxt = mk<C>(pre[e].x - ei * sr, pre[e].y - ei * si);
                if (hand_over) {
                    gst((C*)d.Mout + bt<T>(i, s, np), nxt);
                    continue;
                }
            } else {
                nxt = mk<C>(ei * sr, ei * si);
                if (d.Zp) gst((C*)d.Zp + bt<T>(i, s, np), nxt);
            }
        } else {
            // x_j = w_j - G_j z_j; the next step's z = E x_j
            if (i < nx) {
                const C xn = mk<C>(pre[e].x - sr, pre[e].y - si);
                gst(X + (size_t)s * d.ldx + (size_t)j * nx + i, xn);
                nxt = mk<C>(ei * xn.x, ei * xn.y);
            }
        }
        gst(Yout + bt<T>(i, s, np), nxt);
    }
}

// ------------------------------------------------------------ narrow grids --
// A step's product is then smaller than a launch (np = 80 in complex64: 2 us
// of work in a launch of 3.6 us), so one workgroup takes a front and 16
// columns through all its rows, with the coupling vector in LDS and the next
// row's factor block and vectors on their way while this row is multiplied.
// The fronts meet between two launches: the first goes forward to row k, the
// second starts with row k in both fronts' workgroups (each needs x_k) and
// goes back.  A row takes 1.3 us (np = 16) to 2.5 us; the matrix cores of one
// compute unit bound it from np = 64 (complex128) or 96 (complex64) on, where
// a launch per step, whose row tiles fill several, takes over.  Solves of 64
// columns, a launch per step against this, in us: complex128 16 x 90 309 /
// 120, 48 x 60 245 / 159, 64 x 90 366 / 267, 80 x 60 264 / 320 (the launches
// keep it); complex64 with its refinement 48 x 60 503 / 253, 80 x 60 547 /
// 372, 96 x 60 554 / 427, 112 x 46 440 / 442 (the launches keep it).
// A front's row tiles times ks parts of the contraction are one wavefront
// each; the parts are summed in order.
constexpr int SWC_W = 16, SWC_T = 64 * SWC_W;
constexpr int SWC_E = 2;   // vector entries per thread (at most 96 x 16)

template <typename T, bool FWD, bool CONJB, int CN>
__global__ __launch_bounds__(SWC_T) void k_sweep_chain(const SweepTab* __restrict__ tab) {
    using C = typename CT<T>::c;
    using V = typename CT<T>::v4;
    extern __shared__ __attribute__((aligned(16))) char chain_smem[];
    C (*red)[16][17] = (C(*)[16][17])chain_smem;          // [wavefront]
    C (*sy)[17] = (C(*)[17])(red + SWC_W);                // the coupling vector
    const SweepInfo d = load_entry(tab->c, blockIdx.y);
    const int S = d.S, s0 = 16 * blockIdx.x, np = d.np, nx = d.nx;
    if (s0 >= S) return;
    const bool bottom = d.Mout != nullptr;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, lr = l & 15, lg = l >> 4;
    // rows: forward all of a bottom front's, a top front's but row k;
    // backward row k, then the front's from there
    const int kk = d.row0 + d.dir * (bottom ? d.nfwd : d.nfwd - 1);
    const int steps = FWD ? (bottom ? d.nfwd : d.nfwd - 1) : d.nbwd + 1;
    auto row = [&](int t) { return FWD ? d.row0 + d.dir * t : t == 0 ? kk : d.brow0 - d.dir * (t - 1); };
    // this thread's entries of the vectors: row i, column c (rows along the
    // right-hand sides)
    int ei[SWC_E], ec[SWC_E];
    bool own[SWC_E], in[SWC_E];
#pragma unroll
    for (int e = 0; e < SWC_E; ++e) {
        const int q = tid + SWC_T * e;
        own[e] = q < 16 * np;
        ec[e] = own[e] ? q / np : 0;
        ei[e] = own[e] ? q - ec[e] * np : 0;
        in[e] = own[e] && ei[e] < nx && s0 + ec[e] < S;
    }
    const C zero = mk<C>(0.0, 0.0);
    const C* Bv = (const C*)d.B;
    C* X = (C*)d.X;
    // forward: the right-hand side of row j + dir; backward: w of row j
    auto fetch = [&](C (&v)[SWC_E], const C* src, int64_t ld, int j) {
#pragma unroll
        for (int e = 0; e < SWC_E; ++e)
            v[e] = gld(src + (size_t)min(s0 + ec[e], S - 1) * ld + (size_t)j * nx + min(ei[e], nx - 1));
    };
    // this wavefront's part of a product
    // (five row tiles: halves of 2 and 3 chunks, placed so that no SIMD, which
    // wavefront w runs on by w % 4, gets more than 7 of the 25)
    const int rt = np >> 4, ks = rt <= 4 ? 4 : 2;
    const int it = ks == 4 ? w >> 2 : w < rt ? w : rt == 5 && w == 8 ? rt : w - rt - (rt == 5 && w > 8 ? 1 : 0);
    const int part = ks == 4 ? w & 3 : w < rt ? 1 : 0;
    const int cb = part * rt / ks, ce = it < rt ? (part + 1) * rt / ks : cb;
    C g[CN][4];
    auto gload = [&](int c, int j) {
        if (it >= rt) return;
        const int cc = min(cb + c, max(ce - 1, 0));
        const C* G = (const C*)d.G + (size_t)j * np * np + (size_t)it * (np >> 2) * 64;
        if constexpr (sizeof(T) == 4) {
            typedef float gv4f __attribute__((ext_vector_type(4)));
            const HELM_GLOBAL gv4f* p = (const HELM_GLOBAL gv4f*)(G + 4 * l + (size_t)cc * 256);
            const gv4f a = p[0], b = p[1];
            g[c][0] = mk<C>(a.x, a.y);
            g[c][1] = mk<C>(a.z, a.w);
            g[c][2] = mk<C>(b.x, b.y);
            g[c][3] = mk<C>(b.z, b.w);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) g[c][q] = gld(G + l + (size_t)(4 * cc + q) * 64);
        }
    };
    C pre[SWC_E];
    if (FWD) {
        if (steps == 0) return;
        fetch(pre, Bv, d.ldb, d.row0);
#pragma unroll
        for (int e = 0; e < SWC_E; ++e)
            if (own[e]) sy[ei[e]][ec[e]] = in[e] ? conj_if(pre[e], CONJB) : zero;
    } else {
        // y_k: what the bottom front left (or b_k, read and conjugated by the
        // forward launch's type), less the top front's E w_{k-1}
        const C* M = (const C*)(bottom ? d.Mout : d.Bm);
        const C* top = (const C*)(bottom ? d.Zp : d.Y0);
        fetch(pre, Bv, d.ldb, kk);
#pragma unroll
        for (int e = 0; e < SWC_E; ++e) {
            const size_t at = bt<T>(ei[e], s0 + ec[e], np);
            C v = M ? gld(M + at) : conj_if(pre[e], CONJB);
            if (kk > 0) {
                const C q = gld(top + at);
                v = mk<C>(v.x - q.x, v.y - q.y);
            }
            if (own[e]) sy[ei[e]][ec[e]] = in[e] ? v : zero;
        }
    }
#pragma unroll
    for (int c = 0; c < CN; ++c) gload(c, row(0));
    if (FWD) fetch(pre, Bv, d.ldb, min(max(row(0) + d.dir, 0), d.nz - 1));
    __syncthreads();
    // one row: cur holds its vectors, ahead takes the next row's (two sets in
    // turn: a copy between them would wait for the loads)
    auto step = [&](int t, C (&cur)[SWC_E], C (&ahead)[SWC_E]) {
        const int j = row(t), jn = row(min(t + 1, steps - 1));
        V p1, p2, p3;
#pragma unroll
        for (int e = 0; e < 4; ++e) { p1[e] = 0; p2[e] = 0; p3[e] = 0; }
#pragma unroll
        for (int c = 0; c < CN; ++c) {
            if (cb + c < ce) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const C y = sy[16 * (cb + c) + 4 * q + lg][lr];
                    cmfma3<T, V>(p1, p2, p3, g[c][q].x, g[c][q].y, y.x, y.y);
                }
            }
            // this row's vectors are waited for here, where only older loads
            // are in flight, not behind the next row's
            if (c == 0) {
#pragma unroll
                for (int e = 0; e < SWC_E; ++e) asm volatile("" : "+v"(cur[e].x), "+v"(cur[e].y));
            }
            gload(c, jn);
        }
        if (it < rt) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                red[it * ks + part][acc_row<T>(lg, e)][lr] = mk<C>(p1[e] - p2[e], p3[e] - p1[e] - p2[e]);
        }
        // what the next step needs beside its factor block
        if (FWD) fetch(ahead, Bv, d.ldb, min(max(jn + d.dir, 0), d.nz - 1));
        else fetch(ahead, X, d.ldx, jn);
        __syncthreads();
        const bool last = t + 1 == steps;
#pragma unroll
        for (int e = 0; e < SWC_E; ++e) {
            if (!own[e]) continue;
            const int i = ei[e], r = i & 15, wv = (i >> 4) * ks;
            C part_q[4];   // all read before the first is added
#pragma unroll
            for (int q = 0; q < 4; ++q) part_q[q] = red[wv + min(q, ks - 1)][r][ec[e]];
            C sum = cadd(part_q[0], part_q[1]);
            if (ks == 4) sum = cadd(cadd(sum, part_q[2]), part_q[3]);
            const T sr = sum.x, si = sum.y;
            const T cz = (T)(i >= nx ? 0.0 : ((i == 0 || i == nx - 1) ? -0.5 * d.cz : -d.cz));
            C* xo = X + (size_t)(s0 + ec[e]) * d.ldx + (size_t)j * nx + i;
            C nxt = zero;
            if (FWD) {
                const C bn = conj_if(cur[e], CONJB);
                if (in[e]) {
                    gst(xo, mk<C>(sr, si));
                    nxt = last && !bottom ? mk<C>(cz * sr, cz * si) : mk<C>(bn.x - cz * sr, bn.y - cz * si);
                }
                if (last) gst((C*)(bottom ? d.Mout : d.Y0) + bt<T>(i, s0 + ec[e], np), nxt);
            } else if (in[e]) {
                const C xn = t == 0 ? mk<C>(sr, si) : mk<C>(cur[e].x - sr, cur[e].y - si);
                if (t > 0 || !bottom) gst(xo, xn);
                nxt = mk<C>(cz * xn.x, cz * xn.y);
            }
            sy[i][ec[e]] = nxt;
        }
        __syncthreads();
    };
    C other[SWC_E];
    for (int t = 0; t < steps; t += 2) {
        step(t, pre, other);
        if (t + 1 < steps) step(t + 1, other, pre);
    }
}

template <typename T, int CN>
static hipError_t launch_sweep_chain_t(const SweepTab* dtab, int nf, int nct, int np_max, bool conj_b, hipStream_t st) {
    using C = typename CT<T>::c;
    // the attribute is set to the most that this kernel takes, so that no
    // thread lowers it under another's launch
    constexpr size_t most = sizeof(C) * 17 * (16 * SWC_W + (sizeof(T) == 4 ? 96 : 64));
    const size_t lds = sizeof(C) * 17 * (16 * SWC_W + (size_t)np_max);
    const dim3 grid(nct, nf), block(SWC_T);
    auto go = [&](auto kernel) -> hipError_t {
        if (lds > 65536) {
            const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, grid, block, lds, st, dtab);
        return hipSuccess;
    };
    const hipError_t e = conj_b ? go(k_sweep_chain<T, true, true, CN>) : go(k_sweep_chain<T, true, false, CN>);
    if (e != hipSuccess) return e;
    return conj_b ? go(k_sweep_chain<T, false, true, CN>) : go(k_sweep_chain<T, false, false, CN>);
}
hipError_t launch_sweep_chain(const SweepTab* dtab, int nf, int nct, int np_max, bool fp32, bool conj_b, hipStream_t st) {
    if (!fp32) return launch_sweep_chain_t<double, 1>(dtab, nf, nct, np_max, conj_b, st);
    if (np_max <= 64) return launch_sweep_chain_t<float, 1>(dtab, nf, nct, np_max, conj_b, st);
    return launch_sweep_chain_t<float, 3>(dtab, nf, nct, np_max, conj_b, st);
}

void launch_sweep_init(const SweepTab* dtab, int n, int total, bool fp32, bool conj_b, hipStream_t st) {
    if (fp32) {
        if (conj_b) hipLaunchKernelGGL((k_sweep_init<float, true>), dim3(total), dim3(256), 0, st, dtab, n);
        else hipLaunchKernelGGL((k_sweep_init<float, false>), dim3(total), dim3(256), 0, st, dtab, n);
    } else {
        if (conj_b) hipLaunchKernelGGL((k_sweep_init<double, true>), dim3(total), dim3(256), 0, st, dtab, n);
        else hipLaunchKernelGGL((k_sweep_init<double, false>), dim3(total), dim3(256), 0, st, dtab, n);
    }
}

int sweep_uniform(const SweepTab& tab, int n) {
    int uni = sweep_row_tiles(tab.c[0].np);
    for (int q = 0; q < n; ++q)
        if (tab.c[q].tile0 != q * uni || sweep_row_tiles(tab.c[q].np) != uni) uni = 0;
    return uni;
}

int sweep_unroll(int np_max) {
    const int per_wave = ((np_max >> 4) + SW_WAVES - 1) / SW_WAVES;
    return std::min(8, (per_wave + 1) & ~1);
}

template <int U>
static void launch_sweep_u(const SweepTab* dtab, int n, int t, int uni, int groups, int st, bool fp32, bool forward,
                           bool conj_b, hipStream_t st_) {
    const dim3 grid(sweep_grid(groups, st)), block(64 * SW_WAVES);
    if (fp32) {
        if (forward) {
            if (conj_b) hipLaunchKernelGGL((k_sweep<float, true, true, U>), grid, block, 0, st_, n, t, groups, st, uni, dtab);
            else hipLaunchKernelGGL((k_sweep<float, true, false, U>), grid, block, 0, st_, n, t, groups, st, uni, dtab);
        } else hipLaunchKernelGGL((k_sweep<float, false, false, U>), grid, block, 0, st_, n, t, groups, st, uni, dtab);
    } else {
        if (forward) {
            if (conj_b) hipLaunchKernelGGL((k_sweep<double, true, true, U>), grid, block, 0, st_, n, t, groups, st, uni, dtab);
            else hipLaunchKernelGGL((k_sweep<double, true, false, U>), grid, block, 0, st_, n, t, groups, st, uni, dtab);
        } else hipLaunchKernelGGL((k_sweep<double, false, false, U>), grid, block, 0, st_, n, t, groups, st, uni, dtab);
    }
}

void launch_sweep(const SweepTab* dtab, int n, int t, int uni, int unroll, int groups, int st, bool fp32, bool forward,
                  bool conj_b, hipStream_t st_) {
    switch (unroll) {
        case 2: launch_sweep_u<2>(dtab, n, t, uni, groups, st, fp32, forward, conj_b, st_); break;
        case 4: launch_sweep_u<4>(dtab, n, t, uni, groups, st, fp32, forward, conj_b, st_); break;
        case 6: launch_sweep_u<6>(dtab, n, t, uni, groups, st, fp32, forward, conj_b, st_); break;
        default: launch_sweep_u<8>(dtab, n, t, uni, groups, st, fp32, forward, conj_b, st_); break;
    }
}

}  // namespace helm
