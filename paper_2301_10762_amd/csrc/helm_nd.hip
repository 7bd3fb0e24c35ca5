// Nested-dissection factorisation and solves of libhelm (gfx950, complex128).
//
// The elimination tree of the grid (helm_nd_plan.hip) is processed level by
// level, deepest first, every front of a level and every system of a batch
// in the same launches.  A front is the dense symmetric matrix
//     M = [ P  F ; F^T  C ]   (p pivots, b ring nodes)
// made of the operator's entries at its pivots and the two children's Schur
// complements; eliminating its pivots in place by block Gauss-Jordan,
//     M -> [ G  G F ; -F^T G  C - F^T G F ],   G = P^{-1},
// leaves what the solves need (G and R = G F) and the Schur complement for
// the parent.  The five-point operator is complex symmetric, and the form
// above keeps M_JI = M_IJ^T up to the sign of eliminated rows, so only the
// tiles on and above the diagonal are computed.
//
// Against one dense block per grid row (helm_factor.hip) this does
// O(n^3) work instead of O(n^4) and, what counts for one system, a
// chain of about 3 n pivots instead of n^2 / 2.
#include "helm_nd.h"
#include "helm_launch.h"
#include "helm_tile.h"

#include <type_traits>

namespace helm {

// Records of the plan and of the launch tables are read as whole words
// through the constant address space, at wave-uniform indices (scalar loads).
template <typename R>
__device__ __forceinline__ R nd_record(const R* tab, int i) {
    constexpr int W = (int)(sizeof(R) / 4);
    const __attribute__((address_space(4))) uint32_t* p =
        (const __attribute__((address_space(4))) uint32_t*)(tab + __builtin_amdgcn_readfirstlane(i));
    uint32_t v[W];
#pragma unroll
    for (int q = 0; q < W; ++q) v[q] = p[q];
#pragma unroll
    for (int q = 0; q < W; ++q) v[q] = __builtin_amdgcn_readfirstlane(v[q]);
    R r;
    __builtin_memcpy(&r, v, sizeof(R));
    return r;
}


// What a front gathers from: its children's Schur complements, or a leaf
// child's inverse G (its Schur complement is -c_r c_c G at the leaf nodes the
// ring nodes r and c couple to, c the couplings' magnitudes).
struct NdKids {
    const double2* s[2];
    int ld[2];
    double sign[2];
};
__device__ __forceinline__ NdKids nd_kids(const NdTabs& t, const NdFront& f, const NdSys& y, int parity) {
    NdKids k;
    const double2* base = parity ? y.work[0] : y.work[1];   // the level below
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        k.s[c] = base;
        k.ld[c] = 0;
        k.sign[c] = 1.0;
        if (f.child[c] >= 0) {
            const NdFront g = nd_record(t.fronts, f.child[c]);
            k.s[c] = g.leaf ? y.fac + g.fac : base + g.s;
            k.ld[c] = g.leaf ? g.p : g.b;
            k.sign[c] = g.leaf ? -1.0 : 1.0;
        }
    }
    return k;
}

// Row or column q of a front's padded matrix: everything its entries need.
struct NdIndex {
    int i, j;          // grid node; i = -4: padding
    int m[2];          // its places in the children's Schur complements, -1: not there
    int piv, pad_;     // a pivot (padding pivots too)
    double c[2];       // scale of the children's entries
    double cx, cz;     // its couplings along x and z
    double2 dg;        // the operator's diagonal entry (pivots; 1 in the padding)
};
__device__ __forceinline__ NdIndex nd_index(const NdTabs& t, const NdFront& f, const NdKids& k, const Coef& cf, int q) {
    NdIndex r;
    r.piv = q < f.pp;
    r.i = -4 - 4 * q;   // no two padding rows are neighbours
    r.j = 0;
    r.m[0] = r.m[1] = -1;
    r.pad_ = 0;
    r.c[0] = r.c[1] = 1.0;
    r.cx = r.cz = 0.0;
    r.dg = make_double2(1.0, 0.0);
    const int l = r.piv ? (q < f.p ? q : -1) : (q - f.pp < f.b ? f.p + q - f.pp : -1);
    if (l < 0) return r;
    if (f.leaf) {
        r.j = f.z0 + l / f.w;
        r.i = f.x0 + l % f.w;
    } else {
        const int node = t.nodeof[l < f.p ? f.piv0 + l : t.ring[f.ring + l - f.p]];
        r.j = node / cf.nx;
        r.i = node - r.j * cf.nx;
    }
    r.cx = x_coupling(cf, r.j);
    r.cz = z_coupling(cf, r.i);
    if (r.piv) r.dg = diag_entry(cf, r.i, r.j);
    if (!f.leaf) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            r.m[c] = t.map[f.map[c] + l];
            if (k.sign[c] < 0.0) {
                const NdFront& g = t.fronts[f.child[c]];
                r.c[c] = (r.i < g.x0 || r.i >= g.x0 + g.w) ? r.cx : r.cz;
            }
        }
    }
    return r;
}

// Entry (r, c) of a front before its elimination.  Both loads are made at
// in-range addresses whether or not the child has the entry.
__device__ __forceinline__ double2 nd_entry(const NdKids& k, bool kids, const NdIndex& r, const NdIndex& c) {
    double2 o = make_double2(0.0, 0.0);
    if (kids) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bool has = r.m[q] >= 0 && c.m[q] >= 0;
            const double2 v =
                gld(k.s[q] + (has ? (int64_t)min(r.m[q], c.m[q]) * k.ld[q] + max(r.m[q], c.m[q]) : 0));
            const double s = k.sign[q] * r.c[q] * c.c[q];
            o.x += has ? s * v.x : 0.0;
            o.y += has ? s * v.y : 0.0;
        }
    }
    if (r.piv | c.piv) {
        const int di = abs(c.i - r.i), dj = abs(c.j - r.j);
        if (di + dj == 0) {
            o.x += r.dg.x;
            o.y += r.dg.y;
        } else if (di + dj == 1) {
            o.x -= di ? r.cx : r.cz;
        }
    }
    return o;
}

// Notes how far a system's tile inverses grow (m2: this lane's largest
// |T_ij|^2 over the couplings' scale), one bit per step of ND_GROWN: a box near
// resonance, behind which solves lose digits (ND_GROWN).
__device__ __forceinline__ void nd_grown(const NdSys& y, float m2, bool valid) {
    const float sc = (float)fmax(y.cf.hz / y.cf.hx, y.cf.hx / y.cf.hz), v = m2 * sc * sc;
    int bits = 0;
#pragma unroll
    for (int k = 0; k < ND_STEPS; ++k)
        if (__any(valid && !(v <= ND_GROWN[k]))) bits |= 1 << k;
    if (bits && (threadIdx.x & 63) == 0 && (bits & ~y.status[3])) atomicOr(&y.status[3], bits);
}
__device__ __forceinline__ float nd_max2(const double2 (&a)[4]) {
    float m2 = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) m2 = fmaxf(m2, (float)(a[e].x * a[e].x + a[e].y * a[e].y));
    return m2;
}

// Inverse of the n x n tile in S (row stride ld) with partial pivoting, by
// one wavefront in LDS; the inverse is left in D.  Only reached where the
// diagonal pivots are too small.  Returns the first step without a nonzero
// pivot, or -1.
__device__ __noinline__ int nd_pivoted(double2* S, double2* D, int ld, int n) {
    const int l = threadIdx.x & 63;
    int zero = -1;
    for (int i = l; i < n * n; i += 64) D[(i / n) * ld + i % n] = make_double2(i / n == i % n ? 1.0 : 0.0, 0.0);
    for (int p = 0; p < n; ++p) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        int best = p;
        double bm = -1.0;
        for (int i = p; i < n; ++i) {   // every lane scans the column
            const double2 v = S[i * ld + p];
            const double m = v.x * v.x + v.y * v.y;
            if (m > bm) { bm = m; best = i; }
        }
        if (!(bm > 0.0) && zero < 0) zero = p;
        const double2 d = bm > 0.0 ? crcp(S[best * ld + p]) : make_double2(0.0, 0.0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        for (int c = l; c < 2 * n; c += 64) {   // exchange rows, scale the pivot row
            double2* M = c < n ? S + c : D + c - n;
            const double2 a = M[best * ld], b = M[p * ld];
            M[best * ld] = b;
            M[p * ld] = cmul(a, d);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        for (int i = 0; i < n; ++i) {
            if (i == p) continue;
            const double2 f = S[i * ld + p];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            for (int c = l; c < 2 * n; c += 64) {
                double2* M = c < n ? S + c : D + c - n;
                const double2 r = M[p * ld], a = M[i * ld];
                M[i * ld] = make_double2(a.x - (f.x * r.x - f.y * r.y), a.y - (f.x * r.y + f.y * r.x));
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    return zero;
}

// ------------------------------------------------------------------- leaves --
// G = A^{-1} of a leaf box (at most ND_LEAF_MAX nodes), one wavefront per leaf: the
// upper 16 x 16 tiles in accumulator registers, panels of 16 pivots through
// LDS.  Per panel K, with C_I = M_IK (from the stored upper tiles; M_KI =
// s_I M_IK^T, s_I = -1 where I is eliminated) and T the inverse of tile KK:
//     W_I = -C_I T,  M_IJ += s_J W_I C_J^T,  M_IK = W_I,  M_KJ = -s_J W_J^T,
//     M_KK = T.
// Panels may be taken in any order: a tile that is nearly singular by itself
// waits until the others are eliminated.  A single leaf is a chain of three
// tile inverses (6 k of its 33 k cycles each, 27 us a launch at 101^2); many
// are bound by vector instructions, two wavefronts to a SIMD: 20480 leaves of
// 36 nodes take 420 us, whose factor is 425 MB to write (94 us at the rate of
// a copy).
constexpr int LT = 3;
static_assert(16 * LT >= ND_LEAF_MAX, "a leaf's tiles");
__global__ __launch_bounds__(64, 2) void k_nd_leaf(NdTabs t, int first, const NdSysTab* __restrict__ stab) {
    constexpr int NTT = LT * (LT + 1) / 2;
    __shared__ double2 sC[LT * 16][17];   // C; rows of the panel itself hold its diagonal tile
    __shared__ double2 sW[LT * 16][17];   // W; rows of the panel itself hold the tile's inverse
    const NdSys y = nd_record(stab->s, blockIdx.y);
    const NdFront f = nd_record(t.fronts, first + (int)blockIdx.x);
    const int l = threadIdx.x, lr = l & 15, lg = l >> 4, nt = f.pp >> 4;
    NdKids kids;
    kids.sign[0] = kids.sign[1] = 1.0;
    NdIndex* sidx = (NdIndex*)&sW[0][0];
    if (l < f.pp) sidx[l] = nd_index(t, f, kids, y.cf, l);
    __syncthreads();
    v4d re[NTT], im[NTT];
#pragma unroll
    for (int j = 0, i = 0; j < LT; ++j)
#pragma unroll
        for (int ii = 0; ii <= j; ++ii, ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                re[i][e] = 0.0;
                im[i][e] = 0.0;
                if (j < nt) {
                    const double2 v = nd_entry(kids, false, sidx[16 * ii + lg + 4 * e], sidx[16 * j + lr]);
                    re[i][e] = v.x;
                    im[i][e] = v.y;
                }
            }
    __syncthreads();   // sidx shares sW
    uint32_t left = (1u << nt) - 1u;
    while (left) {
        int K = -1;
        for (uint32_t cand = y.pivot ? 0u : left; cand; cand &= cand - 1) {
            const int c = __builtin_ctz(cand);
            double2 q[4];   // the tile is symmetric: its columns are its rows
#pragma unroll
            for (int j = 0, i = 0; j < LT; ++j)
#pragma unroll
                for (int ii = 0; ii <= j; ++ii, ++i)
                    if (ii == j && j == c) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) q[e] = make_double2(re[i][e], im[i][e]);
                    }
            const float thr = TAU2 * __uint_as_float(wave_max_u32(__float_as_uint(nd_max2(q))));
            bool small = false;
            gj16_wave<double>(q, thr, small);
            if (!small) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sW[16 * c + lg + 4 * e][lr] = q[e];
                nd_grown(y, nd_max2(q), true);
                K = c;
                break;
            }
        }
        if (K < 0) {
            K = __builtin_ctz(left);
#pragma unroll
            for (int j = 0, i = 0; j < LT; ++j)
#pragma unroll
                for (int ii = 0; ii <= j; ++ii, ++i)
                    if (ii == j && j == K) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) sC[16 * K + lg + 4 * e][lr] = make_double2(re[i][e], im[i][e]);
                    }
            __syncthreads();
            const int zero = nd_pivoted(&sC[16 * K][0], &sW[16 * K][0], 17, 16);
            double2 q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = sW[16 * K + lr][4 * lg + e];
            nd_grown(y, nd_max2(q), true);
            if (zero >= 0 && l == 0) report_zero_pivot(y.status, first + (int)blockIdx.x, 16 * K + zero);
        }
        const uint32_t done = ((1u << nt) - 1u) & ~left;   // eliminated before this one
        left &= ~(1u << K);
#pragma unroll
        for (int j = 0, i = 0; j < LT; ++j)
#pragma unroll
            for (int ii = 0; ii <= j; ++ii, ++i) {
                if (j >= nt || ii == j) continue;
                if (j == K) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sC[16 * ii + lg + 4 * e][lr] = make_double2(re[i][e], im[i][e]);
                } else if (ii == K) {
                    const double s = (done >> j) & 1u ? -1.0 : 1.0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) sC[16 * j + lr][lg + 4 * e] = make_double2(s * re[i][e], s * im[i][e]);
                }
            }
        __syncthreads();
        for (int I = 0; I < nt; ++I) {
            if (I == K) continue;
            v4d wr, wi;
#pragma unroll
            for (int e = 0; e < 4; ++e) { wr[e] = 0.0; wi[e] = 0.0; }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double2 x = sC[16 * I + lr][4 * q + lg], v = sW[16 * K + 4 * q + lg][lr];
                cmfma<double, v4d>(wr, wi, x.x, x.y, v.x, v.y);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) sW[16 * I + lg + 4 * e][lr] = make_double2(-wr[e], -wi[e]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0, i = 0; j < LT; ++j)
#pragma unroll
            for (int ii = 0; ii <= j; ++ii, ++i) {
                if (j >= nt) continue;
                const double s = (done >> j) & 1u ? -1.0 : 1.0;   // M_KJ = s C_J^T
                if (j == K) {   // also the diagonal tile: its inverse is in its rows of sW
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double2 v = sW[16 * ii + lg + 4 * e][lr];
                        re[i][e] = v.x;
                        im[i][e] = v.y;
                    }
                } else if (ii == K) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double2 v = sW[16 * j + lr][lg + 4 * e];
                        re[i][e] = -s * v.x;
                        im[i][e] = -s * v.y;
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const double2 x = sW[16 * ii + lr][4 * q + lg], v = sC[16 * j + lr][4 * q + lg];
                        cmfma<double, v4d>(re[i], im[i], x.x, x.y, s * v.x, s * v.y);
                    }
                }
            }
        __syncthreads();
    }
    double2* fac = y.fac + f.fac;
#pragma unroll
    for (int j = 0, i = 0; j < LT; ++j)
#pragma unroll
        for (int ii = 0; ii <= j; ++ii, ++i) {
            if (j >= nt) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 16 * ii + lg + 4 * e, col = 16 * j + lr;
                const double2 v = make_double2(re[i][e], im[i][e]);
                if (row < f.p && col < f.p) {
                    gst(fac + col * f.p + row, v);
                    if (ii < j) gst(fac + row * f.p + col, v);
                }
            }
        }
}

// Inverse of the kb x kb tile in a[] (256-thread layout of inv_blocked, in
// the first 256 threads) into L2 (stride 33, plain) with diagonal pivots, or
// with partial pivoting where one of them is small (or pivoting is forced).
// L2: kb x 33, and twice as much for kb = 32.
union NdScratch {
    RowScratch<double> row;
    GJScratch<double> gj;
};
__device__ __forceinline__ void nd_gj(double2 (&a)[4], int kb, const NdSys& y, int front, int k0, NdScratch& sh,
                                      double2* L2) {
    const int t = threadIdx.x, r = t >> 3, cg = t & 7;
    const bool act = r < kb && 4 * cg < kb;
    __syncthreads();
    const int zero = kb == 32 ? gj_invert<double, 32>(a, sh.gj) : gj_invert<double, 16>(a, sh.gj);
    __syncthreads();
    // T[i][c] = M[rowOf[i]][stepOf[c]], row rowOf[i] in step i
    if (act) {
        const int i = sh.gj.stepOf[r];
        int back[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) back[e] = sh.gj.rowOf[4 * cg + e];
#pragma unroll
        for (int e = 0; e < 4; ++e) L2[i * 33 + back[e]] = a[e];
    }
    if (zero >= 0 && t == 0) report_zero_pivot(y.status, front, k0 + zero);
    __syncthreads();
}
template <typename W>
__device__ __forceinline__ void nd_invert(double2 (&a)[4], int kb, const NdSys& y, int front, int k0, NdScratch& sh,
                                          double2* L2, W beside) {
    const int t = threadIdx.x, r = t >> 3, cg = t & 7;
    const bool act = r < kb && 4 * cg < kb;
    bool pivot = y.pivot;
    if (!pivot) pivot = inv_blocked<double>(a, kb, L2, sh.row, TAU2, beside);
    if (pivot) nd_gj(a, kb, y, front, k0, sh, L2);
    double2 q[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = L2[(act ? r : 0) * 33 + (act ? 4 * cg + e : 0)];
    nd_grown(y, nd_max2(q), act);
}

// ------------------------------------------------------------- narrow fronts --
// A front of at most 32 pivots in one workgroup.  The pivot block is inverted
// whole (G); beside it the couplings F^T (one row per ring node) are gathered
// into LDS.  Each wavefront then takes rows of ring tiles by itself:
// R_I = G F_I, whose accumulators are also the A operand of the next product
// (the FP64 result holds rows g + 4 e of column r in lane 16 g + r), so for
// half of the tiles J of the symmetric complement the children's part minus
// R_I^T F_J goes straight there.  No tile is held across a barrier, so
// registers and latency stay low; a tile's children's parts are loaded while
// the one before is multiplied.
// One front is bound by that chain: 90 k cycles at p = 25 when the couplings
// were gathered first and wavefront I took all J >= I, 70 k now (101^2: two
// launches 91 us, now 70).  401^2, 5 systems: two 32-wide levels 459 us, now
// 405; three 16-wide ones 641, now 500, with four workgroups to a compute unit.
template <int KP>
__global__ __launch_bounds__(KP == 16 ? 256 : 512, KP == 16 ? 4 : 2) void k_nd_front(NdTabs t, int first, int parity, int fmax,
                                                                   const NdSysTab* __restrict__ stab) {
    // all of its LDS (nd_front_lds, which decides whether a level comes here)
    extern __shared__ __attribute__((aligned(16))) char nd_smem[];
    constexpr int LD = KP + 1, NTH = KP == 16 ? 256 : 512, NW = NTH / 64;
    double2* L2 = (double2*)nd_smem;                            // G, and for KP = 32 inversion scratch behind it
    double2* sF = L2 + (KP == 16 ? 16 * 33 : 2 * 32 * 33);      // [ring][LD]
    NdIndex* sidx = (NdIndex*)(sF + (size_t)(fmax - 16) * LD);  // fmax entries
    NdScratch& sh = *(NdScratch*)(sidx + fmax);
    const NdSys y = nd_record(stab->s, blockIdx.y);
    const NdFront f = nd_record(t.fronts, first + (int)blockIdx.x);
    const NdKids kids = nd_kids(t, f, y, parity);
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, lr = l & 15, lg = l >> 4;
    const int p = f.p, b = f.b, pp = f.pp, nb = (f.fp - pp) >> 4;
    for (int q = tid; q < f.fp; q += NTH) sidx[q] = nd_index(t, f, kids, y.cf, q);
    __syncthreads();
    {
        const int r = tid >> 3, cg = tid & 7;
        const bool in = r < pp && 4 * cg < pp;
        double2 a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = nd_entry(kids, true, sidx[in ? r : 0], sidx[in ? 4 * cg + e : 0]);
            if (!in) a[e] = make_double2(0.0, 0.0);
        }
        // F^T, the ring index fastest, so that a child's rows are read along:
        // by the wavefronts that the inversion leaves free (all of them
        // before it when every tile is to be pivoted)
        auto couple = [&](int k0, auto nk) {
            constexpr int NK = decltype(nk)::value, PER = (KP + NK - 1) / NK;
            for (int i = l; i < 16 * nb; i += 64) {
                const NdIndex c = sidx[pp + i];
                double2 v[PER];
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    const int k = k0 + NK * q;
                    v[q] = nd_entry(kids, true, sidx[min(k, pp - 1)], c);
                    if (k >= pp) v[q] = make_double2(0.0, 0.0);
                }
#pragma unroll
                for (int q = 0; q < PER; ++q)
                    if (k0 + NK * q < KP) sF[(size_t)i * LD + k0 + NK * q] = v[q];
            }
        };
        if (y.pivot) couple(w, std::integral_constant<int, NW>{});
        nd_invert(a, pp, y, first + (int)blockIdx.x, 0, sh, L2,
                  [&] { couple(w - 1, std::integral_constant<int, NW - 1>{}); });
    }
    __syncthreads();
    double2* fac = y.fac + f.fac;
    for (int c = w; c < p; c += NW)
        if (l < p) gst(fac + c * p + l, L2[l * 33 + c]);
    double2* S = (parity ? y.work[1] : y.work[0]) + f.s;
    const int np = pp >> 4;
    for (int I = w; I < nb; I += NW) {
        double2 s[4];
        auto gather = [&](int J) {
            const NdIndex& c = sidx[pp + 16 * J + lr];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = nd_entry(kids, true, sidx[pp + 16 * I + lg + 4 * e], c);
        };
        gather(I);
        double2 ra[KP / 4];   // -R_I, as results and as operand
#pragma unroll
        for (int kt = 0; kt < KP / 16; ++kt) {
            v4d p1, p2, p3, wr, wi;
#pragma unroll
            for (int e = 0; e < 4; ++e) { p1[e] = 0.0; p2[e] = 0.0; p3[e] = 0.0; }
            if (kt < np)
                for (int m = 0; m < pp; m += 4) {
                    const double2 g = L2[(16 * kt + lr) * 33 + m + lg], x = sF[(size_t)(16 * I + lr) * LD + m + lg];
                    cmfma3<double, v4d>(p1, p2, p3, g.x, g.y, x.x, x.y);
                }
            cacc_final<true, v4d>(p1, p2, p3, wr, wi);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 16 * I + lr, k = 16 * kt + lg + 4 * e;
                if (i < b && k < p) gst(fac + (p + i) * p + k, make_double2(wr[e], wi[e]));
                ra[4 * kt + e] = make_double2(-wr[e], -wi[e]);
            }
        }
        // half of the tiles of row I of the symmetric complement, J = I, I + 1,
        // ... around the ring: every wavefront takes as many
        const int half = (nb & 1) || I < nb / 2 ? nb / 2 + 1 : nb / 2;
        for (int d = 0, J = I; d < half; ++d) {
            v4d a1, a2, a3, re, im;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                re[e] = s[e].x;
                im[e] = s[e].y;
            }
            cacc_seed<true, v4d>(a1, a2, a3, re, im);
            const int J1 = J + 1 < nb ? J + 1 : 0;
            if (d + 1 < half) gather(J1);
#pragma unroll
            for (int q = 0; q < KP / 4; ++q) {
                const double2 x = sF[(size_t)(16 * J + lr) * LD + 4 * q + lg];
                cmfma3<double, v4d>(a1, a2, a3, ra[q].x, ra[q].y, x.x, x.y);
            }
            cacc_final<true, v4d>(a1, a2, a3, re, im);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 16 * I + lg + 4 * e, j = 16 * J + lr;
                if (i < b && j < b) gst(S + (J < I ? (int64_t)j * b + i : (int64_t)i * b + j), make_double2(re[e], im[e]));
            }
            J = J1;
        }
    }
}

// --------------------------------------------------------------- wide fronts --
// The pivot rows [P F] (pp x fp) are eliminated by panels of 32, one launch
// per panel, to [G R]; one more launch forms the Schur complement
// C - F^T R with the whole depth p at once, its children's part gathered on
// the way, so that the ring part (most of the front) is read and written
// once.  (Eliminating the whole front panel by panel rewrote it p / 32
// times: 118 us a panel at 80 fronts with p = 100, b = 400, 3.7 TB/s.)
// Working memory: the gathered rows, kept for F, then two buffers in turn.
// A launch takes the next diagonal tile's inverse in a workgroup of its own
// beside the update tiles.  That chain (26 k cycles: loads, two products, the
// inverse) bounds the levels near the root, 12.5 us a panel at 401^2; with
// many fronts the update tiles do, in 32 x 64 so that three share a compute
// unit (5 systems of 401^2, 39 steps: 1314 us in 64 x 64 tiles of four real
// products, 1132 in these, 1082 with the next tile's workgroup ahead).
__device__ __forceinline__ double2* nd_rows(const NdFront& f, double2* work, int step) {
    const int64_t n = (int64_t)f.pp * f.fp;
    return work + f.work + (step == 0 ? 0 : n * (1 + (step & 1)));
}
__device__ __forceinline__ double2* nd_tslot(const NdFront& f, double2* work, int step) {
    return work + f.work + 3 * (int64_t)f.pp * f.fp + (step & 1) * KB * KB;
}

__global__ __launch_bounds__(256) void k_nd_gather(NdTabs t, int first, int count, int tile0, int parity,
                                                   const NdSysTab* __restrict__ stab) {
    __shared__ double2 L2[2 * 32 * 33];
    __shared__ NdScratch sh;
    __shared__ NdIndex sr[64], sc[64];
    const NdSys y = nd_record(stab->s, blockIdx.y);
    double2* work = parity ? y.work[1] : y.work[0];
    const int b = blockIdx.x, tid = threadIdx.x;
    const bool lead = b < count;
    const NdTile tl = lead ? NdTile{b, 0, 0} : nd_record(t.tiles, tile0 + b - count);
    const NdFront f = nd_record(t.fronts, first + tl.front);
    const NdKids kids = nd_kids(t, f, y, parity);
    const int I0 = KB * tl.ti, J0 = TILE * tl.tj;
    if (tid < 64) sr[tid] = nd_index(t, f, kids, y.cf, min(I0 + tid, f.fp - 1));
    else if (tid < 128) sc[tid - 64] = nd_index(t, f, kids, y.cf, min(J0 + tid - 64, f.fp - 1));
    __syncthreads();
    if (lead) {   // the inverse of the first diagonal tile
        const int r = tid >> 3, cg = tid & 7;
        double2 a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = nd_entry(kids, true, sr[r], sc[4 * cg + e]);
            if (r >= f.pp || 4 * cg >= f.pp) a[e] = make_double2(0.0, 0.0);
        }
        nd_invert(a, min(KB, f.pp), y, first + b, 0, sh, L2, NoWork{});
        store_inverse<double>(min(KB, f.pp), L2, nd_tslot(f, work, 0));
        return;
    }
    double2* X = nd_rows(f, work, 0);
    const int cc = tid & 63, col = J0 + cc;
#pragma unroll 4
    for (int q = 0; q < 8; ++q) {
        const int rr = (tid >> 6) + 4 * q, row = I0 + rr;
        if (row < f.pp && col < f.fp) gst(X + (int64_t)row * f.fp + col, nd_entry(kids, true, sr[rr], sc[cc]));
    }
}

// Next diagonal tile: Z = X_K'K' - X_K'K T X_KK', and its inverse.
__device__ __forceinline__ void nd_next_tile(const NdFront& f, const NdSys& y, int front, int step, const double2* X,
                                             const double2* Tcur, double2* Tnext, char* smem) {
    const int k0 = step * KB, kn0 = k0 + KB;   // a next panel exists, so this one is full
    const int kbn = min(KB, f.pp - kn0), fp = f.fp;
    double2 (*sA)[33] = (double2(*)[33])smem;                            // X_K'K
    double2 (*sT)[33] = (double2(*)[33])(smem + 1 * 32 * 33 * 16);       // T, then the inversion buffers
    double2 (*sB)[33] = (double2(*)[33])(smem + 2 * 32 * 33 * 16);       // X_KK'
    double2 (*sP)[33] = sT;                                              // X_K'K T, once T is read
    NdScratch& sh = *(NdScratch*)sB;                                     // for the pivoted inverse, at the end
    RowScratch<double>& rs = *(RowScratch<double>*)(smem + 3 * 32 * 33 * 16);
    const int t = threadIdx.x, w = t >> 6, l = t & 63, lr = l & 15, lg = l >> 4, wr = w >> 1, wc = w & 1;
    double2 tl[4], xa[4], xb[4], xz[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int idx = t + 256 * i, hi = idx >> 5, lo = idx & 31;
        tl[i] = gld(Tcur + idx);
        xa[i] = gld(X + (int64_t)(kn0 + min(hi, kbn - 1)) * fp + k0 + lo);
        xb[i] = gld(X + (int64_t)(k0 + hi) * fp + kn0 + min(lo, kbn - 1));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int rr = 16 * wr + acc_row<double>(lg, e), cc = 16 * wc + lr;
        xz[e] = gld(X + (int64_t)(kn0 + min(rr, kbn - 1)) * fp + kn0 + min(cc, kbn - 1));
    }
    __builtin_amdgcn_sched_barrier(0);
    const double2 cz = make_double2(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int idx = t + 256 * i, hi = idx >> 5, lo = idx & 31;
        sT[lo][hi] = tl[i];
        sA[hi][lo] = csel_parts(hi < kbn, xa[i], cz);
        sB[hi][lo] = csel_parts(lo < kbn, xb[i], cz);
    }
    v4d zr, zi, pr, pim, p1, p2, p3;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int rr = 16 * wr + acc_row<double>(lg, e), cc = 16 * wc + lr;
        const double2 v = csel_parts(rr < kbn && cc < kbn, xz[e], cz);
        zr[e] = v.x;
        zi[e] = v.y;
        p1[e] = 0.0;
        p2[e] = 0.0;
        p3[e] = 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int s8 = 0; s8 < 8; ++s8) {
        const double2 x = sA[16 * wr + lr][4 * s8 + lg], v = sT[4 * s8 + lg][16 * wc + lr];
        cmfma3<double, v4d>(p1, p2, p3, x.x, x.y, v.x, v.y);
    }
    cacc_final<true, v4d>(p1, p2, p3, pr, pim);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) sP[16 * wr + acc_row<double>(lg, e)][16 * wc + lr] = make_double2(-pr[e], -pim[e]);
    __syncthreads();
    cacc_seed<true, v4d>(p1, p2, p3, zr, zi);
#pragma unroll
    for (int s8 = 0; s8 < 8; ++s8) {
        const double2 x = sP[16 * wr + lr][4 * s8 + lg], v = sB[4 * s8 + lg][16 * wc + lr];
        cmfma3<double, v4d>(p1, p2, p3, x.x, x.y, v.x, v.y);
    }
    cacc_final<true, v4d>(p1, p2, p3, zr, zi);
    double2* L2 = &sT[0][0];   // with the X_KK' buffer behind it, once that is read
    float m2 = 0.0f;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int rr = 16 * wr + acc_row<double>(lg, e), cc = 16 * wc + lr;
        const double2 z = make_double2(zr[e], zi[e]);
        L2[rr * 33 + cc] = z;
        sA[rr][cc] = z;   // kept for the pivoted inverse
        m2 = fmaxf(m2, (float)(zr[e] * zr[e] + zi[e] * zi[e]));
    }
    const uint32_t wm = wave_max_u32(__float_as_uint(m2));
    if (l == 0) rs.amax[w] = __uint_as_float(wm);
    if (t == 0) rs.small = 0;
    __syncthreads();
    const int r = t >> 3, cg = t & 7;
    const bool act = r < kbn && 4 * cg < kbn;
    bool pivot = y.pivot;
    if (!pivot) pivot = inv_blocked_core<double>(kbn, L2, rs, TAU2);
    if (pivot) {
        double2 a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = csel_parts(act, sA[r][4 * cg + e], cz);
        nd_gj(a, kbn, y, front, kn0, sh, L2);
    }
    store_inverse<double>(kbn, L2, Tnext);
    double2 q[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = L2[(act ? r : 0) * 33 + (act ? 4 * cg + e : 0)];
    nd_grown(y, nd_max2(q), act);
}

// One 32 x 64 tile of a panel step on the pivot rows: Y = X' + W V with
// W = [-X_IK T; T - I on rows of K], V = X_KJ (V_KK = I), X' = X with the K
// columns cleared (X'_KK = I).  The last panel writes to the factor store.
__device__ __forceinline__ void nd_update_tile(const NdFront& f, const NdSys& y, int step, int ti, int tj,
                                               const double2* X, double2* Y, const double2* Tcur, char* smem) {
    const int fp = f.fp, pp = f.pp, k0 = step * KB, kb = min(KB, pp - k0);
    const int I0 = ti * KB, J0 = tj * TILE;
    const int t = threadIdx.x, w = t >> 6, l = t & 63, lr = l & 15, lg = l >> 4, wr = w >> 1, wc = w & 1;
    double2 (*sW)[33] = (double2(*)[33])smem;
    double2 (*sV)[33] = (double2(*)[33])(smem + 32 * 33 * 16);
    double2 (*sT)[33] = sV;   // T shares the V buffer until W is formed
    const int R = I0 + 16 * wr;
    const bool vr = R < pp;
    int Cc[2];
    bool vc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        Cc[q] = J0 + 32 * wc + 16 * q;
        vc[q] = Cc[q] < fp;
    }
    double2 xik[4], tv[4], vv[8], xt[2][4];
    {
        const int rr = t >> 3, c4 = 4 * (t & 7), row = min(I0 + rr, pp - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) xik[q] = gld(X + (int64_t)row * fp + k0 + min(c4 + q, kb - 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) tv[q] = gld(Tcur + t + 256 * q);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = t + 256 * q, k = i >> 6, cc = i & 63;
            vv[q] = gld(X + (int64_t)(k0 + min(k, kb - 1)) * fp + min(J0 + cc, fp - 1));
        }
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                xt[bj][e] = gld(X + (int64_t)min(R + acc_row<double>(lg, e), pp - 1) * fp + min(Cc[bj] + lr, fp - 1));
    }
    __builtin_amdgcn_sched_barrier(0);   // keep every load ahead of the first wait
    const double2 zero = make_double2(0.0, 0.0);
    {
        const int rr = t >> 3, c4 = 4 * (t & 7);
#pragma unroll
        for (int q = 0; q < 4; ++q) sW[rr][c4 + q] = csel_parts(I0 + rr < pp && c4 + q < kb, xik[q], zero);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = t + 256 * q, c = i >> 5, k = i & 31;
            sT[k][c] = csel_parts(k < kb && c < kb, tv[q], zero);
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int i = t + 256 * q, k = i >> 6, col = J0 + (i & 63);
        vv[q] = csel_parts(col >= k0 && col < k0 + kb, make_double2(k == col - k0 ? 1.0 : 0.0, 0.0), vv[q]);
        vv[q] = csel_parts(k < kb && col < fp, vv[q], zero);
    }
    __syncthreads();
    {   // W: one 16 x 16 block per wavefront
        v4d wre, wim, q1, q2, q3;
#pragma unroll
        for (int e = 0; e < 4; ++e) { q1[e] = 0; q2[e] = 0; q3[e] = 0; }
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) {
            const int k = 4 * s8 + lg;
            const double2 av = sW[16 * wr + lr][k], bv = sT[k][16 * wc + lr];
            cmfma3<double, v4d>(q1, q2, q3, av.x, av.y, bv.x, bv.y);
        }
        cacc_final<true, v4d>(q1, q2, q3, wre, wim);
        double2 tk[4];   // rows of K: T - I, read before the buffers are rewritten
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = R + acc_row<double>(lg, e), c = 16 * wc + lr;
            const bool in = row >= k0 && row < k0 + kb;
            tk[e] = csel_parts(in, sT[in ? row - k0 : 0][c], zero);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int rl = 16 * wr + acc_row<double>(lg, e), row = I0 + rl, c = 16 * wc + lr;
            const bool in = row >= k0 && row < k0 + kb;
            double2 v = csel_parts(in, tk[e], make_double2(-wre[e], -wim[e]));
            if (in && row - k0 == c) v.x -= 1.0;
            sW[rl][c] = v;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = t + 256 * q, k = i >> 6, cc = i & 63;
            sV[cc][k] = vv[q];
        }
    }
    v4d a1[2], a2[2], a3[2];
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
        const int col = Cc[bj] + lr;
        const bool inK = col >= k0 && col < k0 + kb;
        v4d re, im;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = R + acc_row<double>(lg, e);
            double2 v = csel_parts(inK, make_double2(row == col ? 1.0 : 0.0, 0.0), xt[bj][e]);
            v = csel_parts(vr && vc[bj], v, zero);
            re[e] = v.x;
            im[e] = v.y;
        }
        cacc_seed<true, v4d>(a1[bj], a2[bj], a3[bj], re, im);
    }
    __syncthreads();
    for (int kk = 0; kk < kb; kk += 16) {
        double2 av[4], bv[2][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            av[s] = sW[16 * wr + lr][kk + 4 * lg + s];
#pragma unroll
            for (int q = 0; q < 2; ++q) bv[q][s] = sV[32 * wc + 16 * q + lr][kk + 4 * lg + s];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
                if (vr && vc[bj]) cmfma3<double, v4d>(a1[bj], a2[bj], a3[bj], av[s].x, av[s].y, bv[bj][s].x, bv[bj][s].y);
    }
    const bool last = step + 1 == f.npan;
    double2* fac = y.fac + f.fac;
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
        if (!(vr && vc[bj])) continue;
        const int col = Cc[bj] + lr;
        v4d re, im;
        cacc_final<true, v4d>(a1[bj], a2[bj], a3[bj], re, im);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = R + acc_row<double>(lg, e);
            const double2 g = make_double2(re[e], im[e]);
            if (!last) {
                yst(Y + (int64_t)row * fp + col, g);
            } else if (row < f.p) {
                const int c = col < pp ? (col < f.p ? col : -1) : (col - pp < f.b ? f.p + col - pp : -1);
                if (c >= 0) gst(fac + (int64_t)c * f.p + row, g);
            }
        }
    }
}

__global__ __launch_bounds__(256, 3) void k_nd_step(NdTabs t, int first, int count, int tile0, int parity, int step,
                                                    const NdSysTab* __restrict__ stab) {
    __shared__ __attribute__((aligned(16))) char smem[3 * 32 * 33 * 16 + sizeof(RowScratch<double>)];
    const NdSys y = nd_record(stab->s, blockIdx.y);
    const int b = blockIdx.x;
    const bool lead = b < count;
    const NdTile tl = lead ? NdTile{b, 0, 0} : nd_record(t.tiles, tile0 + b - count);
    const NdFront f = nd_record(t.fronts, first + tl.front);
    if (step >= f.npan) return;
    double2* work = parity ? y.work[1] : y.work[0];
    const double2* X = nd_rows(f, work, step);
    const double2* Tcur = nd_tslot(f, work, step);
    if (lead) {
        // ahead of the update tiles that share its compute unit
        __builtin_amdgcn_s_setprio(3);
        if (step + 1 < f.npan) nd_next_tile(f, y, first + b, step, X, Tcur, nd_tslot(f, work, step + 1), smem);
    } else {
        nd_update_tile(f, y, step, tl.ti, tl.tj, X, nd_rows(f, work, step + 1), Tcur, smem);
    }
}

// Schur complement S = C - F^T R of wide fronts, one 64 x 64 tile (ti <= tj)
// of the ring per workgroup, depth p in chunks of 32 through LDS; the next
// chunk is loaded while this one is multiplied.  401^2, 5 systems: six levels
// 678 us, about a third of the matrix cores' rate: the gather of the
// children's part, and two workgroups to a compute unit (240 registers).
__global__ __launch_bounds__(256, 2) void k_nd_schur(NdTabs t, int first, int tile0, int parity,
                                                     const NdSysTab* __restrict__ stab) {
    __shared__ double2 sA[64][33], sB[64][33];   // F^T and R^T: [ring][k]
    const NdSys y = nd_record(stab->s, blockIdx.y);
    const NdTile tl = nd_record(t.tiles, tile0 + (int)blockIdx.x);
    const NdFront f = nd_record(t.fronts, first + tl.front);
    const NdKids kids = nd_kids(t, f, y, parity);
    double2* work = parity ? y.work[1] : y.work[0];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, lr = l & 15, lg = l >> 4, wr = w >> 1, wc = w & 1;
    const int I0 = TILE * tl.ti, J0 = TILE * tl.tj, p = f.p, b = f.b;
    NdIndex* sr = (NdIndex*)&sA[0][0];
    NdIndex* sc = sr + 64;
    if (tid < 64) sr[tid] = nd_index(t, f, kids, y.cf, min(f.pp + I0 + tid, f.fp - 1));
    else if (tid < 128) sc[tid - 64] = nd_index(t, f, kids, y.cf, min(f.pp + J0 + tid - 64, f.fp - 1));
    const double2* F = nd_rows(f, work, 0) + f.pp;
    const double2* R = y.fac + f.fac + (int64_t)p * p;
    double2 fa[8], fb[8];
    auto load = [&](int k0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = k0 + (tid >> 6) + 4 * q, i = tid & 63;
            fa[q] = gld(F + (int64_t)min(k, p - 1) * f.fp + min(I0 + i, b - 1));
            const int kb = k0 + (tid & 31), j = (tid >> 5) + 8 * q;
            fb[q] = gld(R + (int64_t)min(J0 + j, b - 1) * p + min(kb, p - 1));
        }
    };
    load(0);
    __syncthreads();
    v4d a1[2][2], a2[2][2], a3[2][2];
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            v4d re, im;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double2 v = nd_entry(kids, true, sr[32 * wr + 16 * bi + lg + 4 * e], sc[32 * wc + 16 * bj + lr]);
                re[e] = v.x;
                im[e] = v.y;
            }
            cacc_seed<true, v4d>(a1[bi][bj], a2[bi][bj], a3[bi][bj], re, im);
        }
    for (int k0 = 0; k0 < p; k0 += 32) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int ka = (tid >> 6) + 4 * q, i = tid & 63;
            sA[i][ka] = csel_parts(k0 + ka < p, make_double2(-fa[q].x, -fa[q].y), make_double2(0.0, 0.0));
            const int kb = tid & 31, j = (tid >> 5) + 8 * q;
            sB[j][kb] = csel_parts(k0 + kb < p, fb[q], make_double2(0.0, 0.0));
        }
        __syncthreads();
        if (k0 + 32 < p) load(k0 + 32);
#pragma unroll
        for (int kk = 0; kk < 32; kk += 16) {
            double2 av[2][4], bv[2][4];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    av[q][s] = sA[32 * wr + 16 * q + lr][kk + 4 * lg + s];
                    bv[q][s] = sB[32 * wc + 16 * q + lr][kk + 4 * lg + s];
                }
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                    for (int bj = 0; bj < 2; ++bj)
                        cacc<true, double, v4d>(a1[bi][bj], a2[bi][bj], a3[bi][bj], av[bi][s].x, av[bi][s].y,
                                                bv[bj][s].x, bv[bj][s].y);
        }
    }
    double2* S = work + f.s;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            v4d re, im;
            cacc_final<true, v4d>(a1[bi][bj], a2[bi][bj], a3[bi][bj], re, im);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = I0 + 32 * wr + 16 * bi + lg + 4 * e, j = J0 + 32 * wc + 16 * bj + lr;
                if (i < b && j < b) gst(S + (int64_t)i * b + j, make_double2(re[e], im[e]));
            }
        }
}

// --------------------------------------------------------------------- solve --
// Vectors have one row of S right-hand sides per node: [row][S].  Forward,
// deepest level first: a front's pivots are
//     y = b + (children's ring contributions there),
// and its own contributions to its ring are
//     u = (children's contributions there) - R^T y.
// Backward, root first: x = G y - R x_ring.  All sums have one fixed order,
// and no result depends on the other columns or systems of a launch.

__device__ __forceinline__ void nd_put_x(double2* x, double2 v, bool add) {
    if (add) {
        const double2 o = gld(x);
        v = make_double2(o.x + v.x, o.y + v.y);
    }
    gst(x, v);
}

// ------------------------------------------------------------------ subtrees --
// One workgroup sweeps a subtree (a box of about 12 x 12 nodes: four leaves,
// three separators) with 16 columns of vectors in LDS, so that the bottom
// levels cost one launch and one pass over the right-hand sides instead of a
// launch and a round trip of ring contributions per level (401^2, 64 columns,
// 5 systems: forward levels of 415 + 659 + 411 us).  It also moves the upper
// separators' right-hand sides and solutions, those right of its box and
// below it, which extend the runs it reads and writes (a launch of its own
// each way took 110 and 144 us there).
// Two workgroups share a compute unit.  What bounds them is their own phases,
// not memory: with every load of right-hand sides and operands and every
// store left out they took 278 of 345 us forward and 370 of 535 us backward
// (201^2, four systems of 256 columns), the matrix cores being busy for about
// half of that.  The right-hand sides, the ring's indices and the next
// phase's operands are therefore on their way ahead of their use; a third
// workgroup per unit (80 registers) gained nothing, and column blocks in turn
// in one workgroup spilled.
// Workgroup b runs on XCD b % 8: an XCD takes neighbouring subtrees, and the
// column blocks of a subtree one after another.
// LDS rows of 16 columns: z rows (separators, then the ring), then w rows
// (leaf nodes), then the outer nodes.
constexpr int SUB_T = 512, SUB_W = SUB_T / 64;
constexpr int SUB_RS = 17;                                  // LDS row: 16 columns, padded (the box goes in by nodes)
constexpr int SUB_LD = (ND_SUB * 16 + SUB_T - 1) / SUB_T;   // (node, column) pairs per thread
constexpr int SUB_LDX = (ND_SUB_EXT * 16 + SUB_T - 1) / SUB_T;
constexpr int SUB_LJ = ND_SUB_LEAVES / SUB_W;               // leaf row tiles per wavefront
constexpr int SUB_K = ND_LEAF_MAX / 4;                      // MFMA steps (of 4) of a leaf's nodes
static_assert(4 * SUB_K == ND_LEAF_MAX, "a leaf's nodes in whole steps");

// record i of a shape's table (in LDS), the same in all lanes
template <typename R>
__device__ __forceinline__ R nd_rec(const int* tab, int at, int i) {
    constexpr int W = (int)(sizeof(R) / 4);
    uint32_t v[W];
#pragma unroll
    for (int q = 0; q < W; ++q) v[q] = __builtin_amdgcn_readfirstlane(tab[at + W * i + q]);
    R r;
    __builtin_memcpy(&r, v, sizeof(R));
    return r;
}

struct SubCtx {
    NdJob d;
    NdSub s;
    NdShape h;
    const int* tab;          // the shape's tables
    int c0, conj;            // first column
};

// this thread's (node, column) pairs of the box (EXT: with its part of the
// upper separators), node fastest (grid rows are read along): f(pair, entry
// of the box table, grid node, column, whether it is one)
template <bool EXT, typename F>
__device__ __forceinline__ void nd_sub_each(const SubCtx& x, F f) {
    const int w = EXT ? x.s.ew : x.s.w, nb = w * (EXT ? x.s.eh : x.s.h);
    const float inv = 1.0f / (float)nb, invw = 1.0f / (float)w;
#pragma unroll
    for (int q = 0; q < (EXT ? SUB_LDX : SUB_LD); ++q) {
        const int p = (int)threadIdx.x + SUB_T * q, e = min(p, 16 * nb - 1);
        const int c = (int)(((float)e + 0.5f) * inv), n = e - c * nb;
        const int j = (int)(((float)n + 0.5f) * invw), i = n - j * w;
        f(q, j * x.s.ew + i, (x.s.z0 + j) * x.d.cf.nx + x.s.x0 + i, c, p == e);
    }
}
template <bool EXT, int N>
__device__ __forceinline__ void nd_sub_fetch(const SubCtx& x, double2 (&b)[N]) {
    nd_sub_each<EXT>(x, [&](int q, int, int k, int c, bool) {
        b[q] = gld(x.d.B + (size_t)min(x.c0 + c, x.d.S - 1) * x.d.ldb + k);
    });
}
// EXT: every row; else the leaves' alone
template <bool EXT, int N>
__device__ __forceinline__ void nd_sub_place(const SubCtx& x, const double2 (&b)[N], double2 (*v)[SUB_RS]) {
    const int nz = x.h.nsep + x.h.nring;
    nd_sub_each<EXT>(x, [&](int q, int n, int, int c, bool) {
        const int r = x.tab[x.h.box + n];
        if (EXT || r >= nz) v[r][c] = make_double2(b[q].x, x.conj ? -b[q].y : b[q].y);
    });
}

__device__ __forceinline__ void nd_sub_leaf_ops(const SubCtx& x, const NdLeaf& f, double2 (&g)[SUB_K]) {
    const int l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
    const double2* G = x.d.fac + x.s.fac + f.fac + min(16 * f.tile + lr, f.p - 1);
#pragma unroll
    for (int p = 0; p < SUB_K; ++p) g[p] = gld(G + min(4 * p + lg, f.p - 1) * f.p);
}

// w <- G w for every leaf: one 16-row tile of a leaf per wavefront and turn
// (its first tile's operands in g), written back once every wavefront has
// read its own operands.
__device__ __forceinline__ void nd_sub_leaves(const SubCtx& x, const double2 (&g0)[SUB_K], double2 (*wv)[SUB_RS]) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
    v4d re[SUB_LJ], im[SUB_LJ];
#pragma unroll
    for (int j = 0; j < SUB_LJ; ++j) {
        const int q = w + SUB_W * j;
        if (q >= x.h.nleaf) continue;
        const NdLeaf f = nd_rec<NdLeaf>(x.tab, x.h.leaf, q);
        double2 g[SUB_K];
        if (j > 0) nd_sub_leaf_ops(x, f, g);
        v4d p1, p2, p3;
#pragma unroll
        for (int e = 0; e < 4; ++e) { p1[e] = 0.0; p2[e] = 0.0; p3[e] = 0.0; }
#pragma unroll
        for (int p = 0; p < SUB_K; ++p)
            if (4 * p < f.p) {
                const int k = 4 * p + lg;
                const double2 b = csel_parts(k < f.p, wv[f.wrow + min(k, f.p - 1)][lr], make_double2(0.0, 0.0));
                const double2 a = j > 0 ? g[p] : g0[p];
                cmfma3<double, v4d>(p1, p2, p3, a.x, a.y, b.x, b.y);
            }
        cacc_final<true, v4d>(p1, p2, p3, re[j], im[j]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < SUB_LJ; ++j) {
        const int q = w + SUB_W * j;
        if (q >= x.h.nleaf) continue;
        const NdLeaf f = nd_rec<NdLeaf>(x.tab, x.h.leaf, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * f.tile + lg + 4 * e;
            if (i < f.p) wv[f.wrow + i][lr] = make_double2(re[j][e], im[j][e]);
        }
    }
}

// v[r] += sum over r's neighbours in `from` of coupling x value, for the rows
// that have any (eight shorts each: the row, its i, j in the box and the
// neighbours' rows, read at a valid row where there is none)
__device__ __forceinline__ void nd_sub_stencil(const SubCtx& x, int tab, int rows, double2 (*v)[SUB_RS],
                                               const double2 (*from)[SUB_RS]) {
    const double rx = x.d.cf.hz / x.d.cf.hx, rz = x.d.cf.hx / x.d.cf.hz;
    for (int q = threadIdx.x; q < 16 * rows; q += SUB_T) {
        const int* e = x.tab + tab + 4 * (q >> 4);
        const int e0 = e[0], e1 = e[1], e2 = e[2], e3 = e[3], c = q & 15;
        const int r = e0 & 0xffff, n[4] = {e1 >> 16, (int)(short)e2, e2 >> 16, (int)(short)e3};
        const double cx = rx * half_at_ends(x.s.z0 + (int)(short)e1, x.d.cf.nz);
        const double cz = rz * half_at_ends(x.s.x0 + (e0 >> 16), x.d.cf.nx);
        double2 a = v[r][c], y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = from[max(n[k], 0)][c];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double g = n[k] < 0 ? 0.0 : k < 2 ? cx : cz;
            a.x += g * (n[k] < 0 ? 0.0 : y[k].x);
            a.y += g * (n[k] < 0 ? 0.0 : y[k].y);
        }
        v[r][c] = a;
    }
}

// Which subtree and column block a workgroup takes; false: none.  The right-
// hand sides (and the ring's indices) need its record only: they are on their
// way before the shape's tables are.
__device__ __forceinline__ bool nd_sub_start(const NdTabs& t, const NdJobTab* jtab, int nsub, int nct, SubCtx& x) {
    const int b = blockIdx.x, k = b >> 3;
    const int per = (nsub + 7) >> 3, sub = (b & 7) * per + k / nct;
    if (sub >= nsub) return false;
    x.d = nd_record(jtab->j, blockIdx.y);
    x.s = nd_record(t.subs, sub);
    x.c0 = 16 * (k % nct);
    return x.c0 < x.d.S;
}
__device__ __forceinline__ void nd_sub_tables(const NdTabs& t, SubCtx& x, int* stab) {
    x.h = nd_record(t.shapes, x.s.shape);
    const int* src = t.tabs + x.h.tab0;
    for (int i = threadIdx.x; i < x.h.ntab; i += SUB_T) stab[i] = src[i];
    x.tab = stab - x.h.tab0;
}

__global__ __launch_bounds__(SUB_T, 4) void k_nd_sub_forward(NdTabs t, int nsub, int nct, int rows,
                                                             int parity, int conj, const NdJobTab* __restrict__ jtab) {
    extern __shared__ __attribute__((aligned(16))) double2 sub_smem[];
    double2 (*z)[SUB_RS] = (double2(*)[SUB_RS])sub_smem;
    SubCtx x;
    if (!nd_sub_start(t, jtab, nsub, nct, x)) return;
    x.conj = conj;
    double2 b[SUB_LDX], g[SUB_K];
    nd_sub_fetch<true>(x, b);
    nd_sub_tables(t, x, (int*)(sub_smem + SUB_RS * rows));
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, lr = l & 15, lg = l >> 4;
    const int nz = x.h.nsep + x.h.nring, S = x.d.S, c0 = x.c0;
    double2 (*wv)[SUB_RS] = z + nz;
    double2 (*u)[SUB_RS] = wv;   // ring contributions, once the leaves' results are used
    for (int q = tid; q < 16 * x.h.nring; q += SUB_T) z[x.h.nsep + (q >> 4)][q & 15] = make_double2(0.0, 0.0);
    __syncthreads();
    if (w < x.h.nleaf) nd_sub_leaf_ops(x, nd_rec<NdLeaf>(x.tab, x.h.leaf, w), g);
    const double2* sfac = x.d.fac + x.s.fac;
    nd_sub_place<true>(x, b, z);
    __syncthreads();
    // the upper rows' right-hand sides
    for (int q = tid; q < 16 * x.h.nx; q += SUB_T) {
        const int e = q >> 4, c = q & 15, k = x.tab[x.h.xring + e];
        const int row = k >= 0 ? t.ring[x.s.ring + k] : x.s.corner;
        if (c0 + c < S) gst(x.d.a + (size_t)row * S + c0 + c, z[x.h.xrow + e][c]);
    }
    nd_sub_leaves(x, g, wv);
    __syncthreads();
    double2 r[4];   // this wavefront's operands of the next level
    auto ops = [&](int step) {
        if (step >= x.h.nstep) return;
        const NdStep st = nd_rec<NdStep>(x.tab, x.h.step, step);
        if (w >= st.nfwd) return;
        const NdFwd f = nd_rec<NdFwd>(x.tab, st.fwd, w);
        const double2* R = sfac + f.fac + (f.p + min(16 * f.tile + lr, f.b - 1)) * f.p;
#pragma unroll
        for (int p = 0; p < 4; ++p) r[p] = gld(R + min(4 * p + lg, f.p - 1));
    };
    ops(0);
    nd_sub_stencil(x, x.h.zst, x.h.nzst, z, wv);
    __syncthreads();
    for (int q = 0; q < x.h.nstep; ++q) {
        const NdStep st = nd_rec<NdStep>(x.tab, x.h.step, q);
        for (int k = w; k < st.nfwd; k += SUB_W) {
            const NdFwd f = nd_rec<NdFwd>(x.tab, st.fwd, k);
            if (k != w) {
                const double2* R = sfac + f.fac + (f.p + min(16 * f.tile + lr, f.b - 1)) * f.p;
#pragma unroll
                for (int p = 0; p < 4; ++p) r[p] = gld(R + min(4 * p + lg, f.p - 1));
            }
            v4d p1, p2, p3, re, im;
#pragma unroll
            for (int e = 0; e < 4; ++e) { p1[e] = 0.0; p2[e] = 0.0; p3[e] = 0.0; }
#pragma unroll
            for (int p = 0; p < 4; ++p)
                if (4 * p < f.p) {
                    const int i = 4 * p + lg;
                    const double2 y = csel_parts(i < f.p, z[f.zp + min(i, f.p - 1)][lr], make_double2(0.0, 0.0));
                    cmfma3<double, v4d>(p1, p2, p3, r[p].x, r[p].y, y.x, y.y);
                }
            cacc_final<true, v4d>(p1, p2, p3, re, im);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 16 * f.tile + lg + 4 * e;
                if (i < f.b) u[f.u + i][lr] = make_double2(re[e], im[e]);
            }
        }
        ops(q + 1);
        __syncthreads();
        for (int k = tid; k < 16 * st.nadd; k += SUB_T) {
            const int e = x.tab[st.add + (k >> 4)], c = k & 15, r0 = e & 1023, a = (e >> 10) & 1023,
                      a2 = (e >> 20) & 1023;
            double2 v = z[r0][c];
            v.x -= u[a][c].x;
            v.y -= u[a][c].y;
            if (a2 != 1023) {
                v.x -= u[a2][c].x;
                v.y -= u[a2][c].y;
            }
            z[r0][c] = v;
        }
        __syncthreads();
    }
    double2* y = x.d.y + (size_t)x.s.row * S + c0;
    double2* uo = (parity ? x.d.u[1] : x.d.u[0]) + (size_t)x.s.urow * S + c0;
    const int nc = min(16, S - c0);
    for (int q = tid; q < 16 * nz; q += SUB_T) {
        const int r0 = q >> 4, c = q & 15;
        if (c < nc) gst(r0 < x.h.nsep ? y + (size_t)r0 * S + c : uo + (size_t)(r0 - x.h.nsep) * S + c, z[r0][c]);
    }
}

// Backward: the rings' solutions and the separators' forward results in, the
// box's solution out.  A front's contraction is shared by two wavefronts.
constexpr int SUB_BK = 9;   // MFMA steps of a wavefront's half, at most, with operands loaded ahead
__global__ __launch_bounds__(SUB_T, 4) void k_nd_sub_backward(NdTabs t, int nsub, int nct, int rows,
                                                              int conj, int add, const NdJobTab* __restrict__ jtab) {
    extern __shared__ __attribute__((aligned(16))) double2 sub_smem[];
    double2 (*z)[SUB_RS] = (double2(*)[SUB_RS])sub_smem;
    double2 (*part)[16][16] = (double2(*)[16][16])(sub_smem + SUB_RS * rows);   // second halves' sums
    SubCtx x;
    if (!nd_sub_start(t, jtab, nsub, nct, x)) return;
    x.conj = conj;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, lr = l & 15, lg = l >> 4;
    const int S = x.d.S, c0 = x.c0, half = w & 1;
    double2 b[SUB_LD], zr[4];
    const double2 corner = gld(x.d.a + (size_t)max(x.s.corner, 0) * S + min(c0 + (tid & 15), S - 1));
    // separator and ring rows, by 16 columns, up to four per thread ahead
    const double2* zp[4];
    const int nz = x.s.nsep + x.s.nring;
    auto zrow = [&](int q) {
        const int r = q >> 4, c = min(c0 + (q & 15), S - 1);
        return r < x.s.nsep ? x.d.y + (size_t)(x.s.row + r) * S + c
                            : x.d.a + (size_t)t.ring[x.s.ring + r - x.s.nsep] * S + c;
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) zp[i] = zrow(min(tid + SUB_T * i, 16 * nz - 1));
#pragma unroll
    for (int i = 0; i < 4; ++i) zr[i] = gld(zp[i]);
    nd_sub_fetch<false>(x, b);
    nd_sub_tables(t, x, (int*)(part + SUB_W / 2));
    double2 (*wv)[SUB_RS] = z + nz;
    const double2* sfac = x.d.fac + x.s.fac;
    __syncthreads();
    // operands of steps s0 .. of a front's contraction, in fours: the pivots
    // (4 of them), then the ring; a level's first are loaded a level ahead
    double2 m[SUB_BK];
    auto steps = [&](const NdBwd& f) { return 4 + ((f.b + 3) >> 2); };
    auto ops = [&](const NdBwd& f, int s0, int hi) {
        const double2* M = sfac + f.fac + min(lr, f.p - 1);
#pragma unroll
        for (int p = 0; p < SUB_BK; ++p) {
            const int s = min(s0 + p, hi - 1), i = 4 * s + lg;
            m[p] = gld(M + (s < 4 ? min(i, f.p - 1) : f.p + min(i - 16, f.b - 1)) * f.p);
        }
    };
    auto first = [&](int q) {
        if (q < 0) return;
        const NdStep st = nd_rec<NdStep>(x.tab, x.h.step, q);
        if ((w >> 1) >= st.nbwd) return;
        const NdBwd f = nd_rec<NdBwd>(x.tab, st.bwd, w >> 1);
        const int n = steps(f);
        ops(f, half ? (n + 1) / 2 : 0, half ? n : (n + 1) / 2);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (tid + SUB_T * i < 16 * nz) z[(tid + SUB_T * i) >> 4][tid & 15] = zr[i];
    for (int q = tid + 4 * SUB_T; q < 16 * nz; q += SUB_T) z[q >> 4][q & 15] = gld(zrow(q));
    first(x.h.nstep - 1);
    nd_sub_place<false>(x, b, z);
    __syncthreads();
    for (int q = x.h.nstep - 1; q >= 0; --q) {
        const NdStep st = nd_rec<NdStep>(x.tab, x.h.step, q);
        for (int k0 = 0; k0 < st.nbwd; k0 += SUB_W / 2) {
            const int k = k0 + (w >> 1);
            v4d p1, p2, p3, re, im;
#pragma unroll
            for (int e = 0; e < 4; ++e) { p1[e] = 0.0; p2[e] = 0.0; p3[e] = 0.0; }
            const NdBwd f = nd_rec<NdBwd>(x.tab, st.bwd, min(k, st.nbwd - 1));
            const int n = steps(f), hi = half ? n : (n + 1) / 2;
            if (k < st.nbwd)
                for (int s0 = half ? (n + 1) / 2 : 0; s0 < hi; s0 += SUB_BK) {
                    if (k0 || s0 != (half ? (n + 1) / 2 : 0)) ops(f, s0, hi);
#pragma unroll
                    for (int p = 0; p < SUB_BK; ++p) {
                        const int s = s0 + p, i = 4 * s + lg;
                        if (s >= hi || (s < 4 && 4 * s >= f.p)) continue;
                        const bool piv = s < 4, in = piv ? i < f.p : i - 16 < f.b;
                        const double2 v = z[piv ? f.zp + min(i, f.p - 1) : x.tab[f.ring + min(i - 16, f.b - 1)]][lr];
                        const double sg = in ? (piv ? 1.0 : -1.0) : 0.0;
                        cmfma3<double, v4d>(p1, p2, p3, m[p].x, m[p].y, sg * v.x, sg * v.y);
                    }
                }
            if (k0 + SUB_W / 2 >= st.nbwd) first(q - 1);
            cacc_final<true, v4d>(p1, p2, p3, re, im);
            if (half && k < st.nbwd) {
#pragma unroll
                for (int e = 0; e < 4; ++e) part[w >> 1][lg + 4 * e][lr] = make_double2(re[e], im[e]);
            }
            __syncthreads();
            if (!half && k < st.nbwd) {   // x overwrites y in place
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = lg + 4 * e;
                    const double2 o = part[w >> 1][i][lr];
                    if (i < f.p) z[f.zp + i][lr] = make_double2(re[e] + o.x, im[e] + o.y);
                }
            }
            __syncthreads();
        }
    }
    double2 g[SUB_K];
    if (w < x.h.nleaf) nd_sub_leaf_ops(x, nd_rec<NdLeaf>(x.tab, x.h.leaf, w), g);
    if (tid < 16) z[x.h.xrow][tid] = corner;   // may lie in the sums' room, which is free now
    nd_sub_stencil(x, x.h.wst, x.h.nwst, wv, z);
    __syncthreads();
    nd_sub_leaves(x, g, wv);
    __syncthreads();
    const int nc = min(16, S - c0);
    nd_sub_each<true>(x, [&](int, int n, int k, int c, bool own) {
        int r = x.tab[x.h.box + n];
        if (r >= x.h.xrow) r = x.tab[x.h.xback + r - x.h.xrow];
        double2 v = z[r][c];
        if (conj) v.y = -v.y;
        if (c < nc && own) nd_put_x(x.d.X + (size_t)(c0 + c) * x.d.ldx + k, v, add);
    });
}

// -------------------------------------------------- levels above the subtrees --
// Forward (401^2, 5 systems, 64 columns: 26 to 130 us a level, latency of the
// gathers; one level of one system 6 us).
// A workgroup takes RT 16-row tiles of a front's product for 16 columns; its
// 4 / RT wavefronts per tile share the contraction and are summed in order.
// The operand vectors, gathered from several places, are staged through LDS
// 32 or 64 rows at a time for all of them (each wavefront gathering its own took
// 3 x as long: three loads and two index loads per value).  The next rows
// are loaded while these are multiplied.  A front without a ring (the root)
// only has y to write, 64 rows per workgroup.  RT is a property of the level
// (launchers below), so that no result depends on what else is in a launch.
constexpr int ROOT_CH = 64;

template <int RT>
__device__ __forceinline__ void nd_reduce(v4d& re, v4d& im, double (*red)[2][4][64]) {
    constexpr int KS = 4 / RT;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, rt = w % RT, ks = w / RT;
    if (KS == 1) return;
    __syncthreads();
    if (ks) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { red[w - RT][0][e][l] = re[e]; red[w - RT][1][e][l] = im[e]; }
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
        for (int q = 0; q < KS - 1; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) { re[e] += red[rt + RT * q][0][e][l]; im[e] += red[rt + RT * q][1][e][l]; }
    }
}

// Workgroup b runs on XCD b % 8: an XCD takes a contiguous range of a level's
// tiles (neighbouring fronts, which read the same rows), and the column
// blocks of a tile one after another (they read the same part of the factor).
__device__ __forceinline__ bool nd_place(int rows, int nct, int& row, int& col) {
    const int b = blockIdx.x, k = b >> 3, per = (rows + 7) >> 3;
    row = (b & 7) * per + k / nct;
    col = k % nct;
    return row < rows && row < ((b & 7) + 1) * per;
}

template <int RT>
__global__ __launch_bounds__(256, 4) void k_nd_forward(NdTabs t, int first, int row0, int rows, int nct, int parity,
                                                    const NdJobTab* __restrict__ jtab) {
    constexpr int KS = 4 / RT, CH = RT == 4 ? 32 : 64;   // staged rows
    __shared__ double2 sy[2][CH][16];
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, lr = l & 15, lg = l >> 4;
    int e0, cb;
    if (!nd_place(rows, nct, e0, cb)) return;
    const NdJob d = nd_record(jtab->j, blockIdx.y);
    const int c0 = 16 * cb, S = d.S;
    if (c0 >= S) return;
    const NdTile tl = nd_record(t.tiles, row0 + e0);
    const NdFront f = nd_record(t.fronts, first + tl.front);
    const int c16 = min(c0 + lr, S - 1);
    const bool on = c0 + lr < S;
    const double2* uin = parity ? d.u[0] : d.u[1];
    double2* uout = parity ? d.u[1] : d.u[0];
    const double2* u0 = uin + (size_t)f.curow[0] * S;
    const double2* u1 = uin + (size_t)f.curow[1] * S;
    const int* m0 = t.map + f.map[0];
    const int* m1 = t.map + f.map[1];
    // children's contributions at local index i, column c
    auto passed = [&](int i, int c) {
        const int a = m0[i], b = m1[i];
        const double2 va = gld(u0 + (size_t)max(a, 0) * S + c), vb = gld(u1 + (size_t)max(b, 0) * S + c);
        return make_double2((a >= 0 ? va.x : 0.0) + (b >= 0 ? vb.x : 0.0), (a >= 0 ? va.y : 0.0) + (b >= 0 ? vb.y : 0.0));
    };
    // staging: thread -> rows (tid / 16) + 16 i, column tid % 16
    const int sr = tid >> 4;
    const int kb = f.b ? 0 : ROOT_CH * tl.ti, ke = f.b ? f.p : min(kb + ROOT_CH, f.p);
    double2 v[CH / 16];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < CH / 16; ++i) {
            if (k0 + 16 * i >= ke) continue;
            const int k = k0 + sr + 16 * i, kc = min(k, ke - 1);
            const double2 b = gld(d.a + (size_t)(f.piv0 + kc) * S + c16), q = passed(kc, c16);
            v[i] = csel_parts(k < ke, make_double2(b.x + q.x, b.y + q.y), make_double2(0.0, 0.0));
        }
    };
    load(kb);
    const int rt = w % RT, ks = w / RT, i0 = 16 * (tl.ti + rt);
    const bool mine = i0 < f.b;
    double2 pre[4];
    if (mine && ks == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) pre[e] = passed(f.p + min(i0 + lg + 4 * e, f.b - 1), c16);
    }
    const double2* R = d.fac + f.fac + (int64_t)(f.p + min(i0 + lr, max(f.b - 1, 0))) * f.p;
    v4d re, im;
#pragma unroll
    for (int e = 0; e < 4; ++e) { re[e] = 0.0; im[e] = 0.0; }
    for (int k0 = kb, c = 0; k0 < ke; k0 += CH, c ^= 1) {
        double2 g[CH / 16 / KS][4];
        if (mine) {
#pragma unroll
            for (int j = 0; j < CH / 16 / KS; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) g[j][q] = gld(R + min(k0 + 16 * (ks + KS * j) + 4 * lg + q, f.p - 1));
        }
#pragma unroll
        for (int i = 0; i < CH / 16; ++i) {
            if (k0 + 16 * i >= ke) continue;
            sy[c][sr + 16 * i][lr] = v[i];
            if ((tl.ti == 0 || f.b == 0) && on && k0 + sr + 16 * i < ke)
                gst(d.y + (size_t)(f.piv0 + k0 + sr + 16 * i) * S + c16, v[i]);
        }
        __syncthreads();
        if (k0 + CH < ke) load(k0 + CH);
        if (mine) {
#pragma unroll
            for (int j = 0; j < CH / 16 / KS; ++j) {
                const int kt = 16 * (ks + KS * j);
                if (k0 + kt >= f.p) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double2 x = sy[c][kt + 4 * lg + q][lr];
                    cmfma<double, v4d>(re, im, g[j][q].x, g[j][q].y, x.x, x.y);
                }
            }
        }
    }
    nd_reduce<RT>(re, im, (double(*)[2][4][64])&sy[0][0][0]);
    if (!mine || ks) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = i0 + lg + 4 * e;
        if (i < f.b && on) gst(uout + (size_t)(f.urow + i) * S + c16, make_double2(pre[e].x - re[e], pre[e].y - im[e]));
    }
}

// Backward: x = G y - R x_ring, one 16-row tile of a front for 16 columns,
// by a wavefront (SPLIT: by four that share the contraction).  The operands
// are read straight from L2: their rows are whole, one load each, and staging
// them in LDS for several tiles was slower at every level (401^2, 64 columns,
// 5 systems: levels of 19 to 80 us against 28 to 90 us).
template <bool SPLIT>
__global__ __launch_bounds__(256) void k_nd_backward(NdTabs t, int first, int row0, int rows, int nct,
                                                     const NdJobTab* __restrict__ jtab) {
    __shared__ double red[SPLIT ? 3 : 1][2][4][64];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
    int e0, cb;
    if (!nd_place(SPLIT ? rows : (rows + 3) >> 2, nct, e0, cb)) return;
    if (!SPLIT) e0 = 4 * e0 + w;
    const NdJob d = nd_record(jtab->j, blockIdx.y);
    const int c0 = 16 * cb, S = d.S;
    if (c0 >= S || e0 >= rows) return;
    const NdTile tl = nd_record(t.tiles, row0 + e0);
    const NdFront f = nd_record(t.fronts, first + tl.front);
    const int col = min(c0 + lr, S - 1), i0 = 16 * tl.ti;
    const bool on = c0 + lr < S;
    const double2* M = d.fac + f.fac + min(i0 + lr, f.p - 1);
    const double2* yv = d.y + (size_t)f.piv0 * S + col;
    const int* ring = t.ring + f.ring;
    const int pt = (f.p + 15) >> 4, nk = pt + ((f.b + 15) >> 4);
    const int kb = SPLIT ? w * nk / 4 : 0, ke = SPLIT ? (w + 1) * nk / 4 : nk;
    v4d p1, p2, p3, re, im;
#pragma unroll
    for (int e = 0; e < 4; ++e) { p1[e] = 0.0; p2[e] = 0.0; p3[e] = 0.0; }
    for (int kt = kb; kt < ke; ++kt) {
        double2 g[4], v[4];
        if (kt < pt) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = 16 * kt + 4 * lg + q, kc = min(k, f.p - 1);
                g[q] = gld(M + (int64_t)kc * f.p);
                v[q] = csel_parts(k < f.p, gld(yv + (size_t)kc * S), make_double2(0.0, 0.0));
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = 16 * (kt - pt) + 4 * lg + q, kc = min(k, f.b - 1);
                g[q] = gld(M + (int64_t)(f.p + kc) * f.p);
                const double2 x = gld(d.a + (size_t)ring[kc] * S + col);
                v[q] = csel_parts(k < f.b, make_double2(-x.x, -x.y), make_double2(0.0, 0.0));
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) cmfma3<double, v4d>(p1, p2, p3, g[q].x, g[q].y, v[q].x, v[q].y);
    }
    cacc_final<true, v4d>(p1, p2, p3, re, im);
    if (SPLIT) {
        if (w) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { red[w - 1][0][e][l] = re[e]; red[w - 1][1][e][l] = im[e]; }
        }
        __syncthreads();
        if (w) return;
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) { re[e] += red[q][0][e][l]; im[e] += red[q][1][e][l]; }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = i0 + lg + 4 * e;
        if (i < f.p && on) gst(d.a + (size_t)(f.piv0 + i) * S + col, make_double2(re[e], im[e]));
    }
}

// ------------------------------------------------------------------ launchers --
template <typename Tab>
__global__ __launch_bounds__(256) void k_nd_put(const Tab src, Tab* dst) {
    static_assert(sizeof(Tab) % 4 == 0, "tables are whole dwords");
    const uint32_t* s = (const uint32_t*)&src;
    for (int i = threadIdx.x; i < (int)(sizeof(Tab) / 4); i += 256) ((uint32_t*)dst)[i] = s[i];
}
void launch_nd_put_sys(const NdSysTab& tab, NdSysTab* dst, hipStream_t st) {
    hipLaunchKernelGGL(k_nd_put<NdSysTab>, dim3(1), dim3(256), 0, st, tab, dst);
}
void launch_nd_put_jobs(const NdJobTab& tab, NdJobTab* dst, hipStream_t st) {
    hipLaunchKernelGGL(k_nd_put<NdJobTab>, dim3(1), dim3(256), 0, st, tab, dst);
}

// LDS of k_nd_front<KP> for a level's widest front
size_t nd_front_lds(int kp, int fmax) {
    return sizeof(double2) * ((size_t)(kp == 16 ? 16 : 64) * 33 + (size_t)(fmax - 16) * (kp + 1)) +
           sizeof(NdIndex) * (size_t)fmax + sizeof(NdScratch);
}
bool nd_narrow(int pmax, int fmax) { return pmax <= 32 && nd_front_lds(pmax <= 16 ? 16 : 32, fmax) <= ND_LDS; }

// More than 64 KB of LDS is asked for by the kernel's attribute, always for
// the most that any launch takes, so that no thread lowers it under another's
// launch.
static hipError_t nd_allow_lds(const void* kernel, size_t lds) {
    if (lds > ND_LDS) return hipErrorInvalidValue;
    return lds > 65536 ? hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ND_LDS) : hipSuccess;
}

template <int KP>
static hipError_t launch_nd_front(const NdTabs& t, const NdLevel& lv, const NdSysTab* dsys, int n, hipStream_t st) {
    const size_t lds = nd_front_lds(KP, lv.fmax);
    const hipError_t e = nd_allow_lds((const void*)k_nd_front<KP>, lds);
    if (e == hipSuccess)
        hipLaunchKernelGGL(k_nd_front<KP>, dim3(lv.count, n), dim3(KP == 16 ? 256 : 512), lds, st, t, lv.first,
                           lv.parity, lv.fmax, dsys);
    return e;
}

hipError_t launch_nd_level(const NdTabs& t, const NdLevel& lv, const NdSysTab* dsys, int n, hipStream_t st, int64_t* launches) {
    *launches += 1;
    if (lv.leaf) {
        hipLaunchKernelGGL(k_nd_leaf, dim3(lv.count, n), dim3(64), 0, st, t, lv.first, dsys);
        return hipSuccess;
    }
    if (lv.small) return lv.pmax <= 16 ? launch_nd_front<16>(t, lv, dsys, n, st) : launch_nd_front<32>(t, lv, dsys, n, st);
    const dim3 grid(lv.count + lv.tiles, n);
    hipLaunchKernelGGL(k_nd_gather, grid, dim3(256), 0, st, t, lv.first, lv.count, lv.tile0, lv.parity, dsys);
    for (int s = 0; s < lv.npan; ++s)
        hipLaunchKernelGGL(k_nd_step, grid, dim3(256), 0, st, t, lv.first, lv.count, lv.tile0, lv.parity, s, dsys);
    if (lv.stiles)
        hipLaunchKernelGGL(k_nd_schur, dim3(lv.stiles, n), dim3(256), 0, st, t, lv.first, lv.stile0, lv.parity, dsys);
    *launches += lv.npan + (lv.stiles ? 1 : 0);
    return hipSuccess;
}

size_t nd_sub_forward_lds(const NdPlan& p) { return (size_t)p.sub_rows * SUB_RS * 16 + 4 * (size_t)p.sub_tab; }
size_t nd_sub_backward_lds(const NdPlan& p) {
    return (size_t)p.sub_brows * SUB_RS * 16 + SUB_W / 2 * 4096 + 4 * (size_t)p.sub_tab;
}
static dim3 nd_sub_grid(const NdPlan& p, int nct, int n) { return dim3(8 * ((p.nsub + 7) / 8) * nct, n); }
hipError_t launch_nd_sub_forward(const NdTabs& t, const NdPlan& p, const NdJobTab* djobs, int n, int smax, bool conj,
                           hipStream_t st) {
    const int nct = (smax + 15) / 16;
    const size_t lds = nd_sub_forward_lds(p);
    const hipError_t e = nd_allow_lds((const void*)k_nd_sub_forward, lds);
    if (e == hipSuccess)
        hipLaunchKernelGGL(k_nd_sub_forward, nd_sub_grid(p, nct, n), dim3(SUB_T), lds, st, t, p.nsub, nct, p.sub_rows,
                           p.sub_parity, conj ? 1 : 0, djobs);
    return e;
}
hipError_t launch_nd_sub_backward(const NdTabs& t, const NdPlan& p, const NdJobTab* djobs, int n, int smax, bool add,
                            bool conj, hipStream_t st) {
    const int nct = (smax + 15) / 16;
    const size_t lds = nd_sub_backward_lds(p);
    const hipError_t e = nd_allow_lds((const void*)k_nd_sub_backward, lds);
    if (e == hipSuccess)
        hipLaunchKernelGGL(k_nd_sub_backward, nd_sub_grid(p, nct, n), dim3(SUB_T), lds, st, t, p.nsub, nct, p.sub_brows,
                           conj ? 1 : 0, add ? 1 : 0, djobs);
    return e;
}

void launch_nd_forward(const NdTabs& t, const NdLevel& lv, const NdJobTab* djobs, int n, int smax, hipStream_t st) {
    const int nct = (smax + 15) / 16;
    const dim3 grid(8 * ((lv.frows + 7) / 8) * nct, n);
#define HELM_ND(RT) hipLaunchKernelGGL(k_nd_forward<RT>, grid, dim3(256), 0, st, t, lv.first, lv.frow0, lv.frows, nct, lv.parity, djobs)
    if (lv.frt == 4) HELM_ND(4);
    else HELM_ND(1);
#undef HELM_ND
}
void launch_nd_backward(const NdTabs& t, const NdLevel& lv, const NdJobTab* djobs, int n, int smax, hipStream_t st) {
    const int nct = (smax + 15) / 16;
    // four wavefronts to a row tile where the contraction is long enough: in
    // us, split against not, fronts above 96 rows 17 .. 69 / 30 .. 70 (401^2, 5
    // systems), 5 / 8 .. 12 (101^2); below 57 / 47 and 5 / 7
    if (lv.fmax > 96)
        hipLaunchKernelGGL(k_nd_backward<true>, dim3(8 * ((lv.brows + 7) / 8) * nct, n), dim3(256), 0, st, t, lv.first,
                           lv.brow0, lv.brows, nct, djobs);
    else
        hipLaunchKernelGGL(k_nd_backward<false>, dim3(8 * (((lv.brows + 3) / 4 + 7) / 8) * nct, n), dim3(256), 0, st, t,
                           lv.first, lv.brow0, lv.brows, nct, djobs);
}

}  // namespace helm
