// Inverses of the 16 x 16 and 32 x 32 diagonal tiles, shared by the block
// factorisation (helm_factor.hip) and the nested-dissection one
// (helm_nd.hip): device code only.
#pragma once
#include "helm_device.h"

namespace helm {

// --------------------------------------------------- diagonal-tile inverse --
// Gauss-Jordan inversion of a kb x kb tile (kb = 16 or 32) by 256 threads:
// thread t holds row r = t/8 (wave w = t/64 holds rows 8w..8w+7) and columns
// 4(t%8) .. 4(t%8)+3.  Partial pivoting over the unused rows of the tile.
// Each wave nominates its best candidate row for the next column (key =
// magnitude bits with the row index in the low bits, reduced with DPP) and
// publishes it with the row's values; one barrier per pivot.  Rows are not
// moved: the pivot of column p sits in row rowOf[p], and the inverse is
// T[i][c] = M[rowOf[i]][stepOf[c]].

template <typename T>
struct GJScratch {
    uint32_t key[2][4];
    typename CT<T>::c row[2][4][32];
    int rowOf[32];
    int stepOf[32];
};

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // quad [1,0,3,2]
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // quad [2,3,0,1]
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // row half-mirror
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // row mirror
    const uint32_t a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
    const uint32_t c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(c, d));
}

// value held by lane (l & ~7) | src within each group of 32 lanes
template <int SRC>
__device__ __forceinline__ int swz_row(int v) {
    return __builtin_amdgcn_ds_swizzle(v, 0x18 | (SRC << 5));
}
template <int SRC>
__device__ __forceinline__ double swz_row(double v) {
    const int lo = swz_row<SRC>(__double2loint(v)), hi = swz_row<SRC>(__double2hiint(v));
    return __hiloint2double(hi, lo);
}
template <int SRC>
__device__ __forceinline__ float swz_row(float v) {
    return __int_as_float(swz_row<SRC>(__float_as_int(v)));
}
template <typename T>
__device__ __forceinline__ typename CT<T>::c swz_row_c(typename CT<T>::c v, int src) {
    using C = typename CT<T>::c;
    C r;
    switch (src) {
#define HELM_SWZ(k) case k: r.x = swz_row<k>(v.x); r.y = swz_row<k>(v.y); break;
        HELM_SWZ(0) HELM_SWZ(1) HELM_SWZ(2) HELM_SWZ(3) HELM_SWZ(4) HELM_SWZ(5) HELM_SWZ(6)
        default: r.x = swz_row<7>(v.x); r.y = swz_row<7>(v.y); break;
#undef HELM_SWZ
    }
    return r;
}

// 1 / n, refined by Newton steps
__device__ __forceinline__ double rcp_refined(double n) {
    double y = __builtin_amdgcn_rcp(n);
    y = y * (2.0 - n * y);
    return y * (2.0 - n * y);
}
__device__ __forceinline__ float rcp_refined(float n) {
    const float y = __builtin_amdgcn_rcpf(n);
    return y * (2.0f - n * y);
}
// 1 / p for complex p
template <typename C>
__device__ __forceinline__ C crcp(C p) {
    const auto y = rcp_refined(p.x * p.x + p.y * p.y);
    return mk<C>(p.x * y, -p.y * y);
}

template <typename T>
__device__ __forceinline__ uint32_t pivot_key(typename CT<T>::c v, int r, bool cand) {
    if (!cand) return 0u;
    const float mag = (float)(v.x * v.x + v.y * v.y);
    return (__float_as_uint(mag) & ~0x3Fu) | 0x20u | (uint32_t)(31 - r);
}

// Inverts the tile held in a[] (layout above); on return a[] holds M and
// sh.rowOf / sh.stepOf the pivot order (valid after a barrier).  Returns the
// first pivot step whose candidates were all zero, or -1.
template <typename T, int KBT>
__device__ __forceinline__ int gj_invert(typename CT<T>::c (&a)[4], GJScratch<T>& sh) {
    using C = typename CT<T>::c;
    constexpr int NW = KBT / 8;
    const int t = threadIdx.x, w = t >> 6, l = t & 63;
    const int r = t >> 3, cg = t & 7;
    const bool act = (r < KBT) && (4 * cg < KBT);
    uint32_t used = 0u;
    int zero = -1;
    {
        const uint32_t k = pivot_key<T>(a[0], r, act && cg == 0);
        const uint32_t wk = wave_max_u32(k);
        if (w < NW) {
            if (act && wk != 0u && r == 31 - (int)(wk & 31u)) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sh.row[0][w][4 * cg + e] = a[e];
            }
            if (l == 0) sh.key[0][w] = wk;
        }
    }
#pragma unroll
    for (int p = 0; p < KBT; ++p) {
        const int par = p & 1;
        const int pc = p >> 2, pe = p & 3;
        __syncthreads();
        uint32_t best = sh.key[par][0];
        int wb = 0;
#pragma unroll
        for (int q = 1; q < NW; ++q) {
            const uint32_t kq = sh.key[par][q];
            if (kq > best) { best = kq; wb = q; }
        }
        const int rp = 31 - (int)(best & 31u);
        const bool good = (best >> 6) != 0u;
        if (!good && zero < 0) zero = p;
        const C piv = sh.row[par][wb][p];
        C pr[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) pr[e] = sh.row[par][wb][4 * cg + e];
        const C f = swz_row_c<T>(a[pe], pc);
        const C dv = HELM_CSEL(good, crcp(piv), mk<C>(0.0, 0.0));
        if (act) {
            if (r == rp) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = (4 * cg + e == p) ? dv : cmul(pr[e], dv);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (4 * cg + e == p) {
                        a[e] = mk<C>(-(f.x * dv.x - f.y * dv.y), -(f.x * dv.y + f.y * dv.x));
                    } else {
                        const C s = cmul(pr[e], dv);
                        a[e] = mk<C>(a[e].x - (f.x * s.x - f.y * s.y), a[e].y - (f.x * s.y + f.y * s.x));
                    }
                }
            }
        }
        used |= 1u << rp;
        if (t == 0) { sh.rowOf[p] = rp; sh.stepOf[rp] = p; }
        if (p + 1 < KBT) {
            const int pc1 = (p + 1) >> 2, pe1 = (p + 1) & 3;
            const uint32_t k = pivot_key<T>(a[pe1], r, act && cg == pc1 && !((used >> r) & 1u));
            const uint32_t wk = wave_max_u32(k);
            if (w < NW) {
                if (act && wk != 0u && r == 31 - (int)(wk & 31u)) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sh.row[par ^ 1][w][4 * cg + e] = a[e];
                }
                if (l == 0) sh.key[par ^ 1][w] = wk;
            }
        }
    }
    return zero;
}

// Scratch of the unpivoted inverses: the tile maximum of each wavefront and
// the small-pivot flag.
template <typename T>
struct RowScratch {
    float amax[4];
    int small;
};

// ------------------------------------------------ blocked unpivoted inverse --
// The diagonal tile [[A, B], [C, D]] (16 x 16 quadrants) is inverted as
//     A^-1,  X = A^-1 B,  Y = C A^-1,  S = D - C X,  S^-1,
//     T12 = -X S^-1,  T21 = -S^-1 Y,  T22 = S^-1,  T11 = A^-1 - X T21,
// which is unpivoted Gauss-Jordan on the whole tile with its pivots taken in
// the same order (those of A, then those of S), so the small-pivot test is
// the same one.  This is a serial chain and bounds a panel step, so it stays
// in one wavefront's registers as far as it goes: lane l = 16 g + r holds row
// r and columns acc_row(g, e) of A, which after the inversion is the first
// operand of the matrix-core product X = A^-1 B; X comes out as the second
// operand of C X; and S comes out as the rows of S^T, whose inverse is
// (S^-1)^T, again an operand.  A second wavefront forms Y beside it and T21,
// T11 after it.
template <typename C> __device__ __forceinline__ C lane_read(C v, int lane);
template <> __device__ __forceinline__ float2 lane_read(float2 v, int lane) {
    float2 r;
    r.x = __int_as_float(__builtin_amdgcn_ds_bpermute(lane << 2, __float_as_int(v.x)));
    r.y = __int_as_float(__builtin_amdgcn_ds_bpermute(lane << 2, __float_as_int(v.y)));
    return r;
}
template <> __device__ __forceinline__ double2 lane_read(double2 v, int lane) {
    const int a = lane << 2;
    const int xl = __builtin_amdgcn_ds_bpermute(a, __double2loint(v.x));
    const int xh = __builtin_amdgcn_ds_bpermute(a, __double2hiint(v.x));
    const int yl = __builtin_amdgcn_ds_bpermute(a, __double2loint(v.y));
    const int yh = __builtin_amdgcn_ds_bpermute(a, __double2hiint(v.y));
    return make_double2(__hiloint2double(xh, xl), __hiloint2double(yh, yl));
}
// the value of lane `lane` in every lane (lane is wave-uniform)
template <typename C> __device__ __forceinline__ C lane_bcast(C v, int lane);
template <> __device__ __forceinline__ float2 lane_bcast(float2 v, int lane) {
    return make_float2(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v.x), lane)),
                       __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v.y), lane)));
}
template <> __device__ __forceinline__ double2 lane_bcast(double2 v, int lane) {
    const int xl = __builtin_amdgcn_readlane(__double2loint(v.x), lane);
    const int xh = __builtin_amdgcn_readlane(__double2hiint(v.x), lane);
    const int yl = __builtin_amdgcn_readlane(__double2loint(v.y), lane);
    const int yh = __builtin_amdgcn_readlane(__double2hiint(v.y), lane);
    return make_double2(__hiloint2double(xh, xl), __hiloint2double(yh, yl));
}

// the value of lane P of each row of 16 lanes, in every lane of that row
// (DPP row broadcast, complex128 halves whole; P compile-time)
template <int P> __device__ __forceinline__ float row_bcast_p(float v) {
    return __builtin_amdgcn_update_dpp(v, v, 0x150 + P, 0xF, 0xF, true);
}
template <int P> __device__ __forceinline__ double row_bcast_p(double v) {
    return __builtin_amdgcn_update_dpp(v, v, 0x150 + P, 0xF, 0xF, true);
}
template <int P, typename C> __device__ __forceinline__ C row_bcast(C v) {
    return mk<C>(row_bcast_p<P>(v.x), row_bcast_p<P>(v.y));
}

// One pivot of gj16_wave (below): piv is a_pp and y = 1 / |a_pp|^2 on entry,
// those of the next pivot on return.
template <typename T, int P>
__device__ __forceinline__ void gj16_pivot(typename CT<T>::c (&a)[4], typename CT<T>::c& piv, T& y, float thr,
                                           bool& small, int r, int g) {
    using C = typename CT<T>::c;
    // place of column P and P + 1: lane group, entry
    constexpr bool F64 = sizeof(T) == 8;
    constexpr int GP = F64 ? P & 3 : P >> 2, EP = F64 ? P >> 2 : P & 3;
    constexpr int N = P + 1, GN = F64 ? N & 3 : N >> 2, EN = F64 ? (N >> 2) & 3 : N & 3;
    C f = lane_read(a[EP], r + 16 * GP);                   // a[r][p], from another row of lanes
    C pr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) pr[e] = row_bcast<P>(a[e]);   // a[p][..], lane p of this row of lanes
    if (r == P) f.x -= (T)1;
    // (f / a_pp) from f conj(a_pp), which does not wait for the reciprocal
    const C fs = mk<C>((f.x * piv.x + f.y * piv.y) * y, (f.y * piv.x - f.x * piv.y) * y);
    auto update = [&](int e) {
        const C up = mk<C>(fma(-fs.x, pr[e].x, fma(fs.y, pr[e].y, a[e].x)),
                           fma(-fs.x, pr[e].y, fma(-fs.y, pr[e].x, a[e].y)));
        if (e == EP) a[e] = HELM_CSEL(g == GP, mk<C>((r == P ? (T)1 : (T)0) - fs.x, -fs.y), up);
        else a[e] = up;
    };
    // the next pivot's entry first: its reciprocal is the serial part
    update(EN);
    if (P < 15) {
        piv = lane_bcast(a[EN], N + 16 * GN);
        const T n = piv.x * piv.x + piv.y * piv.y;
        if (!((float)n >= thr)) small = true;
        y = rcp_refined(n);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (e != EN) update(e);
}

// Unpivoted Gauss-Jordan of a 16 x 16 tile held by one wavefront (lane
// 16 g + r: row r, columns acc_row(g, e)), in a uniform form with no special
// case for the pivot row: for pivot p, with f = (column p) - e_p and
// d = 1 / a_pp, every entry off column p takes a_ij -= (f_i d) a_pj, and
// column p becomes e_p - f d, which leaves the inverse in place.  Every lane
// reads the old pivot row at its columns and its row's entry of column p from
// the lanes that hold them (the row by a DPP broadcast within each row of 16
// lanes, the column entry by a cross-lane read).  Sets small if
// |a_pp|^2 < thr for some pivot.
template <typename T>
__device__ __forceinline__ void gj16_wave(typename CT<T>::c (&a)[4], float thr, bool& small) {
    using C = typename CT<T>::c;
    const int l = threadIdx.x & 63, r = l & 15, g = l >> 4;
    C piv = lane_bcast(a[0], 0);
    const T n = piv.x * piv.x + piv.y * piv.y;
    if (!((float)n >= thr)) small = true;
    T y = rcp_refined(n);
    gj16_pivot<T, 0>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 1>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 2>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 3>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 4>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 5>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 6>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 7>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 8>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 9>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 10>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 11>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 12>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 13>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 14>(a, piv, y, thr, small, r, g);
    gj16_pivot<T, 15>(a, piv, y, thr, small, r, g);
}

// One wavefront's part of a 16 x 16 complex product on the matrix cores:
// d = c0 + sign A B (the product by itself, then one addition: accumulated onto
// c0 every step rounds at its size, and complex64 solutions of 30 x 60 grids
// were 1.7 times as far off), with A read by rows from LDS (stride 33) or from
// registers (a[e] = A[lr][acc_row(lg, e)]), B from LDS or from registers
// (b[e] = B[acc_row(lg, e)][lr]); results as b is.
template <typename T>
__device__ __forceinline__ void row_ops(const typename CT<T>::c* A, typename CT<T>::c (&a)[4]) {
    const int l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = A[lr * 33 + acc_row<T>(lg, e)];
}
template <typename T>
__device__ __forceinline__ void col_ops(const typename CT<T>::c* B, typename CT<T>::c (&b)[4]) {
    const int l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = B[acc_row<T>(lg, e) * 33 + lr];
}
template <typename T>
__device__ __forceinline__ void col_put(typename CT<T>::c* D, const typename CT<T>::c (&d)[4]) {
    const int l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) D[acc_row<T>(lg, e) * 33 + lr] = d[e];
}
template <typename T>
__device__ __forceinline__ void mm16(const typename CT<T>::c (&a)[4], const typename CT<T>::c (&b)[4],
                                     const typename CT<T>::c (&c0)[4], T sign, typename CT<T>::c (&d)[4]) {
    using C = typename CT<T>::c;
    using V = typename CT<T>::v4;
    constexpr bool GAUSS = sizeof(T) == 8;   // three real products per complex one in complex128
    V re, im, a1, a2, a3;
#pragma unroll
    for (int e = 0; e < 4; ++e) { a1[e] = 0; a2[e] = 0; a3[e] = 0; }
#pragma unroll
    for (int e = 0; e < 4; ++e) cacc<GAUSS, T, V>(a1, a2, a3, a[e].x, a[e].y, b[e].x, b[e].y);
    cacc_final<GAUSS, V>(a1, a2, a3, re, im);
#pragma unroll
    for (int e = 0; e < 4; ++e) d[e] = mk<C>(c0[e].x + sign * re[e], c0[e].y + sign * im[e]);
}

// The unpivoted inverse of the kb x kb tile in a[] (256-thread layout of the
// pivoted path: thread t holds row t / 8, columns 4 (t % 8) .. +3), kb = 16
// or 32, left in L[0..kb)[0..kb) (row stride 33; L2 two such buffers).
// Returns whether a pivot was below tau2 * max|tile|^2.
// The second half: the tile already in L2 (rows 0 .. kb-1, stride 33),
// each wavefront's largest |a_ij|^2 in sh.amax and sh.small cleared, all
// visible to the workgroup.
// beside(): work for the other wavefronts while the first inverts A.
struct NoWork {
    __device__ __forceinline__ void operator()() const {}
};
template <typename T, typename W = NoWork>
__device__ __forceinline__ bool inv_blocked_core(int kb, typename CT<T>::c* L2, RowScratch<T>& sh, float tau2,
                                                 W beside = W());

template <typename T, typename W = NoWork>
__device__ __forceinline__ bool inv_blocked(typename CT<T>::c (&a)[4], int kb, typename CT<T>::c* L2,
                                            RowScratch<T>& sh, float tau2, W beside = W()) {
    const int t = threadIdx.x, w = t >> 6, l = t & 63;
    const int r = t >> 3, cg = t & 7;
    const bool act = (r < kb) && (4 * cg < kb);
    {
        float m2 = 0.0f;
        if (act) {
#pragma unroll
            for (int e = 0; e < 4; ++e) m2 = fmaxf(m2, (float)(a[e].x * a[e].x + a[e].y * a[e].y));
        }
        const uint32_t wm = wave_max_u32(__float_as_uint(m2));
        if (l == 0 && w < 4) sh.amax[w] = __uint_as_float(wm);   // more than 256 threads: the first four wavefronts hold the tile
        if (t == 0) sh.small = 0;
        if (act) {
#pragma unroll
            for (int e = 0; e < 4; ++e) L2[r * 33 + 4 * cg + e] = a[e];
        }
    }
    __syncthreads();
    return inv_blocked_core<T>(kb, L2, sh, tau2, beside);
}

template <typename T, typename W>
__device__ __forceinline__ bool inv_blocked_core(int kb, typename CT<T>::c* L2, RowScratch<T>& sh, float tau2,
                                                 W beside) {
    using C = typename CT<T>::c;
    const int t = threadIdx.x, w = t >> 6, l = t & 63;
    C* L = L2;               // the tile, then its inverse
    C* Lb = L2 + 32 * 33;    // X
    const float thr = tau2 * fmaxf(fmaxf(sh.amax[0], sh.amax[1]), fmaxf(sh.amax[2], sh.amax[3]));
    bool small = false;
    C* B = L + 16;
    C* Cq = L + 16 * 33;
    C* D = Cq + 16;
    C q[4], x[4], o[4], d[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = mk<C>(0, 0);
    if (w == 0) {   // A^-1, kept as rows
        const int lr = l & 15, lg = l >> 4;
        row_ops<T>(L, q);
        gj16_wave<T>(q, thr, small);
#pragma unroll
        for (int e = 0; e < 4; ++e) L[lr * 33 + acc_row<T>(lg, e)] = q[e];
    } else {
        beside();
    }
    if (kb == 32) {
        __syncthreads();
        if (w == 0) {
            C b[4], c[4];
            col_ops<T>(B, b);
            row_ops<T>(Cq, c);
            col_ops<T>(D, d);
            mm16<T>(q, b, o, (T)1, x);      // X = A^-1 B
            mm16<T>(c, x, d, (T)-1, d);     // S = D - C X: the rows of S^T
            col_put<T>(Lb, x);
            gj16_wave<T>(d, thr, small);    // the rows of (S^-1)^T
            col_put<T>(D, d);
        } else if (w == 1) {
            C c[4], b[4];
            row_ops<T>(Cq, c);
            col_ops<T>(L, b);
            mm16<T>(c, b, o, (T)1, x);      // Y = C A^-1
        }
        __syncthreads();
        if (w == 0) {
            row_ops<T>(Lb, q);
            mm16<T>(q, d, o, (T)-1, x);     // T12 = -X S^-1
            col_put<T>(B, x);
        } else if (w == 1) {
            C a[4];
            row_ops<T>(D, a);
            mm16<T>(a, x, o, (T)-1, q);     // T21 = -S^-1 Y
            col_put<T>(Cq, q);
            row_ops<T>(Lb, a);
            col_ops<T>(L, d);
            mm16<T>(a, q, d, (T)-1, x);     // T11 = A^-1 - X T21
            col_put<T>(L, x);
        }
    }
    if (small) sh.small = 1;
    __syncthreads();
    return sh.small != 0;
}

// Device-coherent store of one complex64 value: a relaxed agent-scope atomic
// store, which writes through the XCD's L2 to memory.
__device__ __forceinline__ void cst(float2* p, float2 v) {
    const unsigned long long w = (unsigned long long)__float_as_uint(v.x) |
                                 ((unsigned long long)__float_as_uint(v.y) << 32);
    __hip_atomic_store((HELM_GLOBAL unsigned long long*)p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Store of an updated panel element.  Complex64: a device-coherent store
// (written through to memory, no dirty line left in the XCD's L2); with
// every step rewriting the whole block, lines left dirty at the end of a
// launch delay the start of the next launch's workgroups (measured: the
// last workgroups entered ~4 us after the first, ~2 us with these stores).
// Complex128: a non-temporal store (two coherent 8-byte halves cost more
// than they save).
__device__ __forceinline__ void yst(float2* p, float2 v) { cst(p, v); }
__device__ __forceinline__ void yst(double2* p, double2 v) {
    gv2d w;
    w.x = v.x;
    w.y = v.y;
    __builtin_nontemporal_store(w, (HELM_GLOBAL gv2d*)p);
}

// Pivot tolerance of the unpivoted path: |a_pp|^2 >= TAU2 * max|a|^2.
constexpr float TAU2 = 1e-4f;

// The unpivoted inverse in L2 (stride 33) to Tt, transposed, row stride KB.
// Tt is device memory (the factor's tile slots) or LDS (the standalone
// tile-inverse kernel), so it is written through a generic pointer.
template <typename T>
__device__ __forceinline__ void store_inverse(int kb, const typename CT<T>::c* L2, typename CT<T>::c* Tt) {
    const int t = threadIdx.x, r = t >> 3, cg = t & 7;
    if ((r < kb) && (4 * cg < kb)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = 4 * cg + e;
            Tt[c * KB + r] = L2[r * 33 + c];
        }
    }
}

// Invert the kb x kb tile in a[] and store its inverse transposed
// (Tt[c][k] = T^{-1}[k][c]) with row stride KB.  M is a kb x 33 LDS buffer
// (pivoted path), L2 two 32 x 33 LDS buffers (unpivoted path).  Returns the
// first zero-pivot step (pivoted path) or -1; *small is set when the
// unpivoted path met a pivot below the tolerance.  Tt may be device memory
// or LDS (generic stores).
template <typename T>
__device__ __forceinline__ int invert_and_store(typename CT<T>::c (&a)[4], int kb, int pivot, GJScratch<T>& sh,
                                                typename CT<T>::c (*M)[33], typename CT<T>::c* L2,
                                                typename CT<T>::c* Tt, bool* small) {
    const int t = threadIdx.x, r = t >> 3, cg = t & 7;
    const bool act = (r < kb) && (4 * cg < kb);
    if (!pivot) {
        // diagonal pivots: the blocked form (two 16 x 16 inverses in one
        // wavefront each, the products around them on the matrix cores)
        RowScratch<T>& rs = *(RowScratch<T>*)&sh;
        *small = inv_blocked<T>(a, kb, L2, rs, TAU2);
        store_inverse<T>(kb, L2, Tt);
        return -1;
    }
    *small = false;
    int zero = (kb == 32) ? gj_invert<T, 32>(a, sh) : gj_invert<T, 16>(a, sh);
    if (act) {
#pragma unroll
        for (int e = 0; e < 4; ++e) M[r][4 * cg + e] = a[e];
    }
    __syncthreads();
    if (act) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = 4 * cg + e;
            Tt[c * KB + r] = M[sh.rowOf[r]][sh.stepOf[c]];
        }
    }
    return zero;
}

__device__ __forceinline__ void report_zero_pivot(int* status, int block, int row) {
    if (atomicCAS(&status[0], 0, 1) == 0) {
        status[1] = block;
        status[2] = row;
    }
}

}  // namespace helm
