// Block factorisation kernels of libhelm (gfx950).
//
// For each system the Schur complements of the block-tridiagonal operator,
//     D_0 = A_0,   D_{j+1} = A_{j+1} - E D_j^{-1} E,
// are inverted in place by block Gauss-Jordan on panels of KB = 32 columns.
// Panel K of block j, with T = (X_KK)^{-1} the inverse of its diagonal tile
// (pivoting inside the tile only), maps the working block X to
//     Y = X' + W V,   W = [-X_{:,K} T ; T - I],   V = [X_{K,:} with V_KK = I],
// X' = X with the K columns cleared except X'_KK = I.  After the last panel Y
// is D_j^{-1}; the same launch also writes D_{j+1} for the next block.
//
// One launch per panel step serves every chain of the batch.  Its
// workgroups are the 32 x 64 output tiles of Y (each forms its rows of W
// from X and T itself, so X and Y live in different buffers and no copy of
// V is needed) plus one workgroup per chain that builds the diagonal tile
// the NEXT step needs,
//     Z = X_{K'K'} - X_{K'K} T X_{KK'}            (next panel K' of block j), or
//     Z = A_{j+1}[K'K'] - E (Y restricted) E       (first panel of block j+1),
// and inverts it, so the sequential pivoting of the next step runs
// concurrently with this step's matrix-core update.
#include "helm_launch.h"
#include "helm_tile.h"

#include <type_traits>

namespace helm {

// ----------------------------------------------------------------- launches --
// LDS of a step workgroup: update tiles use sW (32 x 33) and sV (64 x 33); the
// next-tile workgroup four 32 x 33 blocks and the pivoting scratch
template <typename T>
constexpr size_t sm_bytes() {
    using C = typename CT<T>::c;
    constexpr size_t upd = (32 + 64) * 33 * sizeof(C), nxt = 4 * 32 * 33 * sizeof(C) + sizeof(GJScratch<T>);
    return upd > nxt ? upd : nxt;
}

__host__ __device__ int init_blocks(int np) { return (int)(((int64_t)np * np + 255) / 256) + 1; }
__host__ __device__ int step_blocks(int np) {
    return ((np + KB - 1) / KB) * ((np + TILE - 1) / TILE) + 1;
}
int factor_init_blocks(int np) { return init_blocks(np); }
int factor_step_blocks(int np) { return step_blocks(np); }

// D = A_{row0} into the first block of each front, and the inverse of its
// first diagonal tile
template <typename T>
__global__ __launch_bounds__(256) void k_factor_init(const ChainTab* __restrict__ tab, int n) {
    using C = typename CT<T>::c;
    __shared__ C M[32][33];
    __shared__ C L2[2 * 32 * 33];
    __shared__ GJScratch<T> sh;
    const int ci = find_chain(tab->c, n, blockIdx.x, [](const ChainInfo& c) { return c.itile0; });
    const ChainInfo d = load_entry(tab->c, ci);
    const int local = blockIdx.x - d.itile0;
    const int np = d.np;
    const int nfill = init_blocks(np) - 1;
    if (local < nfill) {
        const int64_t e = (int64_t)local * 256 + threadIdx.x;
        if (e < (int64_t)np * np) {
            const int r = (int)(e / np), q = (int)(e % np);
            const double2 v = block_entry(d.cf, d.row0, r, q);
            ((C*)d.G)[(size_t)d.row0 * np * np + e] = mk<C>(v.x, v.y);
        }
        return;
    }
    const int kb = min(KB, np);
    const int t = threadIdx.x, r = t >> 3, cg = t & 7;
    C a[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int c = 4 * cg + e;
        const double2 v = (r < kb && c < kb) ? block_entry(d.cf, d.row0, r, c) : make_double2(0.0, 0.0);
        a[e] = mk<C>(v.x, v.y);
    }
    bool small;
    const int zero = invert_and_store<T>(a, kb, d.pivot, sh, M, L2, (C*)d.Tb, &small);
    if (zero >= 0 && t == 0) report_zero_pivot(d.status, d.row0, zero);
    if (small && t == 0) d.status[3] = 1;
}

// Source of A for the block after local block jl of a front: the merge
// block for the top front's last block, else null (assemble from m).
template <typename C>
__device__ __forceinline__ const C* next_a_source(const ChainInfo& d, int jl) {
    return (d.Ain && jl + 1 == d.nblk - 1) ? (const C*)d.Ain : nullptr;
}

// What a lane needs to form entries of A_{j+1} - E G_j E in its columns: the
// couplings and the diagonal entries, prepared while the step's operands are
// on their way.  (Formed entry by entry after the product, with its divisions
// and its load of m behind the branch on the diagonal, this was 20 k of the
// 36 k cycles of a block's last step at np = 48.)
template <int NC>
struct NextBlock {
    double cx, ez;        // x coupling of the row, z coupling between the rows
    double2 dg[NC];       // diagonal entries of the lane's columns
};
// mk: m at the lane's columns (clamped) of row jn
template <int NC>
__device__ __forceinline__ NextBlock<NC> next_block(const Coef& c, int jn, const int (&col)[NC], const double (&mk)[NC]) {
    NextBlock<NC> b;
    b.cx = x_coupling(c, jn);
    b.ez = c.hx / c.hz;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
        b.dg[q] = diag_value(c, min(col[q], c.nx - 1), jn, mk[q]);
        asm volatile("" : "+v"(b.dg[q].x), "+v"(b.dg[q].y));   // here, not where it is used
    }
    asm volatile("" : "+v"(b.cx), "+v"(b.ez));
    return b;
}
// entry (r, col) of A_{j+1} (block_entry)
template <int NC>
__device__ __forceinline__ double2 next_entry(const Coef& c, const NextBlock<NC>& b, int q, int r, int col) {
    const bool in = r < c.nx && col < c.nx, diag = r == col, side = r == col + 1 || col == r + 1;
    return make_double2(diag ? (in ? b.dg[q].x : 1.0) : (in && side ? -b.cx : 0.0), diag && in ? b.dg[q].y : 0.0);
}
// entry a of A_{j+1} (or of the merge block) less that of E G_j E, with g that
// of G_j; ez: hx / hz
template <typename C>
__device__ __forceinline__ C next_schur(const Coef& c, double ez, double2 a, int r, int col, C g) {
    const double er = r < c.nx ? -(ez * half_at_ends(r, c.nx)) : 0.0;
    const double ec = col < c.nx ? -(ez * half_at_ends(col, c.nx)) : 0.0;
    const double s = er * ec;
    return mk<C>(a.x - s * (double)g.x, a.y - s * (double)g.y);
}
// the same in one, for the tile that is inverted next
template <typename C>
__device__ __forceinline__ C next_schur(const ChainInfo& d, const NextBlock<1>& b, const C* Asrc, int r, int col, C g) {
    double2 a;
    if (Asrc) {
        const C v = gld(Asrc + (size_t)r * d.np + col);
        a = make_double2(v.x, v.y);
    } else {
        a = next_entry(d.cf, b, 0, r, col);
    }
    return next_schur<C>(d.cf, b.ez, a, r, col, g);
}

// workgroup that prepares the next step's inverted diagonal tile
template <typename T>
__device__ __forceinline__ void next_tile(const ChainInfo& d, const PanelStep& ps, const typename CT<T>::c* X,
                          const typename CT<T>::c* Tcur, typename CT<T>::c* Tnext, char* smem) {
    using C = typename CT<T>::c;
    const int np = d.np, kb = ps.kb, k0 = ps.k0;
    const int row = d.row0 + d.dir * ps.j;
    int jn, kn0, kbn;
    const C* Asrc = nullptr;
    if (!ps.last_panel) {
        jn = row;
        kn0 = k0 + kb;
    } else {
        if (ps.j + 1 >= d.nblk) return;
        jn = row + d.dir;
        kn0 = 0;
        Asrc = next_a_source<C>(d, ps.j);
    }
    kbn = min(KB, np - kn0);
    C (*sXa)[33] = (C(*)[33])smem;                      // X_{K'K}    kbn x kb
    C (*sT)[33] = (C(*)[33])(smem + 1 * 32 * 33 * sizeof(C));   // T   kb x kb
    C (*sXb)[33] = (C(*)[33])(smem + 2 * 32 * 33 * sizeof(C));  // X_{KK'}    kb x kbn
    C (*sP)[33] = (C(*)[33])(smem + 3 * 32 * 33 * sizeof(C));   // X_{K'K} T  kbn x kb
    GJScratch<T>& sh = *(GJScratch<T>*)(smem + 4 * 32 * 33 * sizeof(C));
    const int t = threadIdx.x, r = t >> 3, cg = t & 7;
    const bool single = ps.last_panel && d.npan == 1;   // next tile is Y = T itself
    const int w = t >> 6, l = t & 63, lr = l & 15, lg = l >> 4;
    const int wr = w >> 1, wc = w & 1;   // this wave's 16 x 16 output tile of the products
    // every global load is issued up front at a clamped (in-range) address;
    // entries outside the kb x kbn tiles are zeroed when they are placed.
    // T arrives transposed (Tt[c][k]): read it in order, place it as sT[k][c]
    C tl[4], xa[4], xb[4], xz[4];
    const double mk1[1] = {m_at(d.cf, min(16 * wc + lr, d.cf.nx - 1), jn)};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int idx = t + 256 * i;
        const int hi = idx >> 5, lo = idx & 31;
        tl[i] = gld(Tcur + idx);
        xa[i] = gld(X + (size_t)(kn0 + min(hi, kbn - 1)) * np + k0 + min(lo, kb - 1));
        xb[i] = gld(X + (size_t)(k0 + min(hi, kb - 1)) * np + kn0 + min(lo, kbn - 1));
    }
    // X_{K'K'} in the accumulator layout of this wave's tile
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int rr = 16 * wr + acc_row<T>(lg, e), cc = 16 * wc + lr;
        xz[e] = gld(X + (size_t)(kn0 + min(rr, kbn - 1)) * np + kn0 + min(cc, kbn - 1));
    }
    __builtin_amdgcn_sched_barrier(0);   // keep every load ahead of the first wait
    C am[4];   // the merge block's entries, or A's
    NextBlock<1> nb{};
    if (Asrc) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            am[e] = gld(Asrc + (size_t)min(16 * wr + acc_row<T>(lg, e), kbn - 1) * np + min(16 * wc + lr, kbn - 1));
    }
    if (ps.last_panel) nb = next_block<1>(d.cf, jn, {16 * wc + lr}, mk1);
    const C cz = mk<C>(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int idx = t + 256 * i;
        const int hi = idx >> 5, lo = idx & 31;
        sT[lo][hi] = HELM_CSEL(hi < kb && lo < kb, tl[i], cz);
        sXa[hi][lo] = HELM_CSEL(!single && hi < kbn && lo < kb, xa[i], cz);
        sXb[hi][lo] = HELM_CSEL(!single && hi < kb && lo < kbn, xb[i], cz);
    }
    using V = typename CT<T>::v4;
    V zr, zi;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int rr = 16 * wr + acc_row<T>(lg, e), cc = 16 * wc + lr;
        const C v = HELM_CSEL(!single && rr < kbn && cc < kbn, xz[e], cz);
        zr[e] = v.x;
        zi[e] = v.y;
    }
    C a[4];
    const bool act = (r < kbn) && (4 * cg < kbn);
    __syncthreads();
    if (single) {
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = HELM_CSEL(act, sT[r][4 * cg + e], mk<C>(0.0, 0.0));
    } else {
        // P = X_{K'K} T on the matrix cores (zero padding beyond kb, kbn), in
        // three real products per complex one like the update tiles' W
        V pr, pim;
        {
            V p1, p2, p3;
#pragma unroll
            for (int e = 0; e < 4; ++e) { p1[e] = 0; p2[e] = 0; p3[e] = 0; }
#pragma unroll
            for (int s8 = 0; s8 < 8; ++s8) {
                const C x = sXa[16 * wr + lr][4 * s8 + lg], y = sT[4 * s8 + lg][16 * wc + lr];
                cacc<true, T, V>(p1, p2, p3, x.x, x.y, y.x, y.y);
            }
            cacc_final<true, V>(p1, p2, p3, pr, pim);
        }
        // -P into sP (accumulator layout -> row-major)
#pragma unroll
        for (int e = 0; e < 4; ++e) sP[16 * wr + acc_row<T>(lg, e)][16 * wc + lr] = mk<C>(-pr[e], -pim[e]);
        __syncthreads();
        // Z = X_{K'K'} - P X_{KK'}
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) {
            const C x = sP[16 * wr + lr][4 * s8 + lg], y = sXb[4 * s8 + lg][16 * wc + lr];
            cmfma<T, V>(zr, zi, x.x, x.y, y.x, y.y);
        }
        if (!d.pivot) {
            // unpivoted: each wave puts its block of the tile (after the
            // Schur complement of the next block on a last panel) straight
            // into the inversion buffer and reports its largest |a_ij|^2
            C* L2 = &sT[0][0];   // T and X_{KK'} are no longer read there
            RowScratch<T>& rs = *(RowScratch<T>*)&sh;
            float m2 = 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int rr = 16 * wr + acc_row<T>(lg, e), cc = 16 * wc + lr;
                C v = mk<C>(zr[e], zi[e]);
                if (ps.last_panel) {
                    const double2 a = Asrc ? make_double2(am[e].x, am[e].y) : next_entry(d.cf, nb, 0, rr, cc);
                    v = next_schur<C>(d.cf, nb.ez, a, rr, cc, v);
                }
                v = HELM_CSEL(rr < kbn && cc < kbn, v, mk<C>(0.0, 0.0));
                m2 = fmaxf(m2, (float)(v.x * v.x + v.y * v.y));
                L2[rr * 33 + cc] = v;
            }
            const uint32_t wm = wave_max_u32(__float_as_uint(m2));
            if (l == 0) rs.amax[w] = __uint_as_float(wm);
            if (t == 0) rs.small = 0;
            __syncthreads();
            const bool small = inv_blocked_core<T>(kbn, L2, rs, TAU2);
            store_inverse<T>(kbn, L2, Tnext);
            if (small && t == 0) d.status[3] = 1;
            return;
        }
        // to the Gauss-Jordan layout through sXa (no longer read)
#pragma unroll
        for (int e = 0; e < 4; ++e) sXa[16 * wr + acc_row<T>(lg, e)][16 * wc + lr] = mk<C>(zr[e], zi[e]);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = HELM_CSEL(act, sXa[r][4 * cg + e], mk<C>(0.0, 0.0));
    }
    if (ps.last_panel && act) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            a[e] = next_schur<C>(d, next_block<1>(d.cf, jn, {4 * cg + e}, {m_at(d.cf, min(4 * cg + e, d.cf.nx - 1), jn)}),
                                 Asrc, r, 4 * cg + e, a[e]);
    }
    __syncthreads();   // sXa is reused as the inversion buffer
    bool small;
    const int zero = invert_and_store<T>(a, kbn, d.pivot, sh, sXa, &sT[0][0], Tnext, &small);
    if (zero >= 0 && t == 0) report_zero_pivot(d.status, jn, kn0 + zero);
    if (small && t == 0) d.status[3] = 1;
}

// Accumulators of the update tile's product seeded with its tile of X'
// (identity on the panel columns K, zero outside the block)
template <bool GAUSS, typename T, typename V, typename C>
__device__ __forceinline__ void seed_y(V (&a1)[2], V (&a2)[2], V (&a3)[2], const C (&xt)[2][4], int R,
                                       const int (&Cc)[2], bool vr, const bool (&vc)[2], int k0, int kb, int lr,
                                       int lg) {
    const C zero = mk<C>(0.0, 0.0);
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
        const int col = Cc[bj] + lr;
        const bool inK = col >= k0 && col < k0 + kb;
        V sre, sim;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = R + acc_row<T>(lg, e);
            C v = HELM_CSEL(inK, mk<C>(row == col ? 1.0 : 0.0, 0.0), xt[bj][e]);
            // complex128 selects part by part; complex64 keeps the branch
            if constexpr (sizeof(T) == 8) v = HELM_CSEL(vr && vc[bj], v, zero);
            else if (!(vr && vc[bj])) v = zero;
            sre[e] = v.x;
            sim[e] = v.y;
        }
        cacc_seed<GAUSS, V>(a1[bj], a2[bj], a3[bj], sre, sim);
    }
}

// update of one 32 x 64 tile of Y (a 64 x 64 one takes 23 k cycles at np = 48,
// longer than the next tile's workgroup beside it)
template <typename T>
__device__ __forceinline__ void update_tile(const ChainInfo& d, const PanelStep& ps, int ti, const typename CT<T>::c* X,
                            typename CT<T>::c* Y, const typename CT<T>::c* Tcur, char* smem) {
    using C = typename CT<T>::c;
    using V = typename CT<T>::v4;
    // three real products per complex one (Gauss) for the Y product in
    // complex128 only: in complex64 its larger rounding of the imaginary
    // parts costs a refinement step.  The W product takes three in both
    // precisions (the complex64 refinement count is unchanged).
    constexpr bool GAUSS = sizeof(T) == 8;
    const int np = d.np, kb = ps.kb, k0 = ps.k0;
    const int tiles_x = (np + TILE - 1) / TILE;
    const int I0 = (ti / tiles_x) * KB, J0 = (ti % tiles_x) * TILE;
    const int t = threadIdx.x, w = t >> 6, l = t & 63;
    const int lr = l & 15, lg = l >> 4;
    const int wr = w >> 1, wc = w & 1;
    C (*sW)[33] = (C(*)[33])smem;                      // W rows I0..I0+31, k < kb
    C (*sV)[33] = (C(*)[33])(smem + 32 * 33 * sizeof(C));  // V^T: sV[c][k], c = J0..J0+63

    const int R = I0 + 16 * wr;
    const bool vr = R < np;
    int Cc[2];
    bool vc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        Cc[q] = J0 + 32 * wc + 16 * q;
        vc[q] = Cc[q] < np;
    }
    const int row_b = d.row0 + d.dir * ps.j, rn = row_b + d.dir;
    C* An = nullptr;
    const C* Asrc = nullptr;
    if (ps.last_panel) {
        if (ps.j + 1 < d.nblk) {
            An = (C*)d.G + (size_t)rn * np * np;
            Asrc = next_a_source<C>(d, ps.j);
        } else if (d.Aout) {
            An = (C*)d.Aout;
        }
    }
    // 1. global loads, all issued up front: X_{I,K} (rows of this tile, panel
    //    columns) and T for the W product, V_J = X_{K,J} for the update (kept
    //    in registers until W is done), and this tile of X'
    C (*sT)[33] = sV;   // T shares the V buffer until W is formed
    // every load is issued at a clamped (in-range) address; out-of-range and
    // identity entries are substituted afterwards
    C xik[4], tv[4], vv[8], xt[2][4];
    const int rm = min(max(rn, 0), d.cf.nz - 1);
    const double mk2[2] = {m_at(d.cf, min(Cc[0] + lr, d.cf.nx - 1), rm), m_at(d.cf, min(Cc[1] + lr, d.cf.nx - 1), rm)};
    {
        const int rr = t >> 3, c4 = 4 * (t & 7), row = min(I0 + rr, np - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) xik[q] = gld(X + (size_t)row * np + k0 + min(c4 + q, kb - 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) tv[q] = gld(Tcur + t + 256 * q);   // Tt[c][k], idx = 32 c + k
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = t + 256 * q, k = i >> 6, cc = i & 63;
            vv[q] = gld(X + (size_t)(k0 + min(k, kb - 1)) * np + min(J0 + cc, np - 1));
        }
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                xt[bj][e] = gld(X + (size_t)min(R + acc_row<T>(lg, e), np - 1) * np + min(Cc[bj] + lr, np - 1));
    }
    __builtin_amdgcn_sched_barrier(0);   // keep every load ahead of the first wait
    NextBlock<2> nb{};
    if (An) nb = next_block<2>(d.cf, rm, {Cc[0] + lr, Cc[1] + lr}, mk2);
    const C zero = mk<C>(0.0, 0.0);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int i = t + 256 * q, k = i >> 6, col = J0 + (i & 63);
        if constexpr (sizeof(T) == 8) {   // part by part, as above
            vv[q] = HELM_CSEL(col >= k0 && col < k0 + kb, mk<C>(k == col - k0 ? 1.0 : 0.0, 0.0), vv[q]);
            vv[q] = HELM_CSEL(k < kb && col < np, vv[q], zero);
        } else {
            if (!(k < kb && col < np)) vv[q] = zero;
            else if (col >= k0 && col < k0 + kb) vv[q] = mk<C>(k == col - k0 ? 1.0 : 0.0, 0.0);
        }
    }
    // Y = X' + W V, accumulated from X'.  complex128 seeds its three
    // accumulators after the W product: the tile of X' is live across it
    // instead of them
    V a1[2], a2[2], a3[2];
    if constexpr (!GAUSS) seed_y<GAUSS, T>(a1, a2, a3, xt, R, Cc, vr, vc, k0, kb, lr, lg);
    // 2. X_{I,K} and T into LDS
    {
        const int rr = t >> 3, c4 = 4 * (t & 7);
        const bool rok = I0 + rr < np;
#pragma unroll
        for (int q = 0; q < 4; ++q) sW[rr][c4 + q] = HELM_CSEL(rok && c4 + q < kb, xik[q], zero);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = t + 256 * q, c = i >> 5, k = i & 31;
            sT[k][c] = HELM_CSEL(k < kb && c < kb, tv[q], mk<C>(0.0, 0.0));
        }
    }
    __syncthreads();
    // 3. W_I = -X_{I,K} T (matrix cores, one 16 x 16 block per wavefront), T - I on rows of K
    {
        V wre, wim, q1, q2, q3;
#pragma unroll
        for (int e = 0; e < 4; ++e) { q1[e] = 0; q2[e] = 0; q3[e] = 0; }
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) {
            const int k = 4 * s8 + lg;
            const C av = sW[16 * wr + lr][k], bv = sT[k][16 * wc + lr];
            cacc<true, T, V>(q1, q2, q3, av.x, av.y, bv.x, bv.y);
        }
        cacc_final<true, V>(q1, q2, q3, wre, wim);
        C tk[4];   // rows of K: T - I, read before the buffers are rewritten
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = R + acc_row<T>(lg, e), c = 16 * wc + lr;
            const bool in = row >= k0 && row < k0 + kb;
            tk[e] = HELM_CSEL(in, sT[in ? row - k0 : 0][c], mk<C>(0.0, 0.0));
        }
        __syncthreads();   // every wave has read X_{I,K} and T
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int rl = 16 * wr + acc_row<T>(lg, e), row = I0 + rl, c = 16 * wc + lr;
            C v;
            if (row >= k0 && row < k0 + kb) {
                v = tk[e];
                if (row - k0 == c) v.x -= (T)1;
            } else {
                v = mk<C>(-wre[e], -wim[e]);
            }
            sW[rl][c] = v;
        }
        // V_J into LDS, transposed (V_KK = I)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = t + 256 * q, k = i >> 6, cc = i & 63;
            sV[cc][k] = vv[q];
        }
    }
    if constexpr (GAUSS) seed_y<GAUSS, T>(a1, a2, a3, xt, R, Cc, vr, vc, k0, kb, lr, lg);
    __syncthreads();
    // 4. Y_IJ = X'_IJ + W_I V_J
    for (int kk = 0; kk < kb; kk += 16) {
        C av[4], bv[2][4];
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
                if (vr && vc[bj]) cacc<GAUSS, T, V>(a1[bj], a2[bj], a3[bj], av[s].x, av[s].y, bv[bj][s].x, bv[bj][s].y);
    }
    // 5. store; after the last panel also D_next = A_next - E Y E, into the
    //    front's next block, or into the merge block after a bottom front's
    //    last block
    auto store = [&](auto mode) {   // 0: Y alone, 1: and D_next from A's entries, 2: and from the merge block
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            if (!(vr && vc[bj])) continue;
            const int col = Cc[bj] + lr;
            V gre, gim;
            cacc_final<GAUSS, V>(a1[bj], a2[bj], a3[bj], gre, gim);
            C am[4];
            if (mode == 2) {
#pragma unroll
                for (int e = 0; e < 4; ++e) am[e] = gld(Asrc + (size_t)(R + acc_row<T>(lg, e)) * np + col);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = R + acc_row<T>(lg, e);
                const C g = mk<C>(gre[e], gim[e]);
                // the finished inverse goes to the sweeps' operand layout
                yst(Y + (ps.last_panel ? (sizeof(T) == 4 ? a_tiled4(row, col, np) : a_tiled(row, col, np))
                                       : (size_t)row * np + col),
                    g);
                if (mode > 0)
                    yst(An + (size_t)row * np + col,
                        next_schur<C>(d.cf, nb.ez, mode == 2 ? make_double2(am[e].x, am[e].y)
                                                             : next_entry(d.cf, nb, bj, row, col), row, col, g));
            }
        }
    };
    if (!An) store(std::integral_constant<int, 0>{});
    else if (!Asrc) store(std::integral_constant<int, 1>{});
    else store(std::integral_constant<int, 2>{});
}

// Workgroups 0 .. n-1 of a step launch prepare the next diagonal tile of
// chains 0 .. n-1 (the critical path of the step, so they are dispatched
// first); the rest update the 32 x 64 tiles, chain by chain (ftile0).
// uni > 0: every chain has uni - 1 update workgroups, laid out by XCD
// (xcd_tile); otherwise in launch order.
// Update tile served by workgroup b (>= n) when consecutive tiles (front by
// front, tile row by tile row) are kept on one XCD: workgroup b runs on XCD
// b % 8, so XCD x takes the contiguous range of tiles after those of XCDs
// 0 .. x-1, and the panel rows, columns and T of a front are fetched into
// one or two L2s instead of all eight.  total = n + update tiles.
__device__ __forceinline__ int xcd_tile(int b, int n, int total) {
    const int x = b & 7, k = b >> 3;
    int start = 0, leads_x = 0;
#pragma unroll
    for (int y = 0; y < 8; ++y) {
        const int wgs = total > y ? (total - 1 - y) / 8 + 1 : 0;
        const int leads = n > y ? (n - 1 - y) / 8 + 1 : 0;
        if (y < x) start += wgs - leads;
        if (y == x) leads_x = leads;
    }
    return start + k - leads_x;
}

template <typename T>
__global__ __launch_bounds__(256, 2) void k_factor_step(int n, int tstep, int uni, const ChainTab* __restrict__ tab) {
    using C = typename CT<T>::c;
    __shared__ __attribute__((aligned(16))) char smem[sm_bytes<T>()];
    const int b = blockIdx.x;
    const bool nxt = b < n;
    const int u = (!nxt && uni > 0) ? xcd_tile(b, n, n * uni) : b - n;
    const int ci = nxt ? b
                       : uni > 0 ? (int)((unsigned)u / (unsigned)(uni - 1))
                                 : find_chain(tab->c, n, u, [](const ChainInfo& c) { return c.ftile0; });
    const ChainInfo d = load_entry(tab->c, ci);
    if (tstep >= d.T) return;
    const PanelStep ps = panel_step(d, tstep);
    const int np = d.np;
    const size_t n2 = (size_t)np * np;
    C* G = (C*)d.G;
    const int row = d.row0 + d.dir * ps.j;
    const C* X = ps.p == 0 ? G + (size_t)row * n2 : (const C*)((ps.p - 1) & 1 ? d.P1 : d.P0);
    C* Y = ps.last_panel ? G + (size_t)row * n2 : (C*)(ps.p & 1 ? d.P1 : d.P0);
    const C* Tcur = (const C*)d.Tb + (size_t)(tstep & 1) * KB * KB;
    C* Tnext = (C*)d.Tb + (size_t)((tstep + 1) & 1) * KB * KB;
    if (nxt) {
        __builtin_amdgcn_s_setprio(3);   // ahead of the update tiles that share its compute unit
        next_tile<T>(d, ps, X, Tcur, Tnext, smem);
    } else {
        update_tile<T>(d, ps, u - d.ftile0, X, Y, Tcur, smem);
    }
}

// standalone tile inverses (the building block above, for tests)
__global__ __launch_bounds__(256) void k_tile_inverse(int kb, int pivot, const double2* A, double2* Tout, int* status) {
    __shared__ double2 M[32][33];
    __shared__ double2 L2[2 * 32 * 33];
    __shared__ GJScratch<double> sh;
    __shared__ double2 Tt[KB * KB];
    const int t = threadIdx.x, r = t >> 3, cg = t & 7;
    const double2* Am = A + (size_t)blockIdx.x * kb * kb;
    double2 a[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int c = 4 * cg + e;
        a[e] = (r < kb && c < kb) ? Am[r * kb + c] : make_double2(0.0, 0.0);
    }
    bool small;
    const int zero = invert_and_store<double>(a, kb, pivot, sh, M, L2, Tt, &small);
    __syncthreads();
    for (int i = t; i < kb * kb; i += 256) {
        const int rr = i / kb, c = i % kb;
        Tout[(size_t)blockIdx.x * kb * kb + i] = Tt[c * KB + rr];
    }
    if (t == 0 && zero >= 0) status[blockIdx.x] = 1 + zero;
    if (t == 0 && small) status[blockIdx.x] = -1;
}

void launch_factor_init(const ChainTab* dtab, int n, int total, bool fp32, hipStream_t st) {
    if (fp32) hipLaunchKernelGGL(k_factor_init<float>, dim3(total), dim3(256), 0, st, dtab, n);
    else hipLaunchKernelGGL(k_factor_init<double>, dim3(total), dim3(256), 0, st, dtab, n);
}
int factor_uniform(const ChainTab& tab, int n) {
    int uni = step_blocks(tab.c[0].np);
    for (int q = 0; q < n; ++q)
        if (tab.c[q].ftile0 != q * (uni - 1) || step_blocks(tab.c[q].np) != uni) uni = 0;
    return uni;
}
void launch_factor_step(const ChainTab* dtab, int n, int t, int uni, int total, bool fp32, hipStream_t st) {
    if (fp32) hipLaunchKernelGGL(k_factor_step<float>, dim3(total), dim3(256), 0, st, n, t, uni, dtab);
    else hipLaunchKernelGGL(k_factor_step<double>, dim3(total), dim3(256), 0, st, n, t, uni, dtab);
}
void launch_tile_inverse(int count, int kb, int pivot, const double* A, double* T, int* status, hipStream_t st) {
    hipLaunchKernelGGL(k_tile_inverse, dim3(count), dim3(256), 0, st, kb, pivot, (const double2*)A, (double2*)T,
                       status);
}

}  // namespace helm
