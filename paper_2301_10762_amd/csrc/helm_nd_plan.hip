// Plan of the nested-dissection factorisation of an nx x nz grid (host).
//
// A box of nodes is cut across its longer side by a line of nodes (its
// separator) into two halves, until a box has at most ND_LEAF nodes.  The
// five-point operator couples the two halves through the line only, so
// eliminating boxes before the lines that bound them leaves, for each box, a
// dense front: its own pivots and the ring of nodes around it.
#include "helm_nd.h"

#include <algorithm>

namespace helm {

namespace {

struct Box {
    int x0, x1, z0, z1, depth;
    int child[2];
    int sep;   // separator column (x cut) or row (z cut); -1: leaf
    bool xcut;
    int size;  // boxes inside, itself included (they follow it)
};

int add_box(std::vector<Box>& v, int leaf, int x0, int x1, int z0, int z1, int depth) {
    const int id = (int)v.size();
    v.push_back({x0, x1, z0, z1, depth, {-1, -1}, -1, false, 1});
    const int w = x1 - x0, h = z1 - z0;
    if ((int64_t)w * h <= leaf) return id;
    int a, b;
    if (w >= h) {
        const int s = x0 + (w - 1) / 2;
        v[id].sep = s;
        v[id].xcut = true;
        a = add_box(v, leaf, x0, s, z0, z1, depth + 1), b = add_box(v, leaf, s + 1, x1, z0, z1, depth + 1);
    } else {
        const int s = z0 + (h - 1) / 2;
        v[id].sep = s;
        a = add_box(v, leaf, x0, x1, z0, s, depth + 1), b = add_box(v, leaf, x0, x1, s + 1, z1, depth + 1);
    }
    v[id].child[0] = a;
    v[id].child[1] = b;
    v[id].size = (int)v.size() - id;
    return id;
}

int pad16(int n) { return (n + 15) / 16 * 16; }

int box_pivots(const Box& b) {
    if (b.sep < 0) return (b.x1 - b.x0) * (b.z1 - b.z0);
    return b.xcut ? b.z1 - b.z0 : b.x1 - b.x0;
}
template <typename F>
void each_pivot(const Box& b, F f) {   // f(i, j)
    if (b.sep < 0) {
        for (int j = b.z0; j < b.z1; ++j)
            for (int i = b.x0; i < b.x1; ++i) f(i, j);
    } else if (b.xcut) {
        for (int j = b.z0; j < b.z1; ++j) f(b.sep, j);
    } else {
        for (int i = b.x0; i < b.x1; ++i) f(i, b.sep);
    }
}
// the nodes around a box that lie in the domain [xa, xb) x [za, zb)
template <typename F>
void each_ring(const Box& b, int xa, int xb, int za, int zb, F f) {
    if (b.z0 > za)
        for (int i = b.x0; i < b.x1; ++i) f(i, b.z0 - 1);
    if (b.x0 > xa)
        for (int j = b.z0; j < b.z1; ++j) f(b.x0 - 1, j);
    if (b.x1 < xb)
        for (int j = b.z0; j < b.z1; ++j) f(b.x1, j);
    if (b.z1 < zb)
        for (int i = b.x0; i < b.x1; ++i) f(i, b.z1);
}
int box_ring(const Box& b, int xa, int xb, int za, int zb) {
    int n = 0;
    each_ring(b, xa, xb, za, zb, [&](int, int) { ++n; });
    return n;
}
int64_t box_elems(const Box& b, int xa, int xb, int za, int zb) {
    const int64_t p = box_pivots(b);
    return b.sep < 0 ? p * p : p * (p + box_ring(b, xa, xb, za, zb));
}

int64_t count_elems(int leaf, int x0, int x1, int z0, int z1, int nx, int nz) {
    Box b{x0, x1, z0, z1, 0, {-1, -1}, -1, false, 1};
    const int w = x1 - x0, h = z1 - z0;
    int64_t in = 0;
    if ((int64_t)w * h > leaf) {
        if (w >= h) {
            b.sep = x0 + (w - 1) / 2;
            b.xcut = true;
            in = count_elems(leaf, x0, b.sep, z0, z1, nx, nz) + count_elems(leaf, b.sep + 1, x1, z0, z1, nx, nz);
        } else {
            b.sep = z0 + (h - 1) / 2;
            in = count_elems(leaf, x0, x1, z0, b.sep, nx, nz) + count_elems(leaf, x0, x1, b.sep + 1, z1, nx, nz);
        }
    }
    return in + box_elems(b, 0, nx, 0, nz);
}

int leaf_of(int nx, int nz) {
    const int64_t np = pad16(nx);
    return 2 * count_elems(ND_LEAF_MAX, 0, nx, 0, nz, nx, nz) <= np * np * nz ? ND_LEAF_MAX : ND_LEAF_MIN;
}

template <typename R>
int put_tab(std::vector<int>& t, const std::vector<R>& v) {
    static_assert(sizeof(R) % 4 == 0, "tables are whole words");
    const int at = (int)t.size();
    t.resize(t.size() + v.size() * sizeof(R) / 4);
    if (!v.empty()) std::copy((const int*)v.data(), (const int*)(v.data() + v.size()), t.begin() + at);
    return at;
}

// The shape of a w x h subtree with rings on the sides of `mask` (1 above,
// 2 left, 4 right, 8 below).
NdShape make_shape(int leaf, int w, int h, int mask, std::vector<int>& tabs) {
    NdShape S{};
    S.tab0 = (int)tabs.size();
    S.w = w;
    S.h = h;
    const int xa = mask & 2 ? -1 : 0, xb = mask & 4 ? w + 1 : w, za = mask & 1 ? -1 : 0, zb = mask & 8 ? h + 1 : h;
    std::vector<Box> box;
    add_box(box, leaf, 0, w, 0, h, 0);
    int depth = 0;
    for (auto& b : box) depth = std::max(depth, b.depth);
    auto at = [&](int i, int j) { return (j + 1) * (w + 2) + i + 1; };
    std::vector<int> zrow((size_t)(w + 2) * (h + 2), -1), wrow(zrow);
    std::vector<int> zi, zj, wi, wj, zp(box.size(), 0), fac(box.size(), 0);
    int64_t off = 0;
    for (size_t q = 0; q < box.size(); ++q) {
        fac[q] = (int)off;
        off += box_elems(box[q], xa, xb, za, zb);
    }
    std::vector<NdLeaf> leaves;
    for (size_t q = 0; q < box.size(); ++q)
        if (box[q].sep < 0) {
            for (int t = 0; t < (box_pivots(box[q]) + 15) / 16; ++t)
                leaves.push_back({box_pivots(box[q]), (int)wi.size(), fac[q], t});
            each_pivot(box[q], [&](int i, int j) {
                wrow[at(i, j)] = (int)wi.size();
                wi.push_back(i);
                wj.push_back(j);
            });
        }
    for (int d = depth; d >= 0; --d)
        for (size_t q = 0; q < box.size(); ++q)
            if (box[q].sep >= 0 && box[q].depth == d) {
                zp[q] = (int)zi.size();
                each_pivot(box[q], [&](int i, int j) {
                    zrow[at(i, j)] = (int)zi.size();
                    zi.push_back(i);
                    zj.push_back(j);
                });
            }
    S.nsep = (int)zi.size();
    each_ring(box[0], xa, xb, za, zb, [&](int i, int j) {
        zrow[at(i, j)] = (int)zi.size();
        zi.push_back(i);
        zj.push_back(j);
    });
    S.nring = (int)zi.size() - S.nsep;
    S.nw = (int)wi.size();
    std::vector<NdFwd> fwd;
    std::vector<NdBwd> bwd;
    std::vector<NdStep> steps;
    std::vector<int> adds, rings;
    for (int d = depth; d >= 0; --d) {
        NdStep st{(int)fwd.size(), 0, (int)adds.size(), 0, (int)bwd.size(), 0};
        int u = 0;
        std::vector<int> first(zi.size(), -1), second(zi.size(), -1), order;
        for (size_t q = 0; q < box.size(); ++q) {
            if (box[q].sep < 0 || box[q].depth != d) continue;
            const int p = box_pivots(box[q]), r0 = (int)rings.size(), u0 = u;
            each_ring(box[q], xa, xb, za, zb, [&](int i, int j) {
                const int r = zrow[at(i, j)];
                rings.push_back(r);
                if (first[r] < 0) {
                    first[r] = u;
                    order.push_back(r);
                } else {
                    second[r] = u;
                }
                ++u;
            });
            const int b = u - u0;
            for (int t = 0; t < (b + 15) / 16; ++t) fwd.push_back({zp[q], p, b, u0, fac[q], t});
            bwd.push_back({zp[q], p, b, r0, fac[q]});
        }
        for (int r : order) adds.push_back(r | first[r] << 10 | (second[r] < 0 ? 1023 : second[r]) << 20);
        st.nfwd = (int)fwd.size() - st.fwd;
        st.nadd = (int)adds.size() - st.add;
        st.nbwd = (int)bwd.size() - st.bwd;
        S.nu = std::max(S.nu, u);
        if (st.nbwd) steps.push_back(st);
    }
    // the box with the separator nodes right of it and below it, which are
    // its part of the upper rows
    const int ew = mask & 4 ? w + 1 : w, eh = mask & 8 ? h + 1 : h;
    S.xrow = S.nsep + S.nring + std::max(S.nw, S.nu);
    std::vector<int> boxt((size_t)ew * eh), xring, xback;
    for (int j = 0; j < eh; ++j)
        for (int i = 0; i < ew; ++i) {
            const int z = zrow[at(i, j)];
            int& b = boxt[(size_t)j * ew + i];
            if (i < w && j < h) {
                b = z >= 0 ? z : S.nsep + S.nring + wrow[at(i, j)];
            } else {
                b = S.xrow + (int)xring.size();
                xring.push_back(z >= 0 ? z - S.nsep : -1);
                xback.push_back(z >= 0 ? z : S.xrow);
            }
        }
    S.nx = (int)xring.size();
    // rows with a neighbour in `row` only
    auto stencil = [&](const std::vector<int>& vi, const std::vector<int>& vj, const std::vector<int>& row, int& count) {
        std::vector<short> t;
        count = 0;
        for (size_t q = 0; q < vi.size(); ++q) {
            const int i = vi[q], j = vj[q];
            auto nb = [&](int a, int b) {
                return (short)(a < -1 || a > w || b < -1 || b > h ? -1 : row[at(a, b)]);
            };
            const short n[4] = {nb(i - 1, j), nb(i + 1, j), nb(i, j - 1), nb(i, j + 1)};
            if (n[0] < 0 && n[1] < 0 && n[2] < 0 && n[3] < 0) continue;
            ++count;
            for (int v : {(int)q, i, j}) t.push_back((short)v);
            for (short v : n) t.push_back(v);
            t.push_back(0);
        }
        std::vector<int> o(t.size() / 2);
        std::copy(t.begin(), t.end(), (short*)o.data());
        return o;
    };
    const int a0 = put_tab(tabs, adds), r0 = put_tab(tabs, rings);
    for (auto& s : steps) s.add += a0;
    for (auto& b : bwd) b.ring += r0;
    const int f0 = put_tab(tabs, fwd), b0 = put_tab(tabs, bwd);
    for (auto& s : steps) {
        s.fwd = f0 + s.fwd * (int)(sizeof(NdFwd) / 4);
        s.bwd = b0 + s.bwd * (int)(sizeof(NdBwd) / 4);
    }
    S.nleaf = (int)leaves.size();
    S.leaf = put_tab(tabs, leaves);
    S.nstep = (int)steps.size();
    S.step = put_tab(tabs, steps);
    S.box = put_tab(tabs, boxt);
    S.xring = put_tab(tabs, xring);
    S.xback = put_tab(tabs, xback);
    S.zst = put_tab(tabs, stencil(zi, zj, wrow, S.nzst));
    S.wst = put_tab(tabs, stencil(wi, wj, zrow, S.nwst));
    S.ntab = (int)tabs.size() - S.tab0;
    return S;
}

}  // namespace

int64_t nd_factor_elems(int nx, int nz) { return count_elems(leaf_of(nx, nz), 0, nx, 0, nz, nx, nz); }

bool nd_build(int nx, int nz, NdPlan* plan) {
    NdPlan& P = *plan;
    P.nx = nx;
    P.nz = nz;
    const int N = nx * nz, leaf = leaf_of(nx, nz);
    std::vector<Box> box;
    box.reserve((size_t)N / 8 + 16);
    add_box(box, leaf, 0, nx, 0, nz, 0);
    int depth = 0, least = 1 << 30;   // deepest level, shallowest leaf
    for (auto& b : box) {
        depth = std::max(depth, b.depth);
        if (b.sep < 0) least = std::min(least, b.depth);
    }
    // subtrees: the boxes of the first level whose boxes are all small enough
    std::vector<int64_t> widest(depth + 1, 0);
    for (auto& b : box) widest[b.depth] = std::max(widest[b.depth], (int64_t)(b.x1 - b.x0) * (b.z1 - b.z0));
    int D = 0;
    while (D < least && widest[D] > ND_SUB) ++D;
    if (widest[D] > ND_SUB) return false;
    // fronts: leaves first, then by level, deepest first; a level's in
    // recursion order
    std::vector<int> id(box.size()), boxof;
    boxof.reserve(box.size());
    std::vector<int> first, level_depth;
    for (int d = depth + 1; d >= 0; --d) {
        first.push_back((int)boxof.size());
        for (size_t q = 0; q < box.size(); ++q)
            if (d > depth ? box[q].sep < 0 : (box[q].sep >= 0 && box[q].depth == d)) {
                id[q] = (int)boxof.size();
                boxof.push_back((int)q);
            }
        if ((int)boxof.size() == first.back()) first.pop_back();
        else level_depth.push_back(d);
    }
    first.push_back((int)boxof.size());
    P.fronts.assign(box.size(), NdFront{});
    // rows: separators above the subtrees, then subtree by subtree
    std::vector<int> row(N, -1);
    auto number = [&](const Box& b, NdFront& F) {
        F.piv0 = P.nrow;
        each_pivot(b, [&](int i, int j) {
            row[j * nx + i] = P.nrow++;
            P.nodeof.push_back(j * nx + i);
        });
    };
    for (size_t f = 0; f < box.size(); ++f) {
        const Box& b = box[boxof[f]];
        if (b.sep >= 0 && b.depth < D) number(b, P.fronts[f]);
    }
    P.nrow_up = P.nrow;
    struct Key {
        int w, h, mask, shape;
    };
    std::vector<Key> keys;
    for (size_t q = 0; q < box.size(); ++q) {
        const Box& b = box[q];
        if (b.depth != D) continue;
        NdSub s{};
        s.x0 = b.x0;
        s.z0 = b.z0;
        s.row = P.nrow;
        s.fac = P.fac_elems;
        const int w = b.x1 - b.x0, h = b.z1 - b.z0;
        const int mask = (b.z0 > 0 ? 1 : 0) | (b.x0 > 0 ? 2 : 0) | (b.x1 < nx ? 4 : 0) | (b.z1 < nz ? 8 : 0);
        s.shape = -1;
        for (auto& k : keys)
            if (k.w == w && k.h == h && k.mask == mask) s.shape = k.shape;
        if (s.shape < 0) {
            s.shape = (int)P.shapes.size();
            keys.push_back({w, h, mask, s.shape});
            P.shapes.push_back(make_shape(leaf, w, h, mask, P.tabs));
            const NdShape& S = P.shapes.back();
            P.sub_rows = std::max(P.sub_rows, S.xrow + S.nx);
            P.sub_brows = std::max(P.sub_brows, S.xrow);
            P.sub_tab = std::max(P.sub_tab, S.ntab);
            if (S.nleaf > ND_SUB_LEAVES) return false;
        }
        s.w = w;
        s.h = h;
        s.ew = b.x1 < nx ? w + 1 : w;
        s.eh = b.z1 < nz ? h + 1 : h;
        s.corner = b.x1 < nx && b.z1 < nz ? row[b.z1 * nx + b.x1] : -1;
        if (s.ew * s.eh > ND_SUB_EXT) return false;
        s.nsep = P.shapes[s.shape].nsep;
        s.nring = P.shapes[s.shape].nring;
        for (int r = 0; r < b.size; ++r) {   // its boxes in the shape's order
            P.fronts[id[q + r]].fac = P.fac_elems;
            P.fac_elems += box_elems(box[q + r], 0, nx, 0, nz);
        }
        for (int d = depth; d >= D; --d)
            for (int r = 0; r < b.size; ++r)
                if (box[q + r].sep >= 0 && box[q + r].depth == d) number(box[q + r], P.fronts[id[q + r]]);
        P.subs.push_back(s);
    }
    P.nsub = (int)P.subs.size();
    for (size_t f = 0; f < box.size(); ++f) {
        const Box& b = box[boxof[f]];
        NdFront& F = P.fronts[f];
        F.leaf = b.sep < 0;
        F.p = box_pivots(b);
        F.b = F.leaf ? 0 : box_ring(b, 0, nx, 0, nz);
        F.pp = pad16(F.p);
        F.fp = F.pp + pad16(F.b);
        F.npan = (F.pp + KB - 1) / KB;
        F.x0 = b.x0;
        F.z0 = b.z0;
        F.w = b.x1 - b.x0;
        F.h = b.z1 - b.z0;
        if (b.depth < D) {
            F.fac = P.fac_elems;
            P.fac_elems += box_elems(b, 0, nx, 0, nz);
        }
        F.ring = (int)P.ring.size();
        if (!F.leaf || b.depth == D) each_ring(b, 0, nx, 0, nz, [&](int i, int j) { P.ring.push_back(row[j * nx + i]); });
        for (int c = 0; c < 2; ++c) F.child[c] = b.child[c] < 0 ? -1 : id[b.child[c]];
    }
    {
        int s = 0;
        for (size_t q = 0; q < box.size(); ++q)
            if (box[q].depth == D) P.subs[s++].ring = P.fronts[id[q]].ring;
    }
    std::vector<int> slot(N, -1), local;
    for (size_t f = 0; f < box.size(); ++f) {
        const Box& b = box[boxof[f]];
        NdFront& F = P.fronts[f];
        if (F.leaf) continue;
        local.clear();
        each_pivot(b, [&](int i, int j) { local.push_back(j * nx + i); });
        each_ring(b, 0, nx, 0, nz, [&](int i, int j) { local.push_back(j * nx + i); });
        for (int c = 0; c < 2; ++c) {
            const Box& cb = box[b.child[c]];
            const bool lf = cb.sep < 0;
            int n = 0;
            each_ring(cb, 0, nx, 0, nz, [&](int i, int j) {
                const int ii = std::min(std::max(i, cb.x0), cb.x1 - 1), jj = std::min(std::max(j, cb.z0), cb.z1 - 1);
                slot[j * nx + i] = lf ? (jj - cb.z0) * (cb.x1 - cb.x0) + ii - cb.x0 : n;
                ++n;
            });
            F.map[c] = (int)P.map.size();
            for (int k : local) P.map.push_back(slot[k]);
            each_ring(cb, 0, nx, 0, nz, [&](int i, int j) { slot[j * nx + i] = -1; });
        }
    }
    P.upper = (int)level_depth.size();
    for (size_t v = 0; v < level_depth.size(); ++v) {
        NdLevel L{};
        const int d = level_depth[v];
        L.first = first[v];
        L.count = first[v + 1] - first[v];
        L.parity = d & 1;
        L.leaf = d > depth;
        for (int q = 0; q < L.count; ++q) {
            const NdFront& F = P.fronts[L.first + q];
            L.npan = std::max(L.npan, F.npan);
            L.pmax = std::max(L.pmax, F.pp);
            L.fmax = std::max(L.fmax, F.fp);
        }
        L.small = !L.leaf && nd_narrow(L.pmax, L.fmax);
        int64_t work = 0;
        for (int q = 0; q < L.count; ++q) {
            NdFront& F = P.fronts[L.first + q];
            F.urow = L.urows;
            if (!F.leaf && d <= D) L.urows += F.b;
            F.work = work;
            if (!L.leaf && !L.small) work += 3 * (int64_t)F.pp * F.fp + 2 * KB * KB;
            F.s = work;
            work += (int64_t)F.b * F.b;
        }
        L.tile0 = (int)P.tiles.size();
        if (!L.leaf && !L.small)
            for (int q = 0; q < L.count; ++q) {
                const NdFront& F = P.fronts[L.first + q];
                for (int i = 0; i < (F.pp + KB - 1) / KB; ++i)
                    for (int j = 0; j < (F.fp + TILE - 1) / TILE; ++j) P.tiles.push_back({q, (short)i, (short)j});
            }
        L.tiles = (int)P.tiles.size() - L.tile0;
        L.stile0 = (int)P.tiles.size();
        if (!L.leaf && !L.small)
            for (int q = 0; q < L.count; ++q) {
                const int n = (P.fronts[L.first + q].b + TILE - 1) / TILE;
                for (int i = 0; i < n; ++i)
                    for (int j = i; j < n; ++j) P.tiles.push_back({q, (short)i, (short)j});
            }
        L.stiles = (int)P.tiles.size() - L.stile0;
        if (d < D) {
            P.upper = std::min(P.upper, (int)v);
            // few fronts: one row tile per workgroup, its wavefronts sharing
            // the contraction (latency); many: a tile per wavefront, so that
            // the gathered vectors are staged once for four.  In us, 1 row tile
            // against 4: 16 to 256 fronts of 401^2, 5 systems, 82 .. 243 /
            // 53 .. 127; 4 fronts of 201^2, 4 systems of 32 columns, 13 / 15;
            // of 101^2 6 / 8
            L.frt = L.count >= 16 ? 4 : 1;
            L.frow0 = (int)P.tiles.size();
            for (int q = 0; q < L.count; ++q) {
                const NdFront& F = P.fronts[L.first + q];
                if (F.b == 0)
                    for (int i = 0; 64 * i < F.p; ++i) P.tiles.push_back({q, (short)i, 0});
                for (int i = 0; 16 * i < F.b; i += L.frt) P.tiles.push_back({q, (short)i, 0});
            }
            L.frows = (int)P.tiles.size() - L.frow0;
            L.brow0 = (int)P.tiles.size();
            for (int q = 0; q < L.count; ++q)
                for (int i = 0; 16 * i < P.fronts[L.first + q].p; ++i) P.tiles.push_back({q, (short)i, 0});
            L.brows = (int)P.tiles.size() - L.brow0;
        }
        P.work_elems[L.parity] = std::max(P.work_elems[L.parity], work);
        P.levels.push_back(L);
    }
    // the subtrees' ring contributions: a vector block of their level, also
    // where a subtree is a single leaf
    P.sub_parity = D & 1;
    int ur = 0, s = 0;
    for (size_t q = 0; q < box.size(); ++q)
        if (box[q].depth == D) {
            P.subs[s++].urow = ur;
            P.fronts[id[q]].urow = ur;
            ur += box_ring(box[q], 0, nx, 0, nz);
        }
    P.urows[P.sub_parity] = ur;
    for (size_t v = P.upper; v < P.levels.size(); ++v)
        P.urows[P.levels[v].parity] = std::max(P.urows[P.levels[v].parity], (int64_t)P.levels[v].urows);
    for (auto& F : P.fronts)
        for (int c = 0; c < 2; ++c) F.curow[c] = F.child[c] < 0 ? 0 : P.fronts[F.child[c]].urow;
    return nd_sub_forward_lds(P) <= ND_LDS && nd_sub_backward_lds(P) <= ND_LDS;
}

}  // namespace helm
