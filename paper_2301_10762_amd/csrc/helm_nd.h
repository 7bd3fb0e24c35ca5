// Nested-dissection factorisation: the elimination tree of a grid (its plan)
// and the tables the kernels read.  Host and device.
#pragma once
#include <memory>
#include <mutex>
#include <utility>
#include <vector>

#include "helm_internal.h"

namespace helm {

// Nodes of a leaf box.  A leaf keeps its whole inverse, so the factor's size
// and the solves' work grow with this, and the number of levels falls: 36
// (6 x 6) is taken where the factor then still fits the room of the complex64
// block factor it replaces, 16 elsewhere (narrow grids).
constexpr int ND_LEAF_MAX = 36, ND_LEAF_MIN = 16;

// Nodes of a subtree that one workgroup sweeps.  With 16 columns its vectors
// and tables take 63 to 75 KB of LDS forward and 73 to 84 KB backward (12 x 12
// boxes at 401^2, 13 x 13 at 55^2), so that two workgroups share a compute unit,
// backward all but the largest.
constexpr int ND_SUB = 170;
static_assert(17 * 17 > ND_SUB, "the subtree kernels take separators of at most 16 nodes");
constexpr int ND_SUB_LEAVES = 16;   // 16-row tiles of its leaves, at most
constexpr int ND_SUB_EXT = 224;     // nodes with the separators right of it and below it, at most

// One front of the elimination tree: the p pivots of a box's separator line
// (or all nodes of a leaf box) and the b nodes of the ring around the box,
// all of which belong to separators eliminated later.  Local indices
// 0 .. p-1 are the pivots, p .. p+b-1 the ring; in the working memory the
// pivots are padded to pp and the ring to fp - pp (multiples of 16), pivots
// with an identity tail.
//
// A leaf keeps G, the inverse of its block of the operator, alone: a ring
// node couples to one node of the leaf, so its R = G F is a scaled column of
// G and its Schur complement a scaled part of G, taken where needed.
struct NdFront {
    int p, b, pp, fp;
    int piv0;          // first pivot's row (separators; rows are numbered below)
    int ring;          // the ring's rows: ring[ring .. ring + b)
    int child[2];      // fronts of the two halves, or -1
    int map[2];        // per local index (p + b of them): its place in the child's ring
                       // (a leaf child: the leaf node it couples to), or -1
    int npan;          // panels of KB pivots
    int urow;          // first row of its ring contributions in the level's vector block
    int curow[2];      // the halves' urow
    int64_t fac;       // factor store: [G | R], p x (p + b), column-major (a leaf: G)
    int64_t work;      // a wide front's working memory (nd_rows, nd_tslot)
    int64_t s;         // Schur complement on the ring (b x b, row-major), valid for row <= column
    int leaf;
    int pad_;
    int x0, z0, w, h;  // box
};
static_assert(sizeof(NdFront) % 8 == 0, "fronts are read as whole words");

// a 32 x 64 tile of a front's pivot rows or (ti <= tj) a 64 x 64 one of its ring, or a 16-row tile of
// a front's sweep product; front: index within the level
struct NdTile {
    int front;
    short ti, tj;
};

struct NdLevel {
    int first, count;         // fronts
    int parity;               // which of the two working regions and vector blocks it uses
    bool leaf;                // the leaves
    bool small;               // narrow fronts: one workgroup each
    int npan;                 // panels of the front with most
    int tile0, tiles;         // 32 x 64 tiles of the pivot rows (wide fronts)
    int stile0, stiles;       // and of the rings' upper halves
    // levels above the subtrees
    int frow0, frows, frt;    // forward sweep: groups of frt 16-row tiles of the rings
    int brow0, brows;         // backward sweep: 16-row tiles of the pivots
    int urows;                // rows of ring contributions
    int pmax, fmax;           // widest pivot block and front (padded)
};

// The bottom of the tree is swept by one workgroup per subtree and 16
// columns, with its vectors in LDS.  Subtrees of one size with rings on the
// same sides share a shape, whose tables use local rows: z rows are the
// subtree's separator nodes (deepest level first) and then its ring, w rows
// the nodes of its leaves.
struct NdLeaf {               // a 16-row tile of a leaf
    int p, wrow, fac, tile;   // nodes, first w row, place in the subtree's factor
};
struct NdFwd {                // a 16-row tile of a front's ring
    int zp, p, b, u, fac, tile;   // first z row of the pivots, rows of u from `u`
};
struct NdBwd {                // a front
    int zp, p, b, ring, fac;  // ring: its z rows, in the shape's ring table
};
struct NdStep {               // a level of a shape, deepest first
    int fwd, nfwd, add, nadd, bwd, nbwd;
};
struct NdShape {
    int w, h, nsep, nring, nw, nu;   // nu: most rows of u of a level
    int nleaf, leaf;          // leaf tiles
    int nstep, step;          // levels
    // per node of the box and of the separators right of it and below it: its
    // row (z rows, then w rows; the nx outer ones from xrow on)
    int box, nx, xrow;
    int xring;                // the outer nodes' places in the ring (-1: the corner)
    int xback;                // and z rows (xrow: the corner)
    // per z row beside a w row, as shorts: the row, its i, j, and the w rows
    // left, right, above, below it (-1: none); per w row beside a z row: the same
    int zst, nzst, wst, nwst;
    int tab0, ntab;           // all of the shape's tables
};
struct NdSub {
    int shape, x0, z0, w, h;
    int ew, eh;               // with the separators right of it and below it
    int corner;               // row of the node right of and below it, or -1
    int nsep, nring;          // rows of its separators and its ring
    int row;                  // row of its first separator node
    int ring;                 // its ring's rows in the ring table
    int urow;                 // its ring contributions' first row
    int64_t fac;
};

// The plan of an nx x nz grid: host description and device tables (one
// allocation, complete when the plan is handed out).  Shared by every factor
// on the grid; it depends on nothing but nx and nz.  Separator nodes have
// rows: those above the subtrees first.
struct NdPlan {
    int nx = 0, nz = 0, dev = 0;
    std::vector<NdFront> fronts;     // leaves, then deepest level first
    std::vector<NdLevel> levels;     // leaves, then in elimination order (the root last)
    int upper = 0;                   // first level above the subtrees
    std::vector<int> ring, map, nodeof;
    std::vector<NdTile> tiles;
    std::vector<NdSub> subs;
    std::vector<NdShape> shapes;
    std::vector<int> tabs;           // the shapes' tables (NdLeaf, NdFwd, NdBwd, NdStep and index tables)
    int sub_rows = 0, sub_brows = 0; // most rows of a subtree in LDS, forward and backward
    int sub_tab = 0;                 // words of a shape's tables
    int sub_parity = 0;
    int nrow = 0, nrow_up = 0;       // separator nodes, those above the subtrees
    int nsub = 0;
    int64_t fac_elems = 0;           // complex128 values of a factor
    int64_t work_elems[2] = {0, 0};  // working memory of even and odd levels, per system
    int64_t urows[2] = {0, 0};       // ring-contribution rows of even and odd levels
    void* mem = nullptr;             // device tables
    size_t mem_bytes = 0;
    // where each stream stood when a factor of this plan was last released on
    // it: once these have passed no kernel reads the tables
    std::mutex mu;
    std::vector<std::pair<hipStream_t, hipEvent_t>> last;
    void* reserve = nullptr;         // scratch of one column's solve (grids beyond the fixed region only)
    size_t reserve_bytes = 0;
    const NdFront* d_fronts = nullptr;
    const int *d_ring = nullptr, *d_map = nullptr, *d_nodeof = nullptr, *d_tabs = nullptr;
    const NdTile* d_tiles = nullptr;
    const NdSub* d_subs = nullptr;
    const NdShape* d_shapes = nullptr;
    size_t col_bytes() const {       // sweep scratch per right-hand side, with a residual
        return sizeof(double) * 2 * ((size_t)nx * nz + (size_t)nx * nz / 256 + 1 + (size_t)(nrow_up + nrow + urows[0] + urows[1]));
    }
};

// host description only (no device memory); false: the grid does not divide
// into subtrees of the size the sweeps take, or whose vectors fit the LDS
bool nd_build(int nx, int nz, NdPlan* plan);
// complex128 values a factor of this grid stores
int64_t nd_factor_elems(int nx, int nz);

// device tables of a plan as the kernels take them
struct NdTabs {
    const NdFront* fronts;
    const int *ring, *map, *nodeof, *tabs;
    const NdTile* tiles;
    const NdSub* subs;
    const NdShape* shapes;
};

constexpr int ND_MAXS = 16;   // systems per launch

// Steps of the largest |T_ij|^2 (tile inverses, in couplings) that count.  A
// plain solve leaves at most 5e-15 max|T|^2 (480 systems, 33^2 to 401^2; up to
// 3 couplings what block factors leave) and each correction multiplies that by
// as much again: above 3, 10^3, 3 10^4 and 2 10^5 couplings a solve without a
// tolerance takes ND_FIXES corrections, above 10^6 the system is factored row
// by row.
constexpr int ND_STEPS = 5;
constexpr float ND_GROWN[ND_STEPS] = {9.0f, 1e6f, 9e8f, 4e10f, 1e12f};
constexpr int ND_FIXES[ND_STEPS - 1] = {1, 2, 3, 5};

struct NdSys {        // one system being factored
    Coef cf;
    double2* fac;
    double2* work[2];   // working memory of even and odd levels
    int* status;        // [0] zero-pivot flag, [1] front, [2] row, [3] steps of ND_GROWN passed (bits)
    int pivot;          // 1: partial pivoting in every tile
    int pad_;
};
struct NdSysTab {
    NdSys s[ND_MAXS];
};
struct NdJob {        // one block of right-hand sides being solved
    Coef cf;
    const double2* fac;
    const double2* B;   // right-hand sides, column-major (ldb)
    double2* X;         // solutions, column-major (ldx)
    int64_t ldb, ldx;
    double2* a;         // rows above the subtrees, [row][S]: right-hand sides, then the solution
    double2* y;         // every row: forward results
    double2* u[2];      // ring contributions of even and odd levels
    int S, pad_;
};
struct NdJobTab {
    NdJob j[ND_MAXS];
};
static_assert(sizeof(NdSysTab) <= 4000 && sizeof(NdJobTab) <= 4000, "tables pass through a kernel argument");

void launch_nd_put_sys(const NdSysTab& tab, NdSysTab* dst, hipStream_t st);
void launch_nd_put_jobs(const NdJobTab& tab, NdJobTab* dst, hipStream_t st);
// LDS a workgroup may take, all of it dynamic: a compute unit's 160 KB with a
// little left for the launch; what a level's narrow fronts (kp: 16 or 32
// pivots) and the subtree sweeps take; whether a level's fronts are narrow
// (those that do not fit go the wide fronts' way)
constexpr size_t ND_LDS = 160 * 1024 - 512;
size_t nd_front_lds(int kp, int fmax);
size_t nd_sub_forward_lds(const NdPlan& p);
size_t nd_sub_backward_lds(const NdPlan& p);
bool nd_narrow(int pmax, int fmax);
// factorisation of one level; adds its launches to *launches
hipError_t launch_nd_level(const NdTabs& t, const NdLevel& lv, const NdSysTab* dsys, int n, hipStream_t st,
                           int64_t* launches);
// one level's forward and backward sweep, above the subtrees
void launch_nd_forward(const NdTabs& t, const NdLevel& lv, const NdJobTab* djobs, int n, int smax, hipStream_t st);
void launch_nd_backward(const NdTabs& t, const NdLevel& lv, const NdJobTab* djobs, int n, int smax, hipStream_t st);
// the subtrees' sweeps: from B to ring contributions, and from the rings' solutions to X
hipError_t launch_nd_sub_forward(const NdTabs& t, const NdPlan& p, const NdJobTab* djobs, int n, int smax, bool conj,
                                 hipStream_t st);
hipError_t launch_nd_sub_backward(const NdTabs& t, const NdPlan& p, const NdJobTab* djobs, int n, int smax, bool add,
                                  bool conj, hipStream_t st);

}  // namespace helm
