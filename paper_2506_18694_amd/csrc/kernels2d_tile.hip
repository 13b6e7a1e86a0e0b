// Fused 2D P1 multigrid passes on LDS tiles, one node per thread.
//
// The same passes as the register-streaming kernels (kernels2d_stream.hip)
// for launches too small to fill the chip with marching wavefronts.  There a
// wavefront advances one row per step through every stage, about 1 us per
// step with nothing beside it to hide the chain, so a four-sweep pass on a
// 64 x 64 mesh took 20 us however short its segments were.  Here a workgroup
// holds one TW x TH region (tile and halo) with x double-buffered in LDS and
// b, the centre value and the Jacobi factor in registers; a stage is six LDS
// reads, one node's arithmetic and one barrier (about 0.3 us; the launch and
// the loads take the other 2 us of a small pass).  The halo is recomputed (the
// four-sweep pass owns 20 x 20 nodes of a 32 x 32 region), which costs nothing
// while most compute units would idle.
//
// Every node gets the streaming kernels' roundings: the formulas are theirs,
// term by term, and nothing lets the compiler fuse a product into a sum, so
// the launch size alone decides which kernel runs and a column's result does
// not depend on how many columns share the launch.
#pragma clang fp contract(off)
#include "launch.h"

namespace helm {

namespace {

template <typename T>
__device__ __forceinline__ cx<T> zero_cx() { return mk((T)0, (T)0); }
template <typename T>
__device__ __forceinline__ cx<T> sel(bool c, cx<T> a, cx<T> b) {
    return mk(c ? a.x : b.x, c ? a.y : b.y);
}
// a + s t for a real s
template <typename T>
__device__ __forceinline__ cx<T> axpy_real(T sc, cx<T> t, cx<T> a) {
    return mk(fmat(sc, t.x, a.x), fmat(sc, t.y, a.y));
}

// LDS plane of a region: one column and row of zeros around it, so that every
// neighbour is a constant offset away (the outermost nodes of a region are
// halo: their results are not used)
template <typename T, int TW, int TH>
using Plane = cx<T>[TH + 2][TW + 2];

// This thread's node.
template <typename T>
struct Node {
    int i, j;        // mesh position (may lie outside the mesh)
    int ic, jc;      // clamped into it
    bool in;         // inside the mesh
    bool keep;       // in the mesh and not on a Dirichlet face: values elsewhere are zero
    bool edge;       // some node of this wavefront lies on or outside the mesh boundary
    T colb, rowb;    // 1 on a boundary column / row, else 0
    cx<T> jf;        // omega / D
    cx<T> kc;        // corner term of the centre (kA or kB)
};

template <typename T, bool DIR>
__device__ __forceinline__ Node<T> node_at(const Op2<T>& L, int i, int j) {
    const int n = L.n;
    Node<T> nd;
    nd.i = i;
    nd.j = j;
    nd.ic = min(max(i, 0), n);
    nd.jc = min(max(j, 0), n);
    nd.in = nd.ic == i && nd.jc == j;
    const bool cb = i == 0 || i == n, rb = j == 0 || j == n, lo = (i == 0) == (j == 0);
    nd.keep = nd.in;
    if (DIR) {
        const unsigned d = L.dir;
        nd.keep = nd.in && !(((d & 1u) && i == 0) || ((d & 2u) && i == n) || ((d & 4u) && j == 0) ||
                             ((d & 8u) && j == n));
    }
    nd.edge = __any((int)(!nd.in || cb || rb));
    nd.colb = cb ? (T)1 : (T)0;
    nd.rowb = rb ? (T)1 : (T)0;
    nd.jf = L.odC;
    nd.kc = zero_cx<T>();
    if (nd.edge) {
        nd.jf = sel(cb && rb, sel(lo, L.odA, L.odB), sel(cb || rb, L.odE, L.odC));
        nd.kc = sel(lo, L.kA, L.kB);
    }
    return nd;
}

// (Op v) at this thread's node, v's plane in s with centre c
template <typename T, int TW, int TH>
__device__ __forceinline__ cx<T> apply_at(const Op2<T>& op, const Plane<T, TW, TH>& s, int lx, int ly,
                                          const Node<T>& nd, cx<T> kc, cx<T> c) {
    const cx<T> ee = s[ly][lx + 1], ww = s[ly][lx - 1], nn = s[ly + 1][lx], ss = s[ly - 1][lx];
    const cx<T> ne = s[ly + 1][lx + 1], sw = s[ly - 1][lx - 1];
    cx<T> acc = cfma(op.wDg, ne + sw, cfma(op.wAx, (ee + ww) + (nn + ss), op.wC * c));
    if (nd.edge) {
        // boundary column, boundary row, corner (zero factors elsewhere)
        acc = axpy_real(nd.colb, cfma(op.dN, nn + ss, op.dC * c), acc);
        acc = axpy_real(nd.rowb, cfma(op.dN, ee + ww, op.dC * c), acc);
        acc = axpy_real(nd.colb * nd.rowb, kc * c, acc);
    }
    return acc;
}

// P^T r at this thread's (even, even) node
template <typename T, int TW, int TH>
__device__ __forceinline__ cx<T> restrict_at(const Plane<T, TW, TH>& s, int lx, int ly, cx<T> c) {
    const cx<T> s6 = ((s[ly][lx + 1] + s[ly][lx - 1]) + (s[ly + 1][lx] + s[ly - 1][lx])) +
                     (s[ly + 1][lx + 1] + s[ly - 1][lx - 1]);
    return axpy_real((T)0.5, s6, c);
}

template <typename T>
__device__ __forceinline__ cx<T> kept(const Node<T>& nd, cx<T> v) {
    return sel(nd.keep, v, zero_cx<T>());
}

template <typename T, int TW, int TH, int THREADS = TW * TH>
__device__ __forceinline__ void clear_rim(Plane<T, TW, TH>& s) {
    for (int q = threadIdx.x; q < 2 * (TW + 2) + 2 * TH; q += THREADS) {
        if (q < 2 * (TW + 2)) s[q < TW + 2 ? 0 : TH + 1][q % (TW + 2)] = zero_cx<T>();
        else s[1 + (q - 2 * (TW + 2)) / 2][(q & 1) ? TW + 1 : 0] = zero_cx<T>();
    }
}

struct TileGrid {
    int tx, ty;  // tiles per side
};

// x <- x_in [+ P e_c]; S Jacobi sweeps; write x, or u += x (UPDATE); with
// RESID also b_c = P^T (b - L x): k_stream_sweeps on tiles.  S = 0: only the
// residual and its restriction.
template <typename T, int TW, int TH, int S, bool PROLONG, bool RESID, bool UPDATE, bool DIR>
__global__ __launch_bounds__(TW * TH) void k_tile_sweeps(Op2<T> L, Vec<const cx<T>> Xin,
                                                         Vec<const cx<T>> Ec, Vec<const cx<T>> Bv,
                                                         Vec<cx<T>> Xout, Vec<cx<T>> Bc, TileGrid g) {
    constexpr int HALO = S + (RESID ? 2 : 0), OW = TW - 2 * HALO, OH = TH - 2 * HALO;
    static_assert(OW > 0 && OH > 0 && OW % 2 == 0 && OH % 2 == 0, "tile too small for its halo");
    __shared__ Plane<T, TW, TH> pl[2];
    const int slot = (int)blockIdx.x / (g.tx * g.ty), b0 = (int)blockIdx.x % (g.tx * g.ty);
    const int x0 = (int)threadIdx.x % TW, y0 = (int)threadIdx.x / TW, lx = x0 + 1, ly = y0 + 1;
    const Node<T> nd = node_at<T, DIR>(L, (b0 % g.tx) * OW - HALO + x0, (b0 / g.tx) * OH - HALO + y0);
    const bool own = nd.in && x0 >= HALO && x0 < TW - HALO && y0 >= HALO && y0 < TH - HALO;
    const long long np = L.n + 1, npc = L.n / 2 + 1, p = (long long)nd.jc * np + nd.ic;
    cx<T>* xo = S > 0 ? Xout.at(slot) : nullptr;
    cx<T> v = Xin.at(slot)[p];
    const cx<T> b = Bv.at(slot)[p];
    cx<T> uo = zero_cx<T>();
    if (UPDATE) uo = xo[p];
    if (PROLONG) {
        const cx<T>* e = Ec.at(slot);
        const long long c0 = (long long)(nd.jc >> 1) * npc + (nd.ic >> 1);
        v = axpy_real((T)0.5, e[c0] + e[c0 + (nd.ic & 1) + (long long)(nd.jc & 1) * npc], v);
    }
    clear_rim<T, TW, TH>(pl[0]);
    clear_rim<T, TW, TH>(pl[1]);
    v = kept(nd, v);
    pl[0][ly][lx] = v;
#pragma unroll
    for (int s = 1; s <= S; ++s) {
        __syncthreads();
        v = kept(nd, cfma(nd.jf, b - apply_at<T, TW, TH>(L, pl[(s - 1) & 1], lx, ly, nd, nd.kc, v), v));
        if (s < S || RESID) pl[s & 1][ly][lx] = v;
    }
    if (S > 0 && own) xo[p] = UPDATE ? uo + v : v;
    if constexpr (RESID) {
        __syncthreads();
        const cx<T> r = kept(nd, b - apply_at<T, TW, TH>(L, pl[S & 1], lx, ly, nd, nd.kc, v));
        pl[(S + 1) & 1][ly][lx] = r;
        __syncthreads();
        if (own && !(nd.i & 1) && !(nd.j & 1))
            Bc.at(slot)[(long long)(nd.j >> 1) * npc + (nd.i >> 1)] =
                kept(nd, restrict_at<T, TW, TH>(pl[(S + 1) & 1], lx, ly, r));
    }
}

// The two zero-guess pre-smoothing sweeps and the residual restriction, with
// b given (HSS = 0), b = rho = c (R - B u) written (1) or b = rho = c R
// written (2): k_stream_pre on tiles.
template <typename T, int TW, int TH, int HSS, bool DIR>
__global__ __launch_bounds__(TW * TH) void k_tile_pre(Op2<T> L, Op2<T> Bs, T c, Vec<const cx<T>> U,
                                                      Vec<const cx<T>> Rv, Vec<cx<T>> Rho,
                                                      Vec<const cx<T>> Bv, Vec<cx<T>> X, Vec<cx<T>> Bc,
                                                      TileGrid g) {
    constexpr int HALO = HSS == 1 ? 4 : 3, OW = (TW - 2 * HALO) & ~1, OH = (TH - 2 * HALO) & ~1;
    static_assert(OW > 0 && OH > 0, "tile too small for its halo");
    __shared__ Plane<T, TW, TH> pl[2];
    const int slot = (int)blockIdx.x / (g.tx * g.ty), b0 = (int)blockIdx.x % (g.tx * g.ty);
    const int x0 = (int)threadIdx.x % TW, y0 = (int)threadIdx.x / TW, lx = x0 + 1, ly = y0 + 1;
    const Node<T> nd = node_at<T, DIR>(L, (b0 % g.tx) * OW - HALO + x0, (b0 / g.tx) * OH - HALO + y0);
    const bool own = nd.in && x0 >= HALO && x0 < HALO + OW && y0 >= HALO && y0 < HALO + OH;
    const long long np = L.n + 1, npc = L.n / 2 + 1, p = (long long)nd.jc * np + nd.ic;
    cx<T> b = (HSS == 0 ? Bv.at(slot) : Rv.at(slot))[p];
    cx<T> u = zero_cx<T>();
    if (HSS == 1) u = U.at(slot)[p];
    clear_rim<T, TW, TH>(pl[0]);
    clear_rim<T, TW, TH>(pl[1]);
    if (HSS == 1) {
        u = sel(nd.in, u, zero_cx<T>());
        pl[1][ly][lx] = u;
        __syncthreads();
        b = c * (b - apply_at<T, TW, TH>(Bs, pl[1], lx, ly, nd, sel((nd.i == 0) == (nd.j == 0), Bs.kA, Bs.kB), u));
    } else if (HSS == 2) {
        b = c * b;
    }
    if (DIR) b = sel(nd.in && !nd.keep, zero_cx<T>(), b);
    if (HSS != 0 && own) Rho.at(slot)[p] = b;
    cx<T> v = kept(nd, nd.jf * b);
    pl[0][ly][lx] = v;
    __syncthreads();
    v = kept(nd, cfma(nd.jf, b - apply_at<T, TW, TH>(L, pl[0], lx, ly, nd, nd.kc, v), v));
    if (own) X.at(slot)[p] = v;
    pl[1][ly][lx] = v;
    __syncthreads();
    const cx<T> r = kept(nd, b - apply_at<T, TW, TH>(L, pl[1], lx, ly, nd, nd.kc, v));
    pl[0][ly][lx] = r;
    __syncthreads();
    if (own && !(nd.i & 1) && !(nd.j & 1))
        Bc.at(slot)[(long long)(nd.j >> 1) * npc + (nd.i >> 1)] =
            kept(nd, restrict_at<T, TW, TH>(pl[0], lx, ly, r));
}

// Pre-smoothing of two consecutive levels from zero guesses in one launch: on
// the fine level x, the residual and its restriction b_c; on the coarse one
// x_c from b_c, and b_cc = P^T (b_c - L_c x_c).  k_tile_pre twice, without the
// second launch and the trip of b_c through memory.  The coarse pass needs
// three coarse nodes around the ones it owns and the fine one three fine nodes
// around those, so a 32 x 32 region owns only 12 x 12 fine nodes: worth it
// while most compute units would idle.
constexpr int PAIR = 32, PAIR_C = PAIR / 2;  // fine and coarse nodes of a region's side
constexpr int PRE2_HALO = 6;                 // coarse nodes before the first owned one
constexpr int PRE2_OWN = 6;                  // owned coarse nodes (12 fine ones)

template <typename T, bool DIR>
__global__ __launch_bounds__(PAIR * PAIR) void k_tile_pre2(Op2<T> L, Op2<T> Lc, Vec<const cx<T>> Bv,
                                                           Vec<cx<T>> X, Vec<cx<T>> Bc, Vec<cx<T>> Xc,
                                                           Vec<cx<T>> Bcc, TileGrid g) {
    __shared__ Plane<T, PAIR, PAIR> pl[2];
    __shared__ Plane<T, PAIR_C, PAIR_C> pc[2];
    const int slot = (int)blockIdx.x / (g.tx * g.ty), b0 = (int)blockIdx.x % (g.tx * g.ty);
    const int c0x = (b0 % g.tx) * PRE2_OWN - PRE2_HALO, c0y = (b0 / g.tx) * PRE2_OWN - PRE2_HALO;
    constexpr int O0 = PRE2_HALO, O1 = PRE2_HALO + PRE2_OWN;  // owned coarse nodes of the region
    const int tid = (int)threadIdx.x;
    const int x0 = tid % PAIR, y0 = tid / PAIR, lx = x0 + 1, ly = y0 + 1;
    const Node<T> nd = node_at<T, DIR>(L, 2 * c0x + x0, 2 * c0y + y0);
    const long long np = L.n + 1, npc = Lc.n + 1, npcc = Lc.n / 2 + 1, p = (long long)nd.jc * np + nd.ic;
    cx<T> b = Bv.at(slot)[p];
    clear_rim<T, PAIR, PAIR>(pl[0]);
    clear_rim<T, PAIR, PAIR>(pl[1]);
    clear_rim<T, PAIR_C, PAIR_C, PAIR * PAIR>(pc[0]);
    clear_rim<T, PAIR_C, PAIR_C, PAIR * PAIR>(pc[1]);
    if (DIR) b = sel(nd.in && !nd.keep, zero_cx<T>(), b);
    cx<T> v = kept(nd, nd.jf * b);
    pl[0][ly][lx] = v;
    __syncthreads();
    v = kept(nd, cfma(nd.jf, b - apply_at<T, PAIR, PAIR>(L, pl[0], lx, ly, nd, nd.kc, v), v));
    if (nd.in && x0 >= 2 * O0 && x0 < 2 * O1 && y0 >= 2 * O0 && y0 < 2 * O1) X.at(slot)[p] = v;
    pl[1][ly][lx] = v;
    __syncthreads();
    pl[0][ly][lx] = kept(nd, b - apply_at<T, PAIR, PAIR>(L, pl[1], lx, ly, nd, nd.kc, v));
    __syncthreads();
    // the coarse level: one node per thread of the first four wavefronts
    const bool act = tid < PAIR_C * PAIR_C;
    const int cx0 = tid % PAIR_C, cy0 = tid / PAIR_C, cu = cx0 + 1, cv = cy0 + 1;
    const Node<T> nc = node_at<T, DIR>(Lc, c0x + cx0, c0y + cy0);
    const bool own = act && nc.in && cx0 >= O0 && cx0 < O1 && cy0 >= O0 && cy0 < O1;
    const long long pcn = (long long)nc.jc * npc + nc.ic;
    b = zero_cx<T>();
    if (act) {
        b = kept(nc, restrict_at<T, PAIR, PAIR>(pl[0], 2 * cx0 + 1, 2 * cy0 + 1, pl[0][2 * cy0 + 1][2 * cx0 + 1]));
        if (own) Bc.at(slot)[pcn] = b;
        v = kept(nc, nc.jf * b);
        pc[0][cv][cu] = v;
    }
    __syncthreads();
    if (act) {
        v = kept(nc, cfma(nc.jf, b - apply_at<T, PAIR_C, PAIR_C>(Lc, pc[0], cu, cv, nc, nc.kc, v), v));
        if (own) Xc.at(slot)[pcn] = v;
        pc[1][cv][cu] = v;
    }
    __syncthreads();
    cx<T> r = zero_cx<T>();
    if (act) {
        r = kept(nc, b - apply_at<T, PAIR_C, PAIR_C>(Lc, pc[1], cu, cv, nc, nc.kc, v));
        pc[0][cv][cu] = r;
    }
    __syncthreads();
    if (own && !(nc.i & 1) && !(nc.j & 1))
        Bcc.at(slot)[(long long)(nc.j >> 1) * npcc + (nc.i >> 1)] =
            kept(nc, restrict_at<T, PAIR_C, PAIR_C>(pc[0], cu, cv, r));
}

// Post-smoothing of two consecutive levels in one launch: x_c + P e_cc and two
// sweeps on the coarse level, whose result is used here only (e_c), then
// x + P e_c and S sweeps on the fine one, written or added into u (UPDATE),
// and with RESID b_c = P^T (b - L x) into Bcout, another buffer than Bc, which
// other workgroups still read.  A TW x TH fine region needs the coarse result
// on the TW / 2 + 1 by TH / 2 + 1 coarse nodes that cover it, and two more on
// each side to compute it.
template <typename T, int TW, int TH, int S, bool RESID, bool UPDATE, bool DIR>
__global__ __launch_bounds__(TW * TH) void k_tile_post2(Op2<T> L, Op2<T> Lc, Vec<const cx<T>> Xin,
                                                        Vec<const cx<T>> Bv, Vec<const cx<T>> Xc,
                                                        Vec<const cx<T>> Bc, Vec<const cx<T>> Ecc,
                                                        Vec<cx<T>> Xout, Vec<cx<T>> Bcout, TileGrid g) {
    constexpr int HALO = S + (RESID ? 2 : 0), OW = TW - 2 * HALO, OH = TH - 2 * HALO;
    constexpr int CW = TW / 2 + 5, CH = TH / 2 + 5;
    static_assert(CW * CH <= TW * TH, "one coarse node per thread at most");
    static_assert(HALO % 2 == 0 && OW > 0 && OH > 0 && OW % 2 == 0 && OH % 2 == 0, "even regions");
    __shared__ Plane<T, TW, TH> pl[2];
    __shared__ Plane<T, CW, CH> pc[2];
    const int slot = (int)blockIdx.x / (g.tx * g.ty), b0 = (int)blockIdx.x % (g.tx * g.ty);
    const int tid = (int)threadIdx.x, x0 = tid % TW, y0 = tid / TW, lx = x0 + 1, ly = y0 + 1;
    const int fx = (b0 % g.tx) * OW - HALO, fy = (b0 / g.tx) * OH - HALO;  // both even
    const Node<T> nd = node_at<T, DIR>(L, fx + x0, fy + y0);
    const bool own = nd.in && x0 >= HALO && x0 < TW - HALO && y0 >= HALO && y0 < TH - HALO;
    const bool act = tid < CW * CH;
    const int cx0 = tid % CW, cy0 = tid / CW, cu = cx0 + 1, cv = cy0 + 1;
    const Node<T> nc = node_at<T, DIR>(Lc, fx / 2 - 2 + cx0, fy / 2 - 2 + cy0);
    const long long np = L.n + 1, npc = Lc.n + 1, npcc = Lc.n / 2 + 1, p = (long long)nd.jc * np + nd.ic;
    cx<T> v = Xin.at(slot)[p];
    const cx<T> b = Bv.at(slot)[p];
    cx<T>* xo = Xout.at(slot);
    cx<T> uo = zero_cx<T>();
    if (UPDATE) uo = xo[p];
    cx<T> vc = zero_cx<T>(), bc = zero_cx<T>();
    if (act) {
        const long long q = (long long)nc.jc * npc + nc.ic;
        const long long c0 = (long long)(nc.jc >> 1) * npcc + (nc.ic >> 1);
        const cx<T>* e = Ecc.at(slot);
        vc = Xc.at(slot)[q];
        bc = Bc.at(slot)[q];
        vc = kept(nc, axpy_real((T)0.5, e[c0] + e[c0 + (nc.ic & 1) + (long long)(nc.jc & 1) * npcc], vc));
        pc[0][cv][cu] = vc;
    }
    clear_rim<T, TW, TH>(pl[0]);
    clear_rim<T, TW, TH>(pl[1]);
    clear_rim<T, CW, CH, TW * TH>(pc[0]);
    clear_rim<T, CW, CH, TW * TH>(pc[1]);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        __syncthreads();
        if (act) {
            vc = kept(nc, cfma(nc.jf, bc - apply_at<T, CW, CH>(Lc, pc[s], cu, cv, nc, nc.kc, vc), vc));
            pc[1 - s][cv][cu] = vc;
        }
    }
    __syncthreads();
    const int eu = (x0 >> 1) + 3, ev = (y0 >> 1) + 3;
    v = kept(nd, axpy_real((T)0.5, pc[0][ev][eu] + pc[0][ev + (y0 & 1)][eu + (x0 & 1)], v));
    pl[0][ly][lx] = v;
#pragma unroll
    for (int s = 1; s <= S; ++s) {
        __syncthreads();
        v = kept(nd, cfma(nd.jf, b - apply_at<T, TW, TH>(L, pl[(s - 1) & 1], lx, ly, nd, nd.kc, v), v));
        if (s < S || RESID) pl[s & 1][ly][lx] = v;
    }
    if (own) xo[p] = UPDATE ? uo + v : v;
    if constexpr (RESID) {
        __syncthreads();
        const cx<T> r = kept(nd, b - apply_at<T, TW, TH>(L, pl[S & 1], lx, ly, nd, nd.kc, v));
        pl[(S + 1) & 1][ly][lx] = r;
        __syncthreads();
        if (own && !(nd.i & 1) && !(nd.j & 1))
            Bcout.at(slot)[(long long)(nd.j >> 1) * npc + (nd.i >> 1)] =
                kept(nd, restrict_at<T, TW, TH>(pl[(S + 1) & 1], lx, ly, r));
    }
}

constexpr int TW = 32;  // tile columns

inline TileGrid tile_grid(int n, int halo, int th) {
    const int ow = (TW - 2 * halo) & ~1, oh = (th - 2 * halo) & ~1;
    return TileGrid{(n + ow) / ow, (n + oh) / oh};
}

// Tile height for a pass of the given halo on a mesh of n cells and ns
// columns: 16 rows (512 threads, the shorter stages) while that many
// workgroups stay within about `most16`, then 32 rows (1024 threads, less
// halo) up to `most32` workgroups, else 0: the streaming kernel, whose
// wavefronts then fill the chip and recompute less halo.  Measured (us per
// launch, FP64, streaming / 16 rows / 32 rows):
//   four sweeps + restriction   128^2 20.2 / 4.6 / 5.9,  256^2 20.4 / 8.2 / 6.2,
//                               512^2 22.0 / 21.5 / 14.1, 4 x 512^2 38.6 / 73 / 47
//   HSS residual + pre          128^2 13.2 / 4.0 / 5.1,  352^2 14.1 / 6.3 / 5.7,
//                               1024^2 25.8 / 26.9 / 28.4
//   pre + restriction           128^2 6.2 / 3.5 / 4.3,   512^2 7.1 / 6.5 / 6.3,
//                               4 x 352^2 9.0 / 9.7 / 9.6
//   prolongation + two sweeps   128^2 5.2 / 3.4 / 4.1,   4 x 256^2 6.9 / 5.7 / 6.1,
//                               4 x 352^2 8.4 / 8.7 / 8.7
// (FP32 crosses over at the same sizes.)
int tile_height(int n, int halo, int ns, int most16, int most32) {
    const TileGrid g16 = tile_grid(n, halo, 16), g32 = tile_grid(n, halo, 32);
    if ((long long)g16.tx * g16.ty * ns <= most16) return 16;
    if ((long long)g32.tx * g32.ty * ns <= most32) return 32;
    return 0;
}

// Most workgroups of the two-level passes: the down pass while each has a
// compute unit to itself, the up pass up to about four per compute unit (its
// halo is small).  Measured (us per launch, FP64; FP32 in parentheses; the two
// launches that it replaces, without the 1 us between them):
//   down  92^2 6.3 (5.0) : 3.8 + 3.7,   128^2 5.9 (5.1) : 4.1 + 4.0,
//         4 x 92^2 6.6 (5.3) : 4.4 + 3.9,   256^2 (484) 11.3 (9.8) : 4.4 + 4.0
//   up    92^2 5.4 (4.7) : 3.7 + 3.7,   256^2 5.8 (5.0) : 4.0 + 3.9,
//         512^2 (817) 10.0 (8.0) : 6.5 + 4.0,   8 x 176^2 (1560) 15.4 : 9.0 + 6.0
constexpr int PRE2_MOST = 256, POST2_MOST = 1024;
// With the finest level's four-sweep pass, 32 rows up to 400 workgroups (16 as
// that pass alone):
//   128^2 (231, FP32) 6.0 : 4.2 + 3.3,   256^2 (169) 8.6 (7.2) : 7.0 + 3.9 (5.7 + 3.3),
//   2 x 256^2 (338) 14.2 (10.9) : 11.5 + 4.0 (7.9 + 3.5),
//   512^2 (676) 20.2 (15.8) : 15.8 + 4.0 (10.7 + 4.0)
constexpr int POST4_MOST16 = 256, POST4_MOST32 = 400;

}  // namespace

template <typename T>
bool tile_sweeps_2d(hipStream_t st, const Op2<T>& L, int S, Vec<const cx<T>> Xin, Vec<const cx<T>> Ec,
                    Vec<const cx<T>> B, Vec<cx<T>> Xout, Vec<cx<T>> Bc, bool update, int ns) {
    const bool pro = Ec.base != nullptr, resid = Bc.base != nullptr;
    const bool s4 = S == 4 && pro && resid && !update, s2 = S == 2 && pro && !resid;
    if (!s4 && !s2) return false;
    const int halo = s4 ? 6 : 2;
    const int th = s4 ? tile_height(L.n, halo, ns, 256, 1100) : tile_height(L.n, halo, ns, 1024, 0);
    if (th == 0) return false;
    const TileGrid g = tile_grid(L.n, halo, th);
    const unsigned nb = (unsigned)(g.tx * g.ty * ns);
#define HELM_TILE(HH, SS, RR, UU)                                                                   \
    do {                                                                                            \
        if (L.dir) k_tile_sweeps<T, TW, HH, SS, true, RR, UU, true><<<nb, TW * HH, 0, st>>>(L, Xin, Ec, B, Xout, Bc, g); \
        else k_tile_sweeps<T, TW, HH, SS, true, RR, UU, false><<<nb, TW * HH, 0, st>>>(L, Xin, Ec, B, Xout, Bc, g); \
    } while (0)
    if (s4 && th == 16) HELM_TILE(16, 4, true, false);
    else if (s4) HELM_TILE(32, 4, true, false);
    else if (update) HELM_TILE(16, 2, false, true);
    else HELM_TILE(16, 2, false, false);
#undef HELM_TILE
    return true;
}

template <typename T>
void tile_restrict_2d(hipStream_t st, const Op2<T>& L, Vec<const cx<T>> X, Vec<const cx<T>> B, Vec<cx<T>> Bc, int ns) {
    const TileGrid g = tile_grid(L.n, 2, 16);
    const unsigned nb = (unsigned)(g.tx * g.ty * ns);
    const Vec<const cx<T>> none{};
    const Vec<cx<T>> nil{};
    k_tile_sweeps<T, TW, 16, 0, false, true, false, false><<<nb, TW * 16, 0, st>>>(L, X, none, B, nil, Bc, g);
}

template <typename T>
bool tile_pre_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Bs, T c, Vec<const cx<T>> U,
                 Vec<const cx<T>> R, Vec<cx<T>> Rho, Vec<const cx<T>> B, Vec<cx<T>> X, Vec<cx<T>> Bc,
                 int ns) {
    const int hss = B.base ? 0 : (U.base ? 1 : 2);
    const int halo = hss == 1 ? 4 : 3;
    const int th = hss == 1 ? tile_height(L.n, halo, ns, 448, 1024) : tile_height(L.n, halo, ns, 512, 512);
    if (th == 0) return false;
    const TileGrid g = tile_grid(L.n, halo, th);
    const unsigned nb = (unsigned)(g.tx * g.ty * ns);
#define HELM_TPRE(HH, SS)                                                                             \
    do {                                                                                              \
        if (L.dir) k_tile_pre<T, TW, HH, SS, true><<<nb, TW * HH, 0, st>>>(L, Bs, c, U, R, Rho, B, X, Bc, g); \
        else k_tile_pre<T, TW, HH, SS, false><<<nb, TW * HH, 0, st>>>(L, Bs, c, U, R, Rho, B, X, Bc, g); \
    } while (0)
    if (th == 16) {
        if (hss == 0) HELM_TPRE(16, 0);
        else if (hss == 1) HELM_TPRE(16, 1);
        else HELM_TPRE(16, 2);
    } else {
        if (hss == 0) HELM_TPRE(32, 0);
        else if (hss == 1) HELM_TPRE(32, 1);
        else HELM_TPRE(32, 2);
    }
#undef HELM_TPRE
    return true;
}

template <typename T>
bool tile_pre_pair_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Lc, Vec<const cx<T>> B, Vec<cx<T>> X,
                      Vec<cx<T>> Bc, Vec<cx<T>> Xc, Vec<cx<T>> Bcc, int ns) {
    const int t = (L.n / 2 + PRE2_OWN) / PRE2_OWN;
    const TileGrid g{t, t};
    if ((long long)t * t * ns > PRE2_MOST) return false;
    const unsigned nb = (unsigned)(t * t * ns);
    if (L.dir) k_tile_pre2<T, true><<<nb, PAIR * PAIR, 0, st>>>(L, Lc, B, X, Bc, Xc, Bcc, g);
    else k_tile_pre2<T, false><<<nb, PAIR * PAIR, 0, st>>>(L, Lc, B, X, Bc, Xc, Bcc, g);
    return true;
}

template <typename T>
bool tile_post_pair_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Lc, int S, Vec<const cx<T>> X,
                       Vec<const cx<T>> B, Vec<const cx<T>> Xc, Vec<const cx<T>> Bc, Vec<const cx<T>> Ecc,
                       Vec<cx<T>> Xout, Vec<cx<T>> Bcout, bool update, int ns) {
    const bool s4 = S == 4;  // with the restriction
    const int th = s4 ? tile_height(L.n, 6, ns, POST4_MOST16, POST4_MOST32) : tile_height(L.n, 2, ns, POST2_MOST, 0);
    if (th == 0) return false;
    const TileGrid g = tile_grid(L.n, s4 ? 6 : 2, th);
    const unsigned nb = (unsigned)(g.tx * g.ty * ns);
#define HELM_POST2(HH, SS, RR, UU)                                                                  \
    do {                                                                                            \
        if (L.dir) k_tile_post2<T, TW, HH, SS, RR, UU, true><<<nb, TW * HH, 0, st>>>(L, Lc, X, B, Xc, Bc, Ecc, Xout, Bcout, g); \
        else k_tile_post2<T, TW, HH, SS, RR, UU, false><<<nb, TW * HH, 0, st>>>(L, Lc, X, B, Xc, Bc, Ecc, Xout, Bcout, g); \
    } while (0)
    if (s4 && th == 16) HELM_POST2(16, 4, true, false);
    else if (s4) HELM_POST2(32, 4, true, false);
    else if (update) HELM_POST2(16, 2, false, true);
    else HELM_POST2(16, 2, false, false);
#undef HELM_POST2
    return true;
}

template bool tile_sweeps_2d<double>(hipStream_t, const Op2<double>&, int, Vec<const cxd>, Vec<const cxd>,
                                     Vec<const cxd>, Vec<cxd>, Vec<cxd>, bool, int);
template bool tile_sweeps_2d<float>(hipStream_t, const Op2<float>&, int, Vec<const cxf>, Vec<const cxf>,
                                    Vec<const cxf>, Vec<cxf>, Vec<cxf>, bool, int);
template void tile_restrict_2d<double>(hipStream_t, const Op2<double>&, Vec<const cxd>, Vec<const cxd>, Vec<cxd>, int);
template void tile_restrict_2d<float>(hipStream_t, const Op2<float>&, Vec<const cxf>, Vec<const cxf>, Vec<cxf>, int);
template bool tile_pre_2d<double>(hipStream_t, const Op2<double>&, const Op2<double>&, double,
                                  Vec<const cxd>, Vec<const cxd>, Vec<cxd>, Vec<const cxd>, Vec<cxd>,
                                  Vec<cxd>, int);
template bool tile_pre_2d<float>(hipStream_t, const Op2<float>&, const Op2<float>&, float, Vec<const cxf>,
                                 Vec<const cxf>, Vec<cxf>, Vec<const cxf>, Vec<cxf>, Vec<cxf>, int);

template bool tile_pre_pair_2d<double>(hipStream_t, const Op2<double>&, const Op2<double>&, Vec<const cxd>, Vec<cxd>, Vec<cxd>,
                                      Vec<cxd>, Vec<cxd>, int);
template bool tile_post_pair_2d<double>(hipStream_t, const Op2<double>&, const Op2<double>&, int, Vec<const cxd>, Vec<const cxd>,
                                       Vec<const cxd>, Vec<const cxd>, Vec<const cxd>, Vec<cxd>, Vec<cxd>, bool, int);
template bool tile_pre_pair_2d<float>(hipStream_t, const Op2<float>&, const Op2<float>&, Vec<const cxf>, Vec<cxf>, Vec<cxf>,
                                      Vec<cxf>, Vec<cxf>, int);
template bool tile_post_pair_2d<float>(hipStream_t, const Op2<float>&, const Op2<float>&, int, Vec<const cxf>, Vec<const cxf>,
                                       Vec<const cxf>, Vec<const cxf>, Vec<const cxf>, Vec<cxf>, Vec<cxf>, bool, int);

}  // namespace helm
