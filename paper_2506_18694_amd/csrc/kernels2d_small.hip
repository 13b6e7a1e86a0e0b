// One V-cycle over the small 2D levels in a single workgroup per right-hand
// side, with every level's vectors resident in LDS.
//
// The coarse levels of the hierarchy have too few nodes to fill the GPU;
// launched one kernel per smoothing / transfer pass, each costs a fixed few
// microseconds of latency regardless of its size.  This kernel runs the
// whole zero-guess V(2,2) cycle below a given level - pre-smoothing,
// residual restriction, the dense FP64 coarsest solve, prolongation and
// post-smoothing on every small level - in one launch, one workgroup per
// right-hand side, synchronising with workgroup barriers instead.
//
// Its time is the chain of about 14 barrier-separated stages (33^2, 17^2 and
// 9^2 levels), so a stage is kept short: a level's plane carries a rim of
// zeros, so that no neighbour read needs a test; a boundary node has its own
// row weights, so that every node runs the same 22 operations; the finest
// small level keeps its right-hand side, iterate and weights in registers
// (three nodes per thread); and the first zero-guess iterate of a level is
// formed with its restricted right-hand side.  512 threads, because the
// stages of the 17^2 level and below have 1 to 5 wavefronts of work.
// Measured from 33^2 down to 9^2 at 4 columns: 17.5 -> 9.4 us in FP64,
// at 1 column in FP32 13.4 -> 10.7.
#include "launch.h"
#include "stencil_rows.h"

namespace helm {

namespace {

constexpr int NTS = SMALL_THREADS;
constexpr int NPT = SMALL_NODES;  // nodes per thread on the finest small level

template <typename T>
__device__ __forceinline__ cx<T> zero_c() { return mk((T)0, (T)0); }

template <typename T>
__device__ __forceinline__ cx<T> sel(bool c, cx<T> a, cx<T> b) {
    return mk(c ? a.x : b.x, c ? a.y : b.y);
}

// a + s t for a real s
template <typename T>
__device__ __forceinline__ cx<T> axpy_real(T sc, cx<T> t, cx<T> a) {
    return mk(fmat(sc, t.x, a.x), fmat(sc, t.y, a.y));
}

// Node q of a level with W = n + 1 nodes per row: (i, j) = (q mod W, q div W)
// by a multiply with md = ceil(2^20 / W), exact while q W <= 2^20; its place
// p in the level's padded plane, and its row of the operator: centre, east /
// west, north / south and Jacobi factor (the "/" diagonal's weight is the
// same on every node).
template <typename T>
struct Node {
    int i, j, p, s;  // s: row stride of the plane
    cx<T> c, x, y, jf;
};
template <typename T>
__device__ __forceinline__ Node<T> node_of(const Op2<T>& op, int q, int md) {
    const int n = op.n, W = n + 1;
    Node<T> nd;
    nd.j = (int)(((unsigned)q * (unsigned)md) >> 20);
    nd.i = q - nd.j * W;
    nd.s = n + 3;
    nd.p = (nd.j + 1) * nd.s + nd.i + 1;
    const bool cb = (nd.i == 0) | (nd.i == n), rb = (nd.j == 0) | (nd.j == n);
    const bool lo = (nd.i == 0) == (nd.j == 0);
    // an edge misses dC on the centre and dN along it; a corner kA or kB more
    const cx<T> z = zero_c<T>();
    nd.c = op.wC + sel(cb, op.dC, z) + sel(rb, op.dC, z) + sel(cb & rb, sel(lo, op.kA, op.kB), z);
    nd.y = op.wAx + sel(cb, op.dN, z);
    nd.x = op.wAx + sel(rb, op.dN, z);
    nd.jf = sel(cb & rb, sel(lo, op.odA, op.odB), sel(cb | rb, op.odE, op.odC));
    return nd;
}

// (Op s) at a node whose value is c
template <typename T>
__device__ __forceinline__ cx<T> apply_at(cx<T> wDg, const cx<T>* s, const Node<T>& nd, cx<T> c) {
    const cx<T>* q = s + nd.p;
    const int S = nd.s;
    return cfma(wDg, q[S + 1] + q[-S - 1],
                cfma(nd.x, q[1] + q[-1], cfma(nd.y, q[S] + q[-S], nd.c * c)));
}

// b_c = P^T r at coarse node (I, J): the fine residual at (2I, 2J) plus half
// of it at its six neighbours (zero outside the mesh)
template <typename T>
__device__ __forceinline__ cx<T> restrict_at(const cx<T>* r, int n, int I, int J) {
    const int S = n + 3;
    const cx<T>* q = r + (2 * J + 1) * S + 2 * I + 1;
    const cx<T> sum = ((q[1] + q[-1]) + (q[S] + q[-S])) + (q[S + 1] + q[-S - 1]);
    return axpy_real((T)0.5, sum, q[0]);
}

// x + P e at a fine node, e the coarse plane of nc = n / 2 cells
template <typename T>
__device__ __forceinline__ cx<T> prolonged(const cx<T>* e, int n, const Node<T>& nd, cx<T> x) {
    const int S = n / 2 + 3;
    const cx<T>* q = e + ((nd.j >> 1) + 1) * S + (nd.i >> 1) + 1;
    return axpy_real((T)0.5, q[0] + q[(nd.i & 1) + (nd.j & 1) * S], x);
}

template <typename T>
__global__ __launch_bounds__(NTS) void k_vcycle_small(SmallCycle<T> sc, const cxd* __restrict__ Ainv,
                                                      int nc, Vec<const cx<T>> Bin, Vec<cx<T>> Xout) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    cx<T>* lds = reinterpret_cast<cx<T>*>(lds_raw);
    const int slot = blockIdx.x;
    const int tid = threadIdx.x;
    const int L = sc.nlev;
    // finest small level: this thread's right-hand side values
    const Op2<T>& op0 = sc.op[0];
    const int n0 = op0.n, N0 = (n0 + 1) * (n0 + 1);
    const cx<T>* bin = Bin.at(slot);
    cx<T> b0[NPT], x0[NPT];
    Node<T> nd0[NPT];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        const int q = tid + u * NTS;
        b0[u] = bin[q < N0 ? q : 0];
    }
    // coarsest solve x = Ainv b in FP64: thread (r, g) forms the partial sum
    // of row r over the columns g, g + G, ...; its first CW entries of Ainv
    // are loaded now so that their latency is hidden behind the descent
    constexpr int CW = 16;
    const int G = nc < NTS ? NTS / nc : 1;
    const int cr = tid / G, cg = tid % G;
    const bool crow = cr < nc;
    cxd av[CW];
#pragma unroll
    for (int u = 0; u < CW; ++u) {
        const int cc = cg + u * G;
        av[u] = (crow && cc < nc) ? Ainv[(long long)cr * nc + cc] : mk(0.0, 0.0);
    }
    // the rims of all planes (and everything else) start at zero
    for (int q = tid; q < sc.total; q += NTS) lds[q] = zero_c<T>();
    __syncthreads();
    cx<T>* const A0 = lds + sc.off_a[0];
    cx<T>* const X0 = lds + sc.off_x[0];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        const int q = tid + u * NTS;
        nd0[u] = node_of(op0, q < N0 ? q : 0, sc.mdiv[0]);
        x0[u] = nd0[u].jf * b0[u];
        if (q < N0) A0[nd0[u].p] = x0[u];
    }
    __syncthreads();
    // a Jacobi sweep of the finest small level from plane `from` (whose
    // values at this thread's nodes are x0) to plane `to`
    auto sweep0 = [&](const cx<T>* from, cx<T>* to) {
#pragma unroll
        for (int u = 0; u < NPT; ++u) {
            if (tid + u * NTS >= N0) continue;
            x0[u] = cfma(nd0[u].jf, b0[u] - apply_at(op0.wDg, from, nd0[u], x0[u]), x0[u]);
            to[nd0[u].p] = x0[u];
        }
        __syncthreads();
    };
    sweep0(A0, X0);
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        if (tid + u * NTS >= N0) continue;
        A0[nd0[u].p] = b0[u] - apply_at(op0.wDg, X0, nd0[u], x0[u]);
    }
    __syncthreads();
    // restriction to level l + 1: its right-hand side and (unless it is the
    // coarsest) its first pre-smoothing iterate
    auto down = [&](int l) {
        const Op2<T>& opc = sc.op[l + 1];
        const int Wc = opc.n + 1;
        if (tid < Wc * Wc) {
            const Node<T> nd = node_of(opc, tid, sc.mdiv[l + 1]);
            const cx<T> b = restrict_at(lds + sc.off_a[l], sc.op[l].n, nd.i, nd.j);
            lds[sc.off_b[l + 1] + tid] = b;
            if (l + 1 < L - 1) lds[sc.off_a[l + 1] + nd.p] = nd.jf * b;
        }
        __syncthreads();
    };
    down(0);
    for (int l = 1; l < L - 1; ++l) {
        const Op2<T>& op = sc.op[l];
        const bool on = tid < (op.n + 1) * (op.n + 1);
        const Node<T> nd = node_of(op, on ? tid : 0, sc.mdiv[l]);
        cx<T>* A = lds + sc.off_a[l];
        cx<T>* X = lds + sc.off_x[l];
        const cx<T> b = lds[sc.off_b[l] + (on ? tid : 0)];
        cx<T> x = A[nd.p];
        x = cfma(nd.jf, b - apply_at(op.wDg, A, nd, x), x);
        if (on) X[nd.p] = x;
        __syncthreads();
        if (on) A[nd.p] = b - apply_at(op.wDg, X, nd, x);
        __syncthreads();
        down(l);
    }
    // coarsest: the partials meet in the scratch area, then one thread per
    // row adds its G partials in a fixed order
    {
        const cx<T>* B = lds + sc.off_b[L - 1];
        cxd* part = reinterpret_cast<cxd*>(lds + sc.off_part);
        if (crow) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int u = 0; u < CW; ++u) {
                const int cc = cg + u * G;
                if (cc < nc) {
                    const cxd bv = cvt<double>(B[cc]);
                    re = fma(av[u].x, bv.x, fma(-av[u].y, bv.y, re));
                    im = fma(av[u].x, bv.y, fma(av[u].y, bv.x, im));
                }
            }
            for (int cc = cg + CW * G; cc < nc; cc += G) {
                const cxd a = Ainv[(long long)cr * nc + cc];
                const cxd bv = cvt<double>(B[cc]);
                re = fma(a.x, bv.x, fma(-a.y, bv.y, re));
                im = fma(a.x, bv.y, fma(a.y, bv.x, im));
            }
            part[tid] = mk(re, im);
        }
        __syncthreads();
        if (tid < nc) {
            double re = 0.0, im = 0.0;
            for (int q = 0; q < G; ++q) {
                re += part[tid * G + q].x;
                im += part[tid * G + q].y;
            }
            lds[sc.off_x[L - 1] + node_of(sc.op[L - 1], tid, sc.mdiv[L - 1]).p] = mk((T)re, (T)im);
        }
        __syncthreads();
    }
    // up: prolongate and correct, post-smooth twice
    for (int l = L - 2; l > 0; --l) {
        const Op2<T>& op = sc.op[l];
        const bool on = tid < (op.n + 1) * (op.n + 1);
        const Node<T> nd = node_of(op, on ? tid : 0, sc.mdiv[l]);
        cx<T>* A = lds + sc.off_a[l];
        cx<T>* X = lds + sc.off_x[l];
        const cx<T> b = lds[sc.off_b[l] + (on ? tid : 0)];
        cx<T> x = prolonged(lds + sc.off_x[l + 1], op.n, nd, X[nd.p]);
        if (on) X[nd.p] = x;
        __syncthreads();
        x = cfma(nd.jf, b - apply_at(op.wDg, X, nd, x), x);
        if (on) A[nd.p] = x;
        __syncthreads();
        x = cfma(nd.jf, b - apply_at(op.wDg, A, nd, x), x);
        if (on) X[nd.p] = x;
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        if (tid + u * NTS >= N0) continue;
        x0[u] = prolonged(lds + sc.off_x[1], n0, nd0[u], x0[u]);
        X0[nd0[u].p] = x0[u];
    }
    __syncthreads();
    sweep0(X0, A0);
    // the last sweep goes straight to memory
    cx<T>* xo = Xout.at(slot);
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        const int q = tid + u * NTS;
        if (q < N0) xo[q] = cfma(nd0[u].jf, b0[u] - apply_at(op0.wDg, A0, nd0[u], x0[u]), x0[u]);
    }
}

}  // namespace

template <typename T>
void vcycle_small(hipStream_t st, const SmallCycle<T>& sc, size_t lds_bytes, const cxd* Ainv,
                  int nc, Vec<const cx<T>> B, Vec<cx<T>> X, int ns) {
    k_vcycle_small<T><<<ns, NTS, lds_bytes, st>>>(sc, Ainv, nc, B, X);
}

template void vcycle_small<double>(hipStream_t, const SmallCycle<double>&, size_t, const cxd*,
                                   int, Vec<const cxd>, Vec<cxd>, int);
template void vcycle_small<float>(hipStream_t, const SmallCycle<float>&, size_t, const cxd*, int,
                                  Vec<const cxf>, Vec<cxf>, int);

}  // namespace helm
