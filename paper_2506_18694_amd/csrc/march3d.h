// Fused z-marching passes for the 3D Q1 levels (included with contraction
// switched off, see planes3d.h).
//
// Every operator a K + b M + c M_Gamma on the uniform hexahedral mesh is a
// sum of tensor products of the 1D linear-element rows (K1 = (1/h)[-1 2 -1],
// M1 = (h/6)[1 4 1]; a boundary row halves the centre; E = 1 on the end
// nodes):
//   K = K1 M1 M1 + M1 K1 M1 + M1 M1 K1,  M = M1 M1 M1,
//   M_Gamma = E M1 M1 + M1 E M1 + M1 M1 E.
// With the values outside the mesh taken as zero, the row of node (i, j, l)
// splits into in-plane parts and one 1D pass along z.  Per plane p of the
// node's column the in-plane sums
//   a0 = x(i, j),  H = x(i-1, j) + x(i+1, j),  V = x(i, j-1) + x(i, j+1),
//   a2 = the four diagonal neighbours
// give, with the node's x and y factors (halved centres on a boundary
// line),
//   PMM = (M1 M1) x,  PK = (K1 M1 + M1 K1) x,  PG = (E M1 + M1 E) x,
// and the row is
//   L x (l) = T1(l-1) + T1(l+1) + T0(l)                (interior plane l)
//   L x (l) = T1(l-1) + T1(l+1) + T0(l)/2 + c PMM(l)   (l = 0 or n)
// with T1 = (h/6)(a PK + b PMM + c PG) - (a/h) PMM and
// T0 = 4 (h/6)(a PK + b PMM + c PG) + 2 (a/h) PMM.  Interior, face, edge and
// corner nodes run the same code; no separate boundary kernel is needed.
//
// One workgroup owns a tile of mesh columns and a segment of planes and
// marches up the segment.  Each plane of the input passes once through a
// double-buffered LDS plane with a one-node halo (the plane after the next
// already requested), and every dependent pass is a pipeline stage behind the
// previous one: a stage's output plane reaches the next stage through a second
// double-buffered LDS plane, read at the next step, so that one barrier per
// step orders every plane exchange.  A pass has one or two stencil stages: one
// operator application, residual or Jacobi sweep, two sweeps (from a guess, or
// from the guess plus the prolonged coarse correction, the HSS update u += x
// on the last output), a zero-guess pair of sweeps or a sweep with the
// restriction of the residual (in-plane weights 1, 1/2, 1/4; across planes 1/2,
// 1, 1/2).
//
// What bounds it: in FP64 at 256^3 the prolongation with two sweeps moves 0.97
// GB (849 MB without the halo) in 196 us, 4.9 TB/s where a device copy reaches
// 5.1; the two-stage passes keep 8 wavefronts per CU (209 to 235 VGPRs), active
// half of the time and waiting for LDS and barriers a third of it.  The update
// pass (UPD) takes all 256 VGPRs and spills 12 (24 with Dirichlet faces): 250 us,
// 220 for its bytes.  In FP32 the instructions bound them.  Median times in a
// solve at 256^3, FP64 and FP32, with the passes of one stage (FP64) and of 512
// threads (FP32) that they replaced: two sweeps 188 us (330 in two) and 115
// (157), with the prolongation 196 (327) and 127 (169), the residual restriction
// 140 (144) and 68 (85), both zero-guess sweeps with it 188 (305) and 136; the
// HSS residual 156 (176) and 82.  Three stages a pass spill (508 us for two
// sweeps and the restriction, against 340 in two passes), one column a thread
// on 1024 threads has no registers left (242 us), and 24-row regions double the
// rim in FP32 (155 us).
#pragma once

#include <algorithm>
#include <type_traits>

#include "planes3d.h"

namespace helm {

namespace {

// A workgroup owns an LW x TH region of mesh columns, R vertically adjacent
// ones per thread: R = 2 columns share their in-plane neighbours (12 LDS reads
// for two columns instead of 18), and two independent chains per thread hide
// each other's latency.
constexpr int LW = 32;  // region columns (x); TH: rows (y)

// What a boundary column adds to a plane's terms: with nb boundary lines
// through it and w = bx V + by H, T1 += e1[0] nb a0 + e1[1] w (+ e1[2] a0 when
// nb = 2), T0 likewise with e0, and m -= 8 nb a0 + 2 w (- 4 a0 when nb = 2).  An
// end plane then takes T0 / 2 + cz m.  These coefficients stand in LDS (in
// registers where there is one stage), as do the Jacobi factors by the number
// of boundary coordinates (4: outside the mesh, zero); only wavefronts with
// columns on or outside the boundary and steps near the end planes read them.
template <typename T>
struct EdgeTab {
    cx<T> e1[3], e0[3], cz;
};
template <typename T>
__device__ __forceinline__ void edge_tab(const Op3F<T>& op, EdgeTab<T>* t) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        t->e1[q] = op.e1[q];
        t->e0[q] = op.e0[q];
    }
    t->cz = op.cz;
}

// LDS plane of a region: rows of LW values with a spare row and a spare value
// at either end, so that the neighbours of every column, those of the
// region's outermost ones included, lie inside (their sums are not used).
template <typename T, int TH>
using Plane = cx<T>[(TH + 2) * LW + 2];
__device__ __forceinline__ constexpr int at_plane(int ly, int lx) { return (ly + 1) * LW + lx + 1; }

// in-plane sums of R columns whose first one is at c: centre, east + west,
// north + south, and the four diagonal neighbours
template <typename T, int R>
__device__ __forceinline__ void plane_sums(const cx<T>* c, cx<T> (&a0)[R], cx<T> (&H)[R], cx<T> (&V)[R],
                                           cx<T> (&a2)[R]) {
    cx<T> m[R + 2], h[R + 2];  // centres and east + west of rows -1 .. R
#pragma unroll
    for (int r = 0; r < R + 2; ++r) {
        const cx<T>* q = c + (r - 1) * LW;
        m[r] = q[0];
        h[r] = q[-1] + q[1];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        a0[r] = m[r + 1];
        H[r] = h[r + 1];
        V[r] = m[r] + m[r + 2];
        a2[r] = h[r] + h[r + 2];
    }
}

// Work unit of a workgroup: a tile and a segment of planes of one slot.  Where
// the rim is split off (g.split) the tiles on the mesh's rim come first: their
// columns on and outside the boundary make a step dearer than an interior
// tile's, so they take shorter segments (tz_e planes instead of tz).  The others
// follow.  Of either list each XCD takes a contiguous range, so that
// neighbouring tiles of a segment share halo lines in one L2 (with the rim
// tiles dealt over the XCDs in turn, which are most of the tiles up to 128^3, a
// residual pass of four columns of 128^3 in FP32 took 56 us instead of 45).
// Passes that memory bounds keep all tiles in one list: split, an XCD's tiles
// are two strips with more halo between them and the other XCDs' (an
// application at 256^3 in FP64 took 136 us).  Returns false for a spare
// workgroup.
struct Unit3 {
    int slot, tx, ty, z0, z1;
};
__host__ __device__ inline int rim_tiles(const Grid3F& g) {
    return g.split && g.tiles_x > 2 && g.tiles_y > 2 ? 2 * g.tiles_x + 2 * (g.tiles_y - 2) : g.tiles_x * g.tiles_y;
}
__device__ __forceinline__ bool unit_of(const Grid3F& g, int planes, Unit3& u) {
    const unsigned E = (unsigned)rim_tiles(g), I = (unsigned)(g.tiles_x * g.tiles_y) - E;
    if (blockIdx.x < g.eblocks) {
        const unsigned per = E * (unsigned)g.segs_e;
        unsigned b = xcd_remap(blockIdx.x, g.eblocks);
        if (b >= per * (unsigned)g.slots) return false;
        u.slot = (int)(b / per);
        b %= per;
        const int e = (int)(b % E), seg = (int)(b / E);
        if (I == 0) {
            u.tx = e % g.tiles_x;
            u.ty = e / g.tiles_x;
        } else if (e < 2 * g.tiles_x) {
            u.tx = e % g.tiles_x;
            u.ty = e < g.tiles_x ? 0 : g.tiles_y - 1;
        } else {
            const int k = e - 2 * g.tiles_x;
            u.tx = (k & 1) ? g.tiles_x - 1 : 0;
            u.ty = 1 + k / 2;
        }
        u.z0 = seg * g.tz_e;
        u.z1 = min(u.z0 + g.tz_e, planes);
        return true;
    }
    const unsigned per = I * (unsigned)g.segs;
    unsigned b = xcd_remap(blockIdx.x - g.eblocks, gridDim.x - g.eblocks);
    u.slot = (int)(b / per);
    b %= per;
    const int t = (int)(b % I), seg = (int)(b / I);
    u.tx = 1 + t % (g.tiles_x - 2);
    u.ty = 1 + t / (g.tiles_x - 2);
    u.z0 = seg * g.tz;
    u.z1 = min(u.z0 + g.tz, planes);
    return true;
}

// --------------------------------------------------------------- k3_march --
// Passes (FIRST forms the first stage; M stencil stages in all, 1 or 2):
//   F_APPLY  y = L x
//   F_RESID  y = s (b - L x)
//   F_JAC    NJ Jacobi sweeps x <- x + w/D (b - L x) (from x + P e_c: PRO)
//   F_JAC0   x = w/D b, then NJ sweeps: the zero-guess sweeps
//   F_HSS0   rho = s R (written; R in Bv), x = w/D rho, then NJ sweeps with b = rho
// The last x goes to Y (UPD = 1: Y += x, the HSS update u += e with u in Y;
// nothing is written when there is no sweep).  RR adds one more stage, the
// residual b - L x of that x, and restricts it: b_c = P^T (b - L x) to Bc.
//
// At step p stage k takes in the plane p - 2 (k - 1) of its input (staged in
// LDS, or written there by stage k - 1 at the previous step) and completes
// its output plane p - 2 k + 1; the restriction follows one step behind.  One
// barrier per step orders every exchange.  A segment writes the planes
// [z0, z1) (with RR those of its coarse planes [Z0, Z1)), and starts M planes
// (M + 1 with RR) below them.
//
// The march is unrolled UNR steps at a time so that every ring slot is a
// fixed register: the load of a plane goes into a slot that the same step
// consumed, and no value is moved between slots.  Every load is issued
// unconditionally (what lies outside the mesh is out of the range of its
// buffer resource and reads as zero), so the count of requests in flight is
// the same on every path.  (Moving a register whose load is still in flight, or
// merging paths that issued different numbers of requests, makes the step
// wait for every request outstanding, the prefetches it has just issued among
// them.)  The right-hand side's ring also delays it to the later stages: slot
// i % BR holds b of plane i until the last stage has used it.
//
// Prolongation (PRO): (P e)(i, j, l) is trilinear interpolation from the n/2
// mesh.  Each coarse plane C the tile needs is staged once in LDS (the
// CW x CWH coarse columns under the region) and interpolated in-plane to every
// fine column, ce(C) = sum of the four coarse corners of the column (with
// repeats where a coordinate is even); a fine plane 2C takes ce(C) / 4 and
// 2C + 1 takes (ce(C) + ce(C + 1)) / 8 (exact powers of two).  The coarse
// plane for fine step p is written to LDS one step ahead and requested two
// steps ahead of that.
constexpr int CW = LW / 2 + 1;  // coarse columns under a region (prolongation)

template <int FIRST, int NJ, bool PRO, bool RR, int TH>
struct March {
    static constexpr bool J0 = FIRST == F_JAC0 || FIRST == F_HSS0;  // first sweep formed while staging
    static constexpr bool ONE = FIRST == F_APPLY || FIRST == F_RESID;
    static constexpr int M = ONE ? 1 : NJ + (RR ? 1 : 0);  // stencil stages
    static constexpr int KX = M - (RR ? 1 : 0);  // stage whose output is written (0: none)
    // owned columns and rows of a region, and the first of them: with the
    // restriction, whole coarse columns whose fine neighbours' residuals are
    // valid
    static constexpr int RIM = RR ? M + 1 : M;
    static constexpr int OWN = RR ? 2 * ((LW - 3 - 2 * M) / 2 + 1) : LW - 2 * M;
    static constexpr int OWNH = RR ? 2 * ((TH - 3 - 2 * M) / 2 + 1) : TH - 2 * M;
    static constexpr int PF = 2;  // input planes requested ahead of the one in LDS
    // ring of the right-hand side: PF ahead of its first use, kept to its last
    static constexpr int BR = PF + 2 * (M - 1) + (J0 ? 2 : 0);
    // (two steps where there is one stage: a launch of a few planes a workgroup
    // runs every copy of a step once, and their code has to be fetched)
    static constexpr int UNR = M == 1 && !RR ? 2 : BR < 4 ? 4 : BR;
    static_assert(M == 1 || M == 2, "one or two stages");
    static_assert(UNR % PF == 0 && UNR % 2 == 0 && UNR % BR == 0, "unroll must cover the rings");
    static_assert(!(PRO && (FIRST != F_JAC || RR)), "the prolongation feeds plain sweeps");
};

template <typename T, typename TI, int FIRST, int NJ, bool PRO, int UPD, bool RR, bool DIR, int TH, int R, bool COLW>
__global__ __launch_bounds__(LW * TH / R) void k3_march(Op3F<T> L, T s, Vec<const cx<TI>> X, Vec<const cx<T>> Bv,
                                                    Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y,
                                                    Vec<cx<T>> Bc, Grid3F g) {
    using C = March<FIRST, NJ, PRO, RR, TH>;
    constexpr int THREADS = LW * TH / R;
    constexpr int M = C::M, KX = C::KX, PF = C::PF, BR = C::BR, UNR = C::UNR;
    constexpr bool J0 = C::J0;
    constexpr int CWH = TH / 2 + 1;
    constexpr int RC = C::OWN / 2, RCH = C::OWNH / 2;  // coarse columns of a tile (RR)
    constexpr int CPL = CW * CWH > THREADS ? CW * CWH : THREADS;
    __shared__ Plane<T, TH> pl[M + (RR ? 1 : 0)][2];   // input of stage k + 1; with RR also the residual
    __shared__ cx<T> cpl[PRO ? 2 : 1][PRO ? CPL : 1];  // coarse planes, a row of CW values per coarse row
    __shared__ EdgeTab<T> tab;
    __shared__ cx<T> odt[5];
    const int n = L.n, nc = n / 2;
    Unit3 un;
    if (!unit_of(g, RR ? nc + 1 : n + 1, un)) return;
    const int slot = un.slot, tx = un.tx, ty = un.ty;
    const long long sy = n + 1, sz = sy * sy, syc = nc + 1, szc = syc * syc;
    const int lx = (int)threadIdx.x % LW, ly = (int)threadIdx.x / LW * R;
    const int i0 = tx * C::OWN - C::RIM, j0 = ty * C::OWNH - C::RIM;  // first column of the region
    const int i = i0 + lx, j = j0 + ly;                               // this thread's first column
    const int lp = at_plane(ly, lx);
    // the region reaches the mesh boundary (the same on every thread)
    const bool edge_tile = i0 <= 0 || j0 <= 0 || i0 + LW - 1 >= n || j0 + TH - 1 >= n;
    const bool bx = (i == 0) | (i == n), inx = (i >= 0) & (i <= n);
    bool inmesh[R], by[R], dcol[R];
    int cls[R];  // boundary lines through the column
    unsigned ox[R], ob[R], os[R];  // byte offsets in a plane: of x, of b, and of a store
    const unsigned dm = DIR ? L.dir : 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int jr = j + r;
        inmesh[r] = inx & (jr >= 0) & (jr <= n);
        by[r] = (jr == 0) | (jr == n);
        cls[r] = inmesh[r] ? (int)bx + (int)by[r] : 0;
        const bool owned = inmesh[r] & (lx >= C::RIM) & (lx < C::RIM + C::OWN) & (ly + r >= C::RIM) &
                           (ly + r < C::RIM + C::OWNH);
        // DIR: outputs on the nodes of Dirichlet faces are zero (the column
        // lies on an x or y Dirichlet face, or the plane is a z Dirichlet face)
        dcol[r] = DIR && (((dm & 1u) && i == 0) || ((dm & 2u) && i == n) || ((dm & 4u) && jr == 0) ||
                          ((dm & 8u) && jr == n));
        const unsigned col = (unsigned)(jr * (int)sy + i);
        ox[r] = inmesh[r] ? col * (unsigned)sizeof(cx<TI>) : OUTSIDE;
        ob[r] = inmesh[r] ? col * (unsigned)sizeof(cx<T>) : OUTSIDE;
        os[r] = owned ? ob[r] : OUTSIDE;
    }
    bool anyc = false, any2 = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        anyc |= !inmesh[r] | (cls[r] > 0);
        any2 |= cls[r] == 2;
    }
    // this wavefront has columns on or outside the boundary; at a corner line
    const bool edge_wave = __any((int)anyc), corner_wave = __any((int)any2);
    auto zfix = [&](int l) { return ((dm & 16u) && l == 0) || ((dm & 32u) && l == n); };
    const int Z0 = un.z0, Z1 = un.z1;  // with RR: coarse planes of the segment
    const int z0 = RR ? 2 * Z0 : un.z0, z1 = RR ? min(2 * Z1, n + 1) : un.z1;
    const cx<TI>* xs = J0 ? nullptr : X.at(slot);
    const cx<T>* bs = FIRST == F_APPLY ? nullptr : Bv.at(slot);
    cx<T>* rs = FIRST == F_HSS0 ? Rho.at(slot) : nullptr;
    cx<T>* ys = KX > 0 || C::ONE ? Y.at(slot) : nullptr;
    cx<T>* bc = RR ? Bc.at(slot) : nullptr;
    const cx<T> z = mk((T)0, (T)0);

    // the last stage's output planes [qf, ql], and the steps that give them
    const int qf = RR ? z0 - 1 : z0, ql = RR ? 2 * Z1 - 1 : z1 - 1;
    int p0 = qf - M;
    if (PRO || RR) p0 -= p0 & 1;  // an even first plane: the coarse planes follow the step's parity
    const int p1 = ql + 2 * M - 1 + (RR ? 1 : 0);
    const int hi = min(ql + M, n);  // last input plane needed
    // planes l of an input (outside the mesh, or past the last one needed: none)
    // and of an output (outside the segment: none), from the plane's address
    constexpr unsigned ES = (unsigned)sizeof(cx<T>), EI = (unsigned)sizeof(cx<TI>);
    const unsigned szb = (unsigned)sz * ES, szx = (unsigned)sz * EI, szcb = (unsigned)szc * ES;
    auto plane = [&](const void* base, int l, unsigned bytes) {
        return static_cast<const char*>(base) + (long long)l * (long long)bytes;
    };
    auto rin = [&](const char* a, int l, unsigned bytes) { return plane_rsrc(a, bytes, (unsigned)l <= (unsigned)hi); };
    auto rout = [&](const char* a, int l) { return plane_rsrc(a, szb, (unsigned)(l - z0) < (unsigned)(z1 - z0)); };

    // prolongation: this thread's coarse corners in the region's LDS coarse
    // plane, and the coarse value it stages (threads 0 .. CW CWH - 1; the
    // others a spare one)
    const int cI0 = i0 >> 1, cJ0 = j0 >> 1;  // floor: i0 may be negative
    const int cdx = i & 1;
    const int ca = (int)threadIdx.x % CW, cb = (int)threadIdx.x / CW;
    const bool cin = PRO && (int)threadIdx.x < CW * CWH && cI0 + ca >= 0 && cI0 + ca <= nc && cJ0 + cb >= 0 &&
                     cJ0 + cb <= nc;
    const cx<T>* ecs = PRO ? Ec.at(slot) : nullptr;
    const unsigned oc = cin ? (unsigned)((cJ0 + cb) * (int)syc + (cI0 + ca)) * (unsigned)sizeof(cx<T>) : OUTSIDE;
    // coarse plane Cz (staged in LDS as a quarter of it, which is exact)
    auto ldc = [&](int Cz) {
        return bload<T>(plane_rsrc(plane(ecs, Cz, szcb), szcb, (unsigned)Cz <= (unsigned)nc), oc);
    };
    auto interp = [&](int buf, int r) {
        const cx<T>* c = &cpl[buf][(((j + r) >> 1) - cJ0) * CW + (i >> 1) - cI0];
        const cx<T>* d = c + ((j + r) & 1) * CW;
        return (c[0] + c[cdx]) + (d[0] + d[cdx]);
    };
    // restriction: threads 0 .. RC RCH - 1 each take one coarse column, whose
    // fine centre is at (RIM + 2 rci, RIM + 2 rcj) of the region
    const bool cst = RR && (int)threadIdx.x < RC * RCH;
    const int rci = RR ? (int)threadIdx.x % RC : 0, rcj = RR ? (int)threadIdx.x / RC : 0;
    const int I = RC * tx + rci, J = RCH * ty + rcj;
    const bool ccol = DIR && (((dm & 1u) && I == 0) || ((dm & 2u) && I == nc) || ((dm & 4u) && J == 0) ||
                              ((dm & 8u) && J == nc));
    const unsigned occ = cst && I <= nc && J <= nc ? (unsigned)(J * (int)syc + I) * (unsigned)sizeof(cx<T>) : OUTSIDE;
    const int lc = at_plane(C::RIM + 2 * rcj, C::RIM + 2 * rci);

    if (threadIdx.x == 0) {
        if constexpr (M > 1) edge_tab(L, &tab);
        if constexpr (!C::ONE) {
#pragma unroll
            for (int q = 0; q < 4; ++q) odt[q] = L.od[q];
            odt[4] = z;
        }
    }
    auto etab = [&]() -> const auto& {
        if constexpr (M > 1) return tab;
        else return L;
    };

    const Weights<T> w(L);
    // COLW: the row's terms by the column's weights
    ColW<T> w1[COLW ? R : 1], w0[COLW ? R : 1];
    // EDGE: the region has columns on or outside the mesh boundary
    auto march = [&](auto edge) __attribute__((always_inline)) {
        constexpr bool EDGE = decltype(edge)::value;
        cx<T> cur = z, half = z;  // coarse accumulators
        if constexpr (COLW) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                w1[r] = col_weights<T>(L.r1, L.k1, L.e1, EDGE && bx, EDGE && by[r]);
                w0[r] = col_weights<T>(L.r0, L.k0, L.e0, EDGE && bx, EDGE && by[r]);
            }
        }
        cx<T> n1[R], n0[R];  // one stage: what nb boundary lines add to the weights of a0
        if constexpr (M == 1 && EDGE && !COLW) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T nb = (bx ? (T)1 : (T)0) + (by[r] ? (T)1 : (T)0);
                n1[r] = nb * L.e1[0];
                n0[r] = nb * L.e0[0];
            }
        }
        // rings: x at planes p + 1 .. p + PF; b from PF ahead of its first use
        // (plane p - 1, or p + 1 when the first stage is formed while staging)
        // on; y at the output planes of steps p .. p + PF - 1
        constexpr int BF = J0 ? 1 : -1;
        constexpr bool USEB = FIRST != F_APPLY;
        cx<TI> xr[PF][R];
        cx<T> br[BR][R], yr[PF][R];
        cx<T> cA[R], cB[R], cr = z;  // ce of coarse planes C - 1, C; staged coarse value
        // the Jacobi factor w/D on plane l (zero outside the mesh): of an
        // interior column, and of column r
        auto odu = [&](int l) {
            return odt[(unsigned)l <= (unsigned)n ? (int)((l == 0) | (l == n)) : 4];
        };
        auto odc = [&](int l, int r) {
            return odt[(inmesh[r] && (unsigned)l <= (unsigned)n) ? cls[r] + (int)((l == 0) | (l == n)) : 4];
        };
        // the values staged for plane l
        auto stage_in = [&](cx<T> (&v)[R], int l) {
            cx<T> od[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (DIR && J0) v[r] = csel(dcol[r] || zfix(l), z, v[r]);
                if constexpr (J0) od[r] = odu(l);
                // P e does not vanish outside the mesh
                if constexpr (PRO) v[r] = csel((unsigned)l <= (unsigned)n, v[r], z);
            }
            if constexpr (EDGE && (PRO || J0)) {
                if (edge_wave) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        if constexpr (J0) od[r] = odc(l, r);
                        if constexpr (PRO) v[r] = csel(inmesh[r], v[r], z);
                    }
                }
            }
            if constexpr (J0) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = od[r] * v[r];
            }
        };
#pragma unroll
        for (int r = 0; r < R; ++r) cA[r] = cB[r] = z;
        if (PRO) {
            const int m = p0 >> 1;
            cpl[m & 1][threadIdx.x] = (T)0.25 * ldc(m);
            cpl[(m + 1) & 1][threadIdx.x] = (T)0.25 * ldc(m + 1);
            cr = ldc(m + 2);
        }
#pragma unroll
        for (int k = 0; k < BR; ++k)
#pragma unroll
            for (int r = 0; r < R; ++r) br[k][r] = z;
        cx<T> v0[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (J0) v0[r] = bload<T>(rin(plane(bs, p0, szb), p0, szb), ob[r]);
            else v0[r] = cvt<T>(bload<TI>(rin(plane(xs, p0, szx), p0, szx), ox[r]));
        }
#pragma unroll
        for (int u = 0; u < PF; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int lx_ = p0 + 1 + u, lb_ = p0 + BF + u, ly_ = p0 - 2 * KX + 1 + u;
                if constexpr (!J0) xr[u][r] = bload<TI>(rin(plane(xs, lx_, szx), lx_, szx), ox[r]);
                if constexpr (USEB) br[u][r] = bload<T>(rin(plane(bs, lb_, szb), lb_, szb), ob[r]);
                if constexpr (UPD == 1) yr[u][r] = bload<T>(rout(plane(ys, ly_, szb), ly_), os[r]);
            }
        // addresses of the planes that the next step requests and writes
        const char* xa = J0 ? nullptr : plane(xs, p0 + 1 + PF, szx);
        const char* ba = USEB ? plane(bs, p0 + BF + PF, szb) : nullptr;
        const char* ya = KX > 0 || C::ONE ? plane(ys, p0 - 2 * KX + 1, szb) : nullptr;
        const char* ra = FIRST == F_HSS0 ? plane(rs, p0 + 1, szb) : nullptr;
        __syncthreads();  // coarse planes and tables
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (FIRST == F_HSS0) v0[r] = s * v0[r];
            if (J0) br[BR - 1][r] = v0[r];  // plane p0, first used by stage 1 at step p0 + 1
            if (PRO) {
                cB[r] = interp((p0 >> 1) & 1, r);
                v0[r] = v0[r] + cB[r];
            }
        }
        stage_in(v0, p0);
#pragma unroll
        for (int r = 0; r < R; ++r) pl[0][0][lp + r * LW] = v0[r];
        // stage k: acc = T1(q - 1) + T0(q) for its next output plane q, tp =
        // T1(q), xc the input centre of q
        cx<T> acc[M][R], tp[M][R], xc[M][R];
#pragma unroll
        for (int k = 0; k < M; ++k)
#pragma unroll
            for (int r = 0; r < R; ++r) acc[k][r] = tp[k][r] = xc[k][r] = z;

        auto step = [&](auto uc, int p) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            constexpr int kb = u & 1;   // LDS buffer of input plane p
            constexpr int sl = u % PF;  // ring slot of this step
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            // input plane p + 1 into the buffer of plane p - 1 (free since the
            // barrier; past the last plane it is written and never read)
            cx<T> vin[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (J0) {
                    vin[r] = br[u % BR][r];
                    if (FIRST == F_HSS0) {
                        vin[r] = s * vin[r];
                        if (DIR) vin[r] = csel(dcol[r] || zfix(p + 1), z, vin[r]);
                        br[u % BR][r] = vin[r];
                        bstore(rout(ra, p + 1), os[r], vin[r]);
                    }
                } else {
                    vin[r] = cvt<T>(xr[sl][r]);
                }
                if (PRO) {
                    if (kb == 0) {  // p + 1 = 2C - 1
                        cA[r] = cB[r];
                        cB[r] = interp(((p + 2) >> 1) & 1, r);
                        const cx<T> c = cA[r] + cB[r];
                        vin[r] = mk(fmat((T)0.5, c.x, vin[r].x), fmat((T)0.5, c.y, vin[r].y));
                    } else {  // p + 1 = 2C
                        vin[r] = vin[r] + cB[r];
                    }
                }
            }
            stage_in(vin, p + 1);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                pl[0][kb ^ 1][lp + r * LW] = vin[r];
                if constexpr (!J0) xr[sl][r] = bload<TI>(rin(xa, p + 1 + PF, szx), ox[r]);
            }
            if (PRO && kb == 1) {  // coarse plane (p + 3) / 2, needed at step p + 1
                cpl[((p + 3) >> 1) & 1][threadIdx.x] = (T)0.25 * cr;
                cr = ldc((p + 5) >> 1);
            }
            // the stages; k counts from 0
            auto stage = [&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                const int pi = p - 2 * k, q = pi - 1;  // input and output plane
                // b of plane q: slot of the step that took it in
                constexpr int sb = (u - 2 * k - (J0 ? 2 : 0) + 4 * UNR) % BR;
                const bool end = (pi == 0) | (pi == n);
                cx<T> a0[R], H[R], V[R], a2[R];
                plane_sums<T, R>(&pl[k][k == 0 ? kb : kb ^ 1][lp], a0, H, V, a2);
                constexpr bool RES = RR && k == M - 1;  // the restricted residual
                constexpr bool OD = !C::ONE && !RES;
                cx<T> t1[R], t0[R], m[R], od[R];
                if constexpr (COLW) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        t1[r] = col_sum(w1[r], a0[r], H[r], V[r], a2[r]);
                        t0[r] = col_sum(w0[r], a0[r], H[r], V[r], a2[r]);
                        if (end) t0[r] = end_term(etab().cz, bx, by[r], a0[r], H[r], V[r], a2[r], t0[r]);
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        plane_terms<T>(w, a0[r], H[r] + V[r], a2[r], t1[r], t0[r], m[r]);
                    }
                    if constexpr (EDGE) {
                        if (edge_wave) {
                            cx<T> e[R];
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const T fx = bx ? (T)1 : (T)0, fy = by[r] ? (T)1 : (T)0;
                                e[r] = mk(fmat(fx, V[r].x, fy * H[r].x), fmat(fx, V[r].y, fy * H[r].y));
                            }
                            if constexpr (M == 1) {
                                // the weights of nb a0 stand in registers, and
                                // only an end plane needs the mass pattern
#pragma unroll
                                for (int r = 0; r < R; ++r) {
                                    t1[r] = cfma(n1[r], a0[r], cfma(L.e1[1], e[r], t1[r]));
                                    t0[r] = cfma(n0[r], a0[r], cfma(L.e0[1], e[r], t0[r]));
                                }
                                if (corner_wave) {
#pragma unroll
                                    for (int r = 0; r < R; ++r) {
                                        const T f = cls[r] == 2 ? (T)1 : (T)0;
                                        t1[r] = cfma(L.e1[2], f * a0[r], t1[r]);
                                        t0[r] = cfma(L.e0[2], f * a0[r], t0[r]);
                                    }
                                }
                                if (end) {
#pragma unroll
                                    for (int r = 0; r < R; ++r) {
                                        const T fx = bx ? (T)1 : (T)0, fy = by[r] ? (T)1 : (T)0;
                                        m[r] = axpy_real((T)-8 * (fx + fy), a0[r], axpy_real((T)-2, e[r], m[r]));
                                        m[r] = axpy_real(cls[r] == 2 ? (T)4 : (T)0, a0[r], m[r]);
                                    }
                                }
                            } else {
                                cx<T> na[R];
#pragma unroll
                                for (int r = 0; r < R; ++r) na[r] = ((bx ? (T)1 : (T)0) + (by[r] ? (T)1 : (T)0)) * a0[r];
                                __builtin_amdgcn_sched_barrier(0);
                                const cx<T> c0 = tab.e1[0], c1 = tab.e1[1];
#pragma unroll
                                for (int r = 0; r < R; ++r) t1[r] = cfma(c0, na[r], cfma(c1, e[r], t1[r]));
                                __builtin_amdgcn_sched_barrier(0);
                                const cx<T> d0 = tab.e0[0], d1 = tab.e0[1];
#pragma unroll
                                for (int r = 0; r < R; ++r) t0[r] = cfma(d0, na[r], cfma(d1, e[r], t0[r]));
#pragma unroll
                                for (int r = 0; r < R; ++r)
                                    m[r] = mk(fmat((T)-8, na[r].x, fmat((T)-2, e[r].x, m[r].x)),
                                              fmat((T)-8, na[r].y, fmat((T)-2, e[r].y, m[r].y)));
                                if (corner_wave) {
                                    const cx<T> c2 = tab.e1[2], d2 = tab.e0[2];
#pragma unroll
                                    for (int r = 0; r < R; ++r) {
                                        const T f = cls[r] == 2 ? (T)1 : (T)0;
                                        t1[r] = cfma(c2, f * a0[r], t1[r]);
                                        t0[r] = cfma(d2, f * a0[r], t0[r]);
                                        m[r] = mk(fmat((T)4 * f, a0[r].x, m[r].x), fmat((T)4 * f, a0[r].y, m[r].y));
                                    }
                                }
                            }
                        }
                    }
                    if (end) {
                        const cx<T> cz = etab().cz;
#pragma unroll
                        for (int r = 0; r < R; ++r) t0[r] = cfma(cz, m[r], (T)0.5 * t0[r]);
                    }
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if constexpr (OD && EDGE) od[r] = odc(q, r);
                    else if constexpr (OD) od[r] = odu(q);
                    const cx<T> ax = acc[k][r] + t1[r];  // A x at plane q
                    cx<T> v;
                    if constexpr (FIRST == F_APPLY) {
                        v = ax;
                    } else if constexpr (FIRST == F_RESID) {
                        v = s * (br[sb][r] - ax);
                    } else if constexpr (RES) {
                        // zero outside the mesh
                        v = br[sb][r] - ax;
                        v = csel((unsigned)q <= (unsigned)n && (!EDGE || inmesh[r]), v, z);
                    } else {
                        v = cfma(od[r], br[sb][r] - ax, xc[k][r]);
                    }
                    if (DIR) v = csel(dcol[r] || zfix(q), z, v);
                    if constexpr (C::ONE || k == KX - 1) {
                        cx<T> y = v;
                        if constexpr (UPD == 1) {
                            y = yr[sl][r] + v;
                            yr[sl][r] = bload<T>(rout(ya + PF * (long long)szb, q + PF), os[r]);
                        }
                        bstore(rout(ya, q), os[r], y);
                    }
                    if constexpr (k + 1 < M + (RR ? 1 : 0)) pl[k + 1][kb][lp + r * LW] = v;
                    acc[k][r] = tp[k][r] + t0[r];
                    tp[k][r] = t1[r];
                    xc[k][r] = a0[r];
                }
            };
            // a rim tile's boundary branch needs the registers that overlapping
            // the stages would take
            if constexpr (EDGE && M > 1) __builtin_amdgcn_sched_barrier(0);
            stage(IC<0>{});
            if constexpr (EDGE && M > 1) __builtin_amdgcn_sched_barrier(0);
            if constexpr (M > 1) stage(IC<1>{});
            if constexpr (EDGE && M > 1) __builtin_amdgcn_sched_barrier(0);
            // the slot that the last stage has just read
            if constexpr (USEB) {
#pragma unroll
                for (int r = 0; r < R; ++r) br[(u + PF) % BR][r] = bload<T>(rin(ba, p + BF + PF, szb), ob[r]);
            }
            if constexpr (!J0) xa += szx;
            if constexpr (USEB) ba += szb;
            if constexpr (KX > 0 || C::ONE) ya += szb;
            if constexpr (FIRST == F_HSS0) ra += szb;
            // the residual plane p - 2 M that the last stage wrote at the previous step
            if constexpr (RR) {
                if (cst) {
                    const cx<T> r2 = restrict_plane<T, LW>(&pl[M][kb ^ 1][lc]);
                    if (kb == 1) {  // an odd plane: coarse plane Lc is complete
                        const int Lc = (p - 2 * M - 1) >> 1;
                        cx<T> v = axpy_real((T)0.5, r2, cur);
                        if (DIR) v = csel(ccol || ((dm & 16u) && Lc == 0) || ((dm & 32u) && Lc == nc), z, v);
                        bstore(plane_rsrc(plane(bc, Lc, szcb), szcb, (unsigned)(Lc - Z0) < (unsigned)(Z1 - Z0)), occ, v);
                        half = (T)0.5 * r2;
                    } else {
                        cur = half + r2;
                    }
                }
            }
        };
        int pb = p0;
        for (; pb + UNR - 1 <= p1; pb += UNR) {
            step(IC<0>{}, pb);
            step(IC<1>{}, pb + 1);
            if constexpr (UNR > 2) {
                step(IC<2>{}, pb + 2);
                step(IC<3>{}, pb + 3);
            }
            if constexpr (UNR > 4) {
                step(IC<4>{}, pb + 4);
                step(IC<5>{}, pb + 5);
            }
        }
        if (pb <= p1) step(IC<0>{}, pb);
        if constexpr (UNR > 2) {
            if (pb + 1 <= p1) step(IC<1>{}, pb + 1);
            if (pb + 2 <= p1) step(IC<2>{}, pb + 2);
        }
        if constexpr (UNR > 4) {
            if (pb + 3 <= p1) step(IC<3>{}, pb + 3);
            if (pb + 4 <= p1) step(IC<4>{}, pb + 4);
        }
    };
    if (edge_tile) march(std::true_type{});
    else march(std::false_type{});
}

// Workgroups of a kernel that the device holds at once (its occupancy per
// CU, from its register and LDS use, times the CUs), asked once per kernel.
template <auto K, int FT>
int resident_units() {
    static const int units = [] {
        int nb = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, K, FT, 0) != hipSuccess || nb < 1) nb = 1;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
        return nb * cus;
    }();
    return units;
}

// Segment heights: output planes per workgroup (coarse planes with the
// restriction, `per` = 2 input planes each), tz for interior tiles and tz_e
// for those on the rim.  A launch takes ceil(units / resident) rounds, each as
// long as one segment's march, its planes plus the pipeline's head (a rim
// tile's step costs `rim` percent of an interior one's); the heights minimise
// rounds x march.
void seg_planes(Grid3F& g, int planes, int per, int head, int resident, int rim) {
    const long long E = rim_tiles(g), I = (long long)g.tiles_x * g.tiles_y - E;
    long long best = -1;
    for (int segs = 1; segs <= planes; ++segs) {
        const int tz = (planes + segs - 1) / segs;
        // rim segments of the same march time, if they can be
        int te = I == 0 ? tz : ((per * tz + head) * 100 / rim - head) / per;
        te = te < 1 ? 1 : te;
        const int ne = (planes + te - 1) / te;
        te = (planes + ne - 1) / ne;
        const long long ce = (long long)(per * te + head) * (I == 0 ? 100 : rim);
        const long long ci = (long long)(per * tz + head) * 100;
        const int ns = (planes + tz - 1) / tz;
        const long long units = (E * ne + I * ns) * g.slots;
        const long long rounds = (units + resident - 1) / resident;
        const long long cost = rounds * (I > 0 && ci > ce ? ci : ce);
        if (best < 0 || cost < best) {
            best = cost;
            g.tz = tz;
            g.segs = ns;
            g.tz_e = te;
            g.segs_e = ne;
        }
    }
}

// A rim tile's step against an interior one's in percent: 140 where the
// instructions count, 100 for the one-stage passes that memory bounds (at 120
// the residual pass at 256^3 took 210 instead of 181 us, at 160 the two-sweep
// pass 228 instead of 202).
constexpr int RIM_COST = 140, RIM_COST_MEM = 100;

template <typename T, typename TI, int F, int NJ, bool PRO, int UPD, bool RR, bool DIR, int TH, int R, bool COLW>
void launch_h(hipStream_t st, const Op3F<T>& L, T s, Vec<const cx<TI>> X, Vec<const cx<T>> Bv,
              Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y, Vec<cx<T>> Bc, int nslots) {
    using C = March<F, NJ, PRO, RR, TH>;
    constexpr int THREADS = LW * TH / R;
    const int n = L.n, planes = RR ? n / 2 + 1 : n + 1;
    Grid3F g;
    g.tiles_x = (n + C::OWN) / C::OWN;
    g.tiles_y = (n + C::OWNH) / C::OWNH;
    g.slots = nslots;
    g.split = C::M > 1 || RR || TH < LW;
    seg_planes(g, planes, RR ? 2 : 1, 3 * C::M + 2,
               resident_units<k3_march<T, TI, F, NJ, PRO, UPD, RR, DIR, TH, R, COLW>, THREADS>(),
               C::M > 1 || RR ? RIM_COST : RIM_COST_MEM);
    const unsigned E = (unsigned)rim_tiles(g), I = (unsigned)(g.tiles_x * g.tiles_y) - E;
    g.eblocks = (E * (unsigned)g.segs_e * (unsigned)nslots + 7) / 8 * 8;  // whole rounds over the XCDs
    const unsigned grid = g.eblocks + I * (unsigned)g.segs * (unsigned)nslots;
    k3_march<T, TI, F, NJ, PRO, UPD, RR, DIR, TH, R, COLW><<<grid, THREADS, 0, st>>>(L, s, X, Bv, Ec, Rho, Y, Bc, g);
}

template <typename T, typename TI, int F, int NJ, bool PRO, int UPD, bool RR, int TH, int R, bool COLW = false>
void launch_d(hipStream_t st, const Op3F<T>& L, T s, Vec<const cx<TI>> X, Vec<const cx<T>> Bv,
              Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y, Vec<cx<T>> Bc, int nslots) {
    if (L.dir) launch_h<T, TI, F, NJ, PRO, UPD, RR, true, TH, R, COLW>(st, L, s, X, Bv, Ec, Rho, Y, Bc, nslots);
    else launch_h<T, TI, F, NJ, PRO, UPD, RR, false, TH, R, COLW>(st, L, s, X, Bv, Ec, Rho, Y, Bc, nslots);
}

}  // namespace

}  // namespace helm
