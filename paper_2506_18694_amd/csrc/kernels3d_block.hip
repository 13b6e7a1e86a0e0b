// Fused passes on the small 3D Q1 levels, one block of the mesh per workgroup.
//
// The z-marching passes (kernels3d_fused.hip) order every plane by a barrier,
// about half a microsecond each, and a launch adds two more; on a level of a
// few thousand nodes that latency is all of their time (7 us a pass at 16^3).
// Here a workgroup holds every plane that its output needs in LDS at once: a
// stage (a Jacobi sweep, the residual) is one loop over those planes with no
// barrier inside, each thread marching up its own mesh column in registers,
// and a pass is M stages and M barriers.  Each stage loses one node on every
// side of the region, so the halo is recomputed (a two-sweep pass of TZ planes
// forms TZ + 2 planes of the first sweep), which costs nothing while most
// compute units would idle.  Two passes per level and cycle take the place of
// four or more: the pre-smoothing with the residual restriction, and the
// prolongation with the post-smoothing.
//
// Row of node (i, j, l), as in the marching passes: L x = T1(l-1) + T1(l+1) +
// T0(l), with T1, T0 linear in the four in-plane sums of a plane's
// neighbourhood of (i, j): centre, east + west, north + south, diagonals.  A
// boundary column has weights of its own, so the weights are per-lane values
// and every column runs the same code.
#pragma clang fp contract(off)
#include <type_traits>

#include "planes3d.h"

namespace helm {

namespace {

// FIRST, NJ, PRO, UPD, RR as for pass3d: the first stage, NJ Jacobi sweeps, P
// e_c added to the input, Y += result, and the restriction of the last x's
// residual.  TZ: output planes (coarse planes with RR).
template <typename T, int FIRST, int NJ, bool PRO, bool RR, int LW, int LH, int TZ>
struct Block {
    static constexpr bool J0 = FIRST == F_JAC0 || FIRST == F_HSS0;  // first sweep formed while staging
    static constexpr bool HSS = FIRST == F_HSS;
    static constexpr bool ONE = FIRST == F_RESID;
    static constexpr int M = NJ + (HSS || ONE ? 1 : 0) + (RR ? 1 : 0);  // stencil stages
    static constexpr int NO = RR ? 2 * TZ + 1 : TZ;              // output planes of the last stage
    static constexpr int NP = NO + 2 * M;                        // input planes
    static constexpr int RIM = RR ? M + 1 : M;
    static constexpr int OWN = RR ? 2 * ((LW - 3 - 2 * M) / 2 + 1) : LW - 2 * M;
    static constexpr int OWNH = RR ? 2 * ((LH - 3 - 2 * M) / 2 + 1) : LH - 2 * M;
    static constexpr int THREADS = LW * LH;
    static constexpr int PLANE = (LH + 2) * LW + 2;  // a spare row and value at either end
    static constexpr int CW = LW / 2 + 1, CH = LH / 2 + 1, NC = (NP + 1) / 2 + 1;  // coarse values under a region
    // LDS: the input planes (later every second stage's), the first stage's
    // planes, and the coarse planes in the latter's place before that
    static constexpr int SECOND = M > 1 || RR ? (NP - 2) * PLANE : 1;
    static constexpr int ELEMS = NP * PLANE + (PRO && NC * CW * CH > SECOND ? NC * CW * CH : SECOND);
    static_assert(M >= 1 && OWN > 0 && OWNH > 0, "region too small");
};

template <typename T, int FIRST, int NJ, bool PRO, int UPD, bool RR, int LW, int LH, int TZ, bool DIR>
__global__ __launch_bounds__(LW * LH) void k3_block(Op3F<T> L, Op3F<T> B, T s, Vec<const cx<T>> X,
                                                    Vec<const cx<T>> Bv, Vec<const cx<T>> Ec, Vec<cx<T>> Rho,
                                                    Vec<cx<T>> Y, Vec<cx<T>> Bc, int tiles_x, int tiles_y,
                                                    int segs) {
    using C = Block<T, FIRST, NJ, PRO, RR, LW, LH, TZ>;
    constexpr int M = C::M, NP = C::NP, PLANE = C::PLANE;
    constexpr bool WRHO = FIRST == F_HSS || FIRST == F_HSS0;
    __shared__ cx<T> lds[C::ELEMS];
    cx<T>* const pa = lds;               // inputs of stages 1, 3
    cx<T>* const pb = lds + NP * PLANE;  // inputs of stage 2
    const int n = L.n, nc = n / 2;
    const long long sy = n + 1, sz = sy * sy, syc = nc + 1, szc = syc * syc;
    int b = (int)blockIdx.x;
    const int tx = b % tiles_x;
    b /= tiles_x;
    const int ty = b % tiles_y;
    b /= tiles_y;
    const int seg = b % segs, slot = b / segs;
    const int lx = (int)threadIdx.x % LW, ly = (int)threadIdx.x / LW;
    const int i0 = tx * C::OWN - C::RIM, j0 = ty * C::OWNH - C::RIM;
    const int i = i0 + lx, j = j0 + ly;
    const int lp = (ly + 1) * LW + lx + 1;
    const bool inmesh = (i >= 0) & (i <= n) & (j >= 0) & (j <= n);
    const bool bx = (i == 0) | (i == n), by = (j == 0) | (j == n);
    const int cls = (int)bx + (int)by;
    const bool owned = inmesh & (lx >= C::RIM) & (lx < C::RIM + C::OWN) & (ly >= C::RIM) & (ly < C::RIM + C::OWNH);
    const unsigned dm = DIR ? L.dir : 0u;
    const bool dcol = DIR && (((dm & 1u) && i == 0) || ((dm & 2u) && i == n) || ((dm & 4u) && j == 0) ||
                              ((dm & 8u) && j == n));
    // outputs on the nodes of Dirichlet faces are zero
    auto dfix = [&](cx<T> v, int l) {
        if constexpr (!DIR) return v;
        else return csel(dcol || ((dm & 16u) && l == 0) || ((dm & 32u) && l == n), mk((T)0, (T)0), v);
    };
    const unsigned ob = inmesh ? (unsigned)(j * (int)sy + i) * (unsigned)sizeof(cx<T>) : OUTSIDE;
    const unsigned os = owned ? ob : OUTSIDE;
    const cx<T> z = mk((T)0, (T)0);
    // fine output planes [z0, z1), coarse ones [Z0, Z1); plane of input index 0
    const int Z0 = seg * TZ, Z1 = min(Z0 + TZ, (RR ? nc : n) + 1);
    const int z0 = RR ? 2 * Z0 : Z0, z1 = RR ? min(2 * Z1, n + 1) : Z1;
    const int lb = (RR ? z0 - 1 : z0) - M;
    const unsigned szb = (unsigned)sz * (unsigned)sizeof(cx<T>);
    auto plane = [&](const cx<T>* base, int l) { return reinterpret_cast<const char*>(base + (long long)l * sz); };
    auto rin = [&](const cx<T>* base, int l) { return plane_rsrc(plane(base, l), szb, (unsigned)l <= (unsigned)n); };
    auto rout = [&](const cx<T>* base, int l) {
        return plane_rsrc(plane(base, l), szb, (unsigned)(l - z0) < (unsigned)(z1 - z0));
    };
    // this column's Jacobi factor on an interior plane and on an end plane
    auto od_of = [&](int q) { return csel(q < 2, csel(q == 0, L.od[0], L.od[1]), csel(q == 2, L.od[2], L.od[3])); };
    const cx<T> odI = csel(inmesh, od_of(cls), z), odE = csel(inmesh, od_of(cls + 1), z);
    auto odf = [&](int l) { return csel((unsigned)l <= (unsigned)n, csel((l == 0) | (l == n), odE, odI), z); };

    // every load of the pass
    cx<T> v[NP], bv[NP], yo[UPD == 1 ? TZ : 1];
    const cx<T>* xs = C::J0 ? nullptr : X.at(slot);
    const cx<T>* bs = Bv.at(slot);
    cx<T>* ys = NJ > 0 || C::ONE ? Y.at(slot) : nullptr;
    cx<T>* rs = WRHO ? Rho.at(slot) : nullptr;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        if constexpr (!C::J0) v[q] = bload<T>(rin(xs, lb + q), ob);
        if (C::J0 || (q > 0 && q < NP - 1)) bv[q] = bload<T>(rin(bs, lb + q), ob);
    }
    if constexpr (UPD == 1) {
#pragma unroll
        for (int q = 0; q < TZ; ++q) yo[q] = bload<T>(rout(ys, z0 + q), os);
    }
    if constexpr (PRO) {
        // the coarse columns under the region, planes floor(lb / 2) on
        const int cI0 = i0 >> 1, cJ0 = j0 >> 1, cL0 = lb >> 1;
        const cx<T>* es = Ec.at(slot);
        for (int q = (int)threadIdx.x; q < C::NC * C::CW * C::CH; q += C::THREADS) {
            const int ca = q % C::CW, cb = q / C::CW % C::CH, cl = cL0 + q / (C::CW * C::CH);
            const int I = cI0 + ca, J = cJ0 + cb;
            const bool in = I >= 0 && I <= nc && J >= 0 && J <= nc && cl >= 0 && cl <= nc;
            pb[q] = in ? es[(long long)cl * szc + (long long)J * syc + I] : z;
        }
        __syncthreads();
        const cx<T>* c = pb + ((j >> 1) - cJ0) * C::CW + (i >> 1) - cI0;
        const int dx = i & 1, dy = (j & 1) * C::CW;
        cx<T> ce[C::NC];  // in-plane interpolation, 4 times too large
#pragma unroll
        for (int q = 0; q < C::NC; ++q) {
            const cx<T>* a = c + q * C::CW * C::CH;
            ce[q] = (a[0] + a[dx]) + (a[dy] + a[dy + dx]);
        }
        // plane lb + q: an even one takes ce / 4, an odd one the mean of two
        const bool odd = lb & 1;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int l = lb + q;
            cx<T> p;
            if ((q & 1) == 0) {
                // even lb: plane 2C; odd lb: 2C + 1
                const cx<T> c0 = ce[q / 2], c1 = ce[q / 2 + 1 < C::NC ? q / 2 + 1 : q / 2];
                p = csel(odd, (T)0.125 * (c0 + c1), (T)0.25 * c0);
            } else {
                const cx<T> c0 = ce[q / 2], c1 = ce[q / 2 + 1];
                p = csel(odd, (T)0.25 * c1, (T)0.125 * (c0 + c1));
            }
            v[q] = csel(inmesh && (unsigned)l <= (unsigned)n, v[q] + p, z);
        }
    }
    if constexpr (C::J0) {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int l = lb + q;
            if constexpr (FIRST == F_HSS0) {
                bv[q] = dfix(s * bv[q], l);
                bstore(rout(rs, l), os, bv[q]);
            }
            v[q] = dfix(odf(l) * bv[q], l);
        }
    }
    if constexpr (PRO) __syncthreads();  // the coarse values have been read
#pragma unroll
    for (int q = 0; q < NP; ++q) pa[q * PLANE + lp] = v[q];
    __syncthreads();

    // stage k (from 0): input planes lb + k .. in `in`, outputs to `out`
    auto stage = [&](auto kc, const cx<T>* in, cx<T>* out) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        constexpr int NI = NP - 2 * k;  // input planes
        constexpr bool FHSS = C::HSS && k == 0, RES = RR && k == M - 1;
        constexpr bool WR = !RES && k == M - 1 - (RR ? 1 : 0);  // the x that is written
        const Op3F<T>& A = FHSS ? B : L;
        const ColW<T> w1 = col_weights<T>(A.r1, A.k1, A.e1, bx, by), w0 = col_weights<T>(A.r0, A.k0, A.e0, bx, by);
        cx<T> acc = z, tp = z, xc = z;
#pragma unroll
        for (int q = 0; q < NI; ++q) {
            const int pi = lb + k + q;  // input plane
            const cx<T>* c = in + q * PLANE + lp;
            const cx<T> a0 = c[0], H = c[-1] + c[1], V = c[-LW] + c[LW];
            const cx<T> a2 = (c[-LW - 1] + c[-LW + 1]) + (c[LW - 1] + c[LW + 1]);
            const cx<T> t1 = col_sum(w1, a0, H, V, a2);
            cx<T> t0 = col_sum(w0, a0, H, V, a2);
            if (pi == 0 || pi == n) t0 = end_term(A.cz, bx, by, a0, H, V, a2, t0);
            if (q >= 2) {
                const int l = pi - 1;  // output plane
                const cx<T> r = bv[k + q - 1] - (acc + t1);
                cx<T> x;
                if constexpr (RES) {
                    x = csel(inmesh && (unsigned)l <= (unsigned)n, r, z);
                } else if constexpr (C::ONE) {
                    x = s * r;
                } else if constexpr (FHSS) {
                    const cx<T> rho = dfix(s * r, l);
                    bv[k + q - 1] = rho;
                    bstore(rout(rs, l), os, rho);
                    x = odf(l) * rho;
                } else {
                    x = cfma(odf(l), r, xc);
                }
                x = dfix(x, l);
                if constexpr (WR) {
                    cx<T> y = x;
                    if constexpr (UPD == 1) y = yo[q - 2] + x;
                    bstore(rout(ys, l), os, y);
                }
                if constexpr (k + 1 < M || RR) out[(q - 2) * PLANE + lp] = x;
            }
            acc = tp + t0;
            tp = t1;
            xc = a0;
        }
        if constexpr (k + 1 < M || RR) __syncthreads();
    };
    stage(IC<0>{}, pa, pb);
    if constexpr (M > 1) stage(IC<1>{}, pb, pa);
    if constexpr (M > 2) stage(IC<2>{}, pa, pb);
    if constexpr (RR) {
        // residual planes 2 Z0 - 1 .. 2 Z0 + 2 TZ - 1; one coarse node a thread
        const cx<T>* r = (M & 1) ? pb : pa;
        constexpr int RC = C::OWN / 2, RCH = C::OWNH / 2;
        cx<T>* bc = Bc.at(slot);
        for (int q = (int)threadIdx.x; q < RC * RCH * TZ; q += C::THREADS) {
            const int ci = q % RC, cj = q / RC % RCH, cl = q / (RC * RCH);
            const int I = RC * tx + ci, J = RCH * ty + cj, Lc = Z0 + cl;
            const cx<T>* c = r + 2 * cl * PLANE + (C::RIM + 2 * cj + 1) * LW + C::RIM + 2 * ci + 1;
            cx<T> o = axpy_real((T)0.5, restrict_plane<T, LW>(c), restrict_plane<T, LW>(c + PLANE));
            o = axpy_real((T)0.5, restrict_plane<T, LW>(c + 2 * PLANE), o);
            if (DIR && (((dm & 1u) && I == 0) || ((dm & 2u) && I == nc) || ((dm & 4u) && J == 0) ||
                        ((dm & 8u) && J == nc) || ((dm & 16u) && Lc == 0) || ((dm & 32u) && Lc == nc)))
                o = z;
            if (I <= nc && J <= nc && Lc <= nc) bc[(long long)Lc * szc + (long long)J * syc + I] = o;
        }
    }
}

template <typename T, int F, int NJ, bool PRO, int UPD, bool RR, int LW, int LH, int TZ, bool DIR>
void launch_b(hipStream_t st, const Op3F<T>& L, const Op3F<T>& B, T s, Vec<const cx<T>> X, Vec<const cx<T>> Bv,
              Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y, Vec<cx<T>> Bc, int ns) {
    using C = Block<T, F, NJ, PRO, RR, LW, LH, TZ>;
    const int tiles_x = (L.n + C::OWN) / C::OWN, tiles_y = (L.n + C::OWNH) / C::OWNH;
    const int planes = RR ? L.n / 2 + 1 : L.n + 1, segs = (planes + TZ - 1) / TZ;
    k3_block<T, F, NJ, PRO, UPD, RR, LW, LH, TZ, DIR><<<(unsigned)(tiles_x * tiles_y * segs * ns), C::THREADS, 0, st>>>(
        L, B, s, X, Bv, Ec, Rho, Y, Bc, tiles_x, tiles_y, segs);
}

// Workgroups of a pass with the given region and segment height.
template <typename C>
long long units_of(int n, int planes, int tz, int ns) {
    const long long tx = (n + C::OWN) / C::OWN, ty = (n + C::OWNH) / C::OWNH;
    return tx * ty * ((planes + tz - 1) / tz) * ns;
}

// A pass whose 16 x 16 regions of the smallest height fill the chip at most
// twice runs with those; above that a wider region (less halo) if one a
// compute unit suffices, else taller 16 x 16 ones.  Measured (us per launch in
// FP64, 16 x 16 / 32 x 16 / taller): prolongation + two sweeps 32^3 6.6 / 7.9 /
// 7.8, 48^3 9.8 / 8.3 / 9.9, 64^3 19.7 / 24.0 / 19.0; pre-smoothing +
// restriction 32^3 8.0 / 8.1 / 7.6, 48^3 11.7 / 8.5 / 9.7, 64^3 23.0 / 21.4 /
// 17.7.  The marching passes took 15 and 13 us at 16^3 to 48^3, in two launches
// each.
//
// The halo costs nothing only while compute units would idle: from
// BLOCK3D_BYTES a vector on, all columns counted, the marching passes win
// whatever the mesh (kernels3d_columns.hip).  Measured (us per preconditioner of
// four steps, blocks / marching): FP64 64^3 1 column (4.4 MB) 891 / 1087, 48^3 8
// (15 MB) 1657 / 1246, 80^3 1 (8.5 MB) 1276 / 1190, 16 5591 / 4015 at 64^3 and
// 10640 / 6176 at 80^3; FP32 64^3 2 (4.4 MB) 994 / 1122, 80^3 1 (4.3 MB) 956 /
// 1038, 48^3 8 (7.5 MB) 1120 / 1045, 80^3 2 (8.5 MB) 1273 / 1250, 16 5733 / 3790.
constexpr long long FEW = 512, ONE_EACH = 256;

}  // namespace

template <typename T>
bool block3d(hipStream_t st, const Op3F<T>& L, const Op3F<T>& B, int first, int nj, bool pro, int upd, T s,
             Vec<const cx<T>> X, Vec<const cx<T>> Bv, Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y,
             Vec<cx<T>> Bc, int ns) {
    const int n = L.n;
    const bool rr = Bc.base != nullptr;
#define HELM_B3(F, NJ_, PRO_, UPD_, RR_, LW_, LH_, TZ_)                                                            \
    do {                                                                                                           \
        if (L.dir) launch_b<T, F, NJ_, PRO_, UPD_, RR_, LW_, LH_, TZ_, true>(st, L, B, s, X, Bv, Ec, Rho, Y, Bc, ns); \
        else launch_b<T, F, NJ_, PRO_, UPD_, RR_, LW_, LH_, TZ_, false>(st, L, B, s, X, Bv, Ec, Rho, Y, Bc, ns);   \
        return true;                                                                                               \
    } while (0)
    if (n >= BLOCK3D_N) return false;
    if ((long long)(n + 1) * (n + 1) * (n + 1) * ns * (long long)sizeof(cx<T>) > BLOCK3D_BYTES) return false;
    if (rr) {
        if (pro || upd != 0) return false;
        const int planes = n / 2 + 1;
        if ((first == F_JAC0 || first == F_HSS0 || first == F_JAC) && nj == 1) {
            using S = Block<T, F_JAC, 1, false, true, 16, 16, 1>;
            using W = Block<T, F_JAC, 1, false, true, 32, 16, 1>;
            const bool few = units_of<S>(n, planes, 1, ns) <= FEW;
            const bool wide = !few && units_of<W>(n, planes, 1, ns) <= ONE_EACH;
            if (first == F_JAC0) {
                if (few) HELM_B3(F_JAC0, 1, false, 0, true, 16, 16, 1);
                if (wide) HELM_B3(F_JAC0, 1, false, 0, true, 32, 16, 1);
                HELM_B3(F_JAC0, 1, false, 0, true, 16, 16, 2);
            }
            if (first == F_HSS0) {
                if (few) HELM_B3(F_HSS0, 1, false, 0, true, 16, 16, 1);
                HELM_B3(F_HSS0, 1, false, 0, true, 16, 16, 2);
            }
            if (wide) HELM_B3(F_JAC, 1, false, 0, true, 32, 16, 1);
            HELM_B3(F_JAC, 1, false, 0, true, 16, 16, 2);
        }
        // three stages: only while their wider halo is free
        using S = Block<T, F_JAC, 2, false, true, 16, 16, 1>;
        if (units_of<S>(n, planes, 1, ns) > FEW) return false;
        if (first == F_JAC && nj == 2) HELM_B3(F_JAC, 2, false, 0, true, 16, 16, 1);
        if (first == F_HSS && nj == 1) HELM_B3(F_HSS, 1, false, 0, true, 16, 16, 1);
        return false;
    }
    if (!pro && upd == 0 && (first == F_RESID || (first == F_JAC && nj == 1))) {
        using S = Block<T, F_JAC, 1, false, false, 16, 16, 2>;
        if (units_of<S>(n, n + 1, 2, ns) <= FEW) {
            if (first == F_RESID) HELM_B3(F_RESID, 0, false, 0, false, 16, 16, 2);
            HELM_B3(F_JAC, 1, false, 0, false, 16, 16, 2);
        }
        if (first == F_RESID) HELM_B3(F_RESID, 0, false, 0, false, 16, 16, 4);
        HELM_B3(F_JAC, 1, false, 0, false, 16, 16, 4);
    }
    if (first != F_JAC || nj != 2 || !pro) return false;
    using S = Block<T, F_JAC, 2, true, false, 16, 16, 2>;
    using W = Block<T, F_JAC, 2, true, false, 32, 16, 2>;
    if (units_of<S>(n, n + 1, 2, ns) <= FEW) {
        if (upd == 1) HELM_B3(F_JAC, 2, true, 1, false, 16, 16, 2);
        HELM_B3(F_JAC, 2, true, 0, false, 16, 16, 2);
    }
    if (units_of<W>(n, n + 1, 2, ns) <= ONE_EACH) {
        if (upd == 1) HELM_B3(F_JAC, 2, true, 1, false, 32, 16, 2);
        HELM_B3(F_JAC, 2, true, 0, false, 32, 16, 2);
    }
    if (upd == 1) HELM_B3(F_JAC, 2, true, 1, false, 16, 16, 4);
    HELM_B3(F_JAC, 2, true, 0, false, 16, 16, 4);
#undef HELM_B3
}

template bool block3d<double>(hipStream_t, const Op3F<double>&, const Op3F<double>&, int, int, bool, int, double,
                              Vec<const cxd>, Vec<const cxd>, Vec<const cxd>, Vec<cxd>, Vec<cxd>, Vec<cxd>, int);
template bool block3d<float>(hipStream_t, const Op3F<float>&, const Op3F<float>&, int, int, bool, int, float,
                             Vec<const cxf>, Vec<const cxf>, Vec<const cxf>, Vec<cxf>, Vec<cxf>, Vec<cxf>, int);

}  // namespace helm
