// Host-side launchers of the HIP kernels (internal to libhelm).
#pragma once

#include "helm_common.h"

namespace helm {

// ---- 2D P1 stencils (kernels2d.hip) ---------------------------------------
// mode: StencilMode; s: scale for MODE_RESID.  X may be null for JACOBI0,
// B null for APPLY.
template <typename T, typename TI>
void stencil2d(hipStream_t st, const Op2<T>& op, int mode, T s, Vec<const cx<TI>> X,
               Vec<const cx<T>> B, Vec<cx<T>> Y, int nslots);

// b_c = P^T r  (fine level with n cells -> n/2)
template <typename T>
void restrict2d(hipStream_t st, int n, Vec<const cx<T>> R, Vec<cx<T>> Bc, int nslots);

// b_c = P^T (b - L x), residual formed on the fly
template <typename T>
void resid_restrict2d(hipStream_t st, const Op2<T>& op, Vec<const cx<T>> X, Vec<const cx<T>> B,
                      Vec<cx<T>> Bc, int nslots);

// x += P e  (coarse level with n/2 cells -> fine n)
template <typename T>
void prolong2d(hipStream_t st, int n, Vec<const cx<T>> E, Vec<cx<T>> X, int nslots);

// ---- fused 2D multigrid kernels (kernels2d_fused.hip) ----------------------
// x = two Jacobi sweeps for L x = b from x = 0
template <typename T>
void pre0_2d(hipStream_t st, const Op2<T>& L, Vec<const cx<T>> B, Vec<cx<T>> X, int ns);
// rho = c (R - B_shift u) (u = 0 when U.base is null), written; then x as
// in pre0_2d with b = rho
template <typename T>
void hss_pre0_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Bs, T c, Vec<const cx<T>> U,
                 Vec<const cx<T>> R, Vec<cx<T>> Rho, Vec<cx<T>> X, int ns);
// x_out = S Jacobi sweeps from x_in (+ P e_c when Ec.base is set); with
// update, x_out += result instead.  S in {1, 2, 4}.
template <typename T>
void sweeps_2d(hipStream_t st, const Op2<T>& L, int S, Vec<const cx<T>> Xin, Vec<const cx<T>> Ec,
               Vec<const cx<T>> B, Vec<cx<T>> Xout, bool update, int ns);

// as pre0_2d / hss_pre0_2d, and also b_c = P^T (b - L x) on the n/2 mesh
template <typename T>
void pre0r_2d(hipStream_t st, const Op2<T>& L, Vec<const cx<T>> B, Vec<cx<T>> X, Vec<cx<T>> Bc,
              int ns);
template <typename T>
void hss_pre0r_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Bs, T c, Vec<const cx<T>> U,
                  Vec<const cx<T>> R, Vec<cx<T>> Rho, Vec<cx<T>> X, Vec<cx<T>> Bc, int ns);

// ---- register-streaming 2D kernels (kernels2d_stream.hip) -----------------
// Work split: strips of 64 columns (one per lane) x segments of H rows x
// slots; one wavefront per unit.  The units on the mesh boundary (first and
// last strip or segment) form the first `eblocks` workgroups.
struct StreamGrid {
    int H;
    unsigned strips, segs, units;
    unsigned edge_units, eblocks;
};
// x_out = S Jacobi sweeps from x_in (+ P e_c when Ec.base is set); with
// update, x_out += result; when Bc.base is set, also b_c = P^T (b - L x_out)
// on the n/2 mesh.  Supported: (S, prolong, restrict, update) in
// {(4,1,1,0), (2,1,0,1), (2,1,0,0)};
// returns false (and launches nothing) for any other.
template <typename T>
bool stream_sweeps_2d(hipStream_t st, const Op2<T>& L, int S, Vec<const cx<T>> Xin,
                      Vec<const cx<T>> Ec, Vec<const cx<T>> B, Vec<cx<T>> Xout, Vec<cx<T>> Bc,
                      bool update, int ns);
// Measuring segment heights on first use (on by default) for the calling
// thread; returns the previous setting.  Off: heights not measured yet come
// from the model, and no timing launch or event is made.
bool stream_tuning(bool on);
// two zero-guess pre-smoothing sweeps x for L x = b and b_c = P^T (b - L x);
// b given (B.base set), or b = rho = c (R - B_shift u) (U.base set) or
// rho = c R (neither), rho then written.
template <typename T>
void stream_pre_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Bs, T c, Vec<const cx<T>> U,
                   Vec<const cx<T>> R, Vec<cx<T>> Rho, Vec<const cx<T>> B, Vec<cx<T>> X,
                   Vec<cx<T>> Bc, int ns);

// ---- the same passes on LDS tiles (kernels2d_tile.hip) --------------------
// Same arguments, roundings and results as the streaming passes, for launches
// of few nodes: return false (and launch nothing) when the launch is large
// enough for the streaming kernel, and for sweeps other than (S, prolong,
// restrict, update) in {(4,1,1,0), (2,1,0,1), (2,1,0,0)}.
template <typename T>
bool tile_sweeps_2d(hipStream_t st, const Op2<T>& L, int S, Vec<const cx<T>> Xin, Vec<const cx<T>> Ec,
                    Vec<const cx<T>> B, Vec<cx<T>> Xout, Vec<cx<T>> Bc, bool update, int ns);
// b_c = P^T (b - L x), any launch size (no Dirichlet faces)
template <typename T>
void tile_restrict_2d(hipStream_t st, const Op2<T>& L, Vec<const cx<T>> X, Vec<const cx<T>> B, Vec<cx<T>> Bc, int ns);
template <typename T>
bool tile_pre_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Bs, T c, Vec<const cx<T>> U,
                 Vec<const cx<T>> R, Vec<cx<T>> Rho, Vec<const cx<T>> B, Vec<cx<T>> X, Vec<cx<T>> Bc,
                 int ns);

// Two consecutive levels (L, and Lc on the mesh of half the cells) per launch;
// false, and nothing launched, when the launch is too large for it.
// Down: x from zero and b_c = P^T (b - L x) on L, x_c from zero and
// b_cc = P^T (b_c - L_c x_c) on Lc.  Up: x_c + P e_cc and two sweeps on Lc
// (not written), whose result corrects x before S sweeps on L: two, written or
// with update added into Xout, or four, written, with P^T (b - L x) into Bcout
// (not Bc).
template <typename T>
bool tile_pre_pair_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Lc, Vec<const cx<T>> B, Vec<cx<T>> X,
                      Vec<cx<T>> Bc, Vec<cx<T>> Xc, Vec<cx<T>> Bcc, int ns);
template <typename T>
bool tile_post_pair_2d(hipStream_t st, const Op2<T>& L, const Op2<T>& Lc, int S, Vec<const cx<T>> X,
                       Vec<const cx<T>> B, Vec<const cx<T>> Xc, Vec<const cx<T>> Bc, Vec<const cx<T>> Ecc,
                       Vec<cx<T>> Xout, Vec<cx<T>> Bcout, bool update, int ns);

// ---- small-level V-cycle in LDS (kernels2d_small.hip) ---------------------
// Levels 0..nlev-1 of this record are consecutive mesh levels; the last is
// the coarsest (solved with the dense FP64 inverse).  Offsets are in
// complex elements of the dynamic LDS arena (total elements): per level two
// padded planes of (n + 3)^2 values, a and x, and from level 1 on the
// right-hand side b; off_part holds the coarse solve's FP64 partial sums.
// mdiv[l] = ceil(2^20 / (n[l] + 1)) turns a node index into its row by a
// multiply.  Level 0 has at most SMALL_THREADS SMALL_NODES nodes, level 1 and
// the coarsest at most SMALL_THREADS.
constexpr int MAX_SMALL = 8;
constexpr int SMALL_THREADS = 512, SMALL_NODES = 3;
template <typename T>
struct SmallCycle {
    int nlev;
    Op2<T> op[MAX_SMALL];
    int off_a[MAX_SMALL], off_x[MAX_SMALL], off_b[MAX_SMALL];
    int mdiv[MAX_SMALL];
    int off_part, total;
};
template <typename T>
void vcycle_small(hipStream_t st, const SmallCycle<T>& sc, size_t lds_bytes, const cxd* Ainv,
                  int nc, Vec<const cx<T>> B, Vec<cx<T>> X, int ns);

// ---- GMRES smoothing on 2D levels (kernels2d_gmres.hip) -------------------
// x = m iterations of Jacobi-left-preconditioned GMRES for L x = b from x
// (guess) or from 0; L carries the Jacobi factors of omega = 1.
constexpr int GMRES_ONE_ITS = 5;    // most iterations of the one-workgroup form
constexpr int GMRES_MAX_ITS = 20;   // most iterations
constexpr int GMRES_BLOCK = 512;    // nodes per chunk of the other one
constexpr int GMRES_MOST = 768;     // most workgroups per column of the other one
// chunks per workgroup and workgroups per column
inline int gmres_chunks(long long N) {
    return (int)((N + (long long)GMRES_BLOCK * GMRES_MOST - 1) / ((long long)GMRES_BLOCK * GMRES_MOST));
}
inline int gmres_blocks(long long N) {
    const long long nodes = (long long)GMRES_BLOCK * gmres_chunks(N);
    return (int)((N + nodes - 1) / nodes);
}
// in one workgroup per column; false (and nothing launched) for more than
// 2560 nodes or more than GMRES_ONE_ITS iterations
bool gmres_one_2d(hipStream_t st, const Op2<double>& L, int m, Vec<const cxd> B, Vec<cxd> X, bool guess, int ns);
// in 3 m + 2 launches.  Per slot: m + 1 Krylov vectors (basis, bstride apart),
// m columns of m + 1 Hessenberg entries, m + 1 norms, and per workgroup (nblk
// = gmres_blocks) m + 1 partial sums in each of part[0], part[1] and one in
// npart.
struct GmresWs {
    cxd* basis;
    long long bstride;
    cxd* hess;
    double* norms;
    cxd* part[2];
    double* npart;
    int m, nblk, chunks;  // chunks = gmres_chunks
};
void gmres_2d(hipStream_t st, const Op2<double>& L, Vec<const cxd> B, Vec<cxd> X, bool guess, const GmresWs& g, int ns);

// ---- 3D Q1 stencils (kernels3d.hip) ---------------------------------------
// tiled: levels n >= 128 run the z-marching column-tile kernel for the
// interior nodes and a boundary-node kernel; otherwise (and for
// MODE_JACOBI0) one thread per node
template <typename T, typename TI>
void stencil3d(hipStream_t st, const Op3<T>& op, int mode, T s, Vec<const cx<TI>> X,
               Vec<const cx<T>> B, Vec<cx<T>> Y, int nslots, bool tiled = true);
template <typename T>
void restrict3d(hipStream_t st, int n, Vec<const cx<T>> R, Vec<cx<T>> Bc, int nslots);
template <typename T>
void prolong3d(hipStream_t st, int n, Vec<const cx<T>> E, Vec<cx<T>> X, int nslots);

// ---- fused z-marching 3D Q1 passes (kernels3d_fused.hip) ------------------
// Operator record of a K + b M + c M_Gamma on one 3D level for the fused
// passes: the coefficients of the per-plane terms T1 = uK PK + uM PMM +
// uG PG and T0 = vK PK + vM PMM + vG PG (uK = (h/6) a, uM = (h/6) b - a/h,
// uG = (h/6) c, vK = 4 (h/6) a, vM = 4 (h/6) b + 2 a/h, vG = 4 (h/6) c),
// c for the end planes, and omega / D by the number of coordinates of the
// node on the mesh boundary (0 interior, 1 face, 2 edge, 3 corner; the
// diagonal is symmetric in the three axes).
template <typename T>
struct Op3F {
    // weights of (a0, H + V, a2) on interior columns in T1 and T0, split (the
    // K factor a is real): real parts, and the imaginary parts as
    // k * (16, 4, 1) (the in-plane mass pattern m)
    T r1[3], r0[3];
    T k1, k0;
    cx<T> cz;            // T0 of an end plane: T0 / 2 + cz m
    cx<T> e1[3], e0[3];  // changes on a boundary column (see kernels3d_fused.hip)
    cx<T> od[4];
    int n;
    unsigned dir;  // Dirichlet faces (x0=1 .. z1=32): every pass writes zero on their nodes
};
struct Grid3F {
    int tiles_x, tiles_y, slots;     // tiles per side, columns
    int tz, segs, tz_e, segs_e;      // planes per segment and segments: interior and rim tiles
    unsigned eblocks;                // workgroups of the rim tiles
    int split;                       // the rim's tiles are a list of their own (else all are "rim" tiles)
};
// first stage of a fused pass
enum Pass3First : int {
    F_APPLY = 0,  // y = L x
    F_RESID = 1,  // y = s (b - L x)
    F_JAC = 2,    // nj sweeps x + w/D (b - L x) from x (from x + P e_c with the prolongation)
    F_HSS = 3,    // rho = s (R - B u), x = w/D rho, then nj sweeps with b = rho
    F_HSS0 = 4,   // rho = s R, x = w/D rho, then nj sweeps with b = rho
    F_JAC0 = 5,   // x = w/D b, then nj sweeps
};
// One fused pass: the first stage, nj sweeps, the result to Y (upd = 1:
// Y += result), and with Bc.base set b_c = P^T (b - L x) on the n/2 mesh.
// Supported: F_APPLY and F_RESID (any TI), and (TI = T) F_JAC with nj = 1 or
// 2, with nj = 2 and pro (the input is X + P Ec; upd 0 or 1), and with the
// restriction F_JAC with nj = 0 (Y unused), F_HSS0 and F_JAC0 with nj = 1.  X,
// Bv, Ec, Rho, Y as the form needs (rho goes to Rho); Y must not alias X.
// Returns false (and launches nothing) for an unsupported combination.
template <typename T, typename TI>
bool pass3d(hipStream_t st, const Op3F<T>& L, int first, int nj, bool pro, int upd, T s, Vec<const cx<TI>> X,
            Vec<const cx<T>> Bv, Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y, Vec<cx<T>> Bc, int nslots);

// y = w/D b on any level: the sweep from a zero guess alone.
template <typename T>
void jacobi0_3d(hipStream_t st, const Op3F<T>& L, Vec<const cx<T>> B, Vec<cx<T>> Y, int ns);

// ---- the same stages on small 3D levels (kernels3d_block.hip) --------------
// One pass on whole blocks of the mesh; arguments as for pass3d, B the second
// operator of F_HSS.  Supported: F_RESID, F_JAC with nj = 1, with nj = 2 and
// pro (upd 0 or 1), and with the restriction F_JAC0 and F_HSS0 with nj = 1,
// F_JAC with nj = 1 or 2 and F_HSS with nj = 1.  Returns false (and launches
// nothing) for any other, for a level of BLOCK3D_N cells or more, for a launch
// of more than BLOCK3D_BYTES a vector, and where the three stages of the last
// two would not fit the chip at once.
constexpr int BLOCK3D_N = 96;  // cells per side from which the marching passes are faster
constexpr long long BLOCK3D_BYTES = 7000000;  // bytes of a vector (all columns) from which they are below that
template <typename T>
bool block3d(hipStream_t st, const Op3F<T>& L, const Op3F<T>& B, int first, int nj, bool pro, int upd, T s,
             Vec<const cx<T>> X, Vec<const cx<T>> Bv, Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y,
             Vec<cx<T>> Bc, int ns);

// ---- the marching passes with the block passes' roundings (kernels3d_columns.hip)
// For the launches below BLOCK3D_N that block3d declines; arguments as for
// pass3d.  Supported: F_RESID, F_JAC with nj = 2, with or without pro (then upd
// 0 or 1), and with the restriction F_JAC with nj = 0, F_HSS0 and F_JAC0 with
// nj = 1.  Returns false (and launches nothing) for any other.
template <typename T>
bool columns3d(hipStream_t st, const Op3F<T>& L, int first, int nj, bool pro, int upd, T s, Vec<const cx<T>> X,
               Vec<const cx<T>> Bv, Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y, Vec<cx<T>> Bc, int ns);

// ---- mixed [DG0]^2 x P1 formulation (kernels2d_mixed.hip) ------------------
// X, B, Y of mixed vectors [u | sigma] (sigma after the N = (n+1)^2 nodes).
// y = sb B_u + Op u + G^T (sa sigma + sg g) at the nodes (B, G nullable; G
// holds 4 n^2 triangle values per slot); Y addresses node vectors.
template <typename T, typename TI>
void mixed_nodes(hipStream_t st, const Op2<T>& op, cx<T> sb, cx<T> sa, cx<T> sg,
                 Vec<const cx<TI>> X, Vec<const cx<T>> B, Vec<const cx<T>> G, Vec<cx<T>> Y,
                 int nslots);
// sigma rows: y = area (s sigma - grad u)  or  B - area (s sigma - grad u)
template <typename T, typename TI>
void mixed_tris(hipStream_t st, int n, int mode, cx<T> s, Vec<const cx<TI>> X, Vec<const cx<T>> B,
                Vec<cx<T>> Y, int nslots);
// g = nukp sigma + nu grad u + c R_sigma / area
template <typename T>
void mixed_g(hipStream_t st, int n, cx<T> nukp, T nu, T c, Vec<const cx<T>> X, Vec<const cx<T>> R,
             Vec<cx<T>> G, int nslots);
// sigma = inv (grad u + g)
template <typename T>
void mixed_sigma(hipStream_t st, int n, cx<T> inv, Vec<const cx<T>> X, Vec<const cx<T>> G,
                 Vec<cx<T>> Y, int nslots);

// ---- vector kernels (kernels_vec.hip) ----------------------------------------
// x = Ainv b on the coarsest mesh, Ainv dense complex FP64 (nc x nc, row-major)
template <typename T>
void coarse_apply(hipStream_t st, const cxd* Ainv, int nc, Vec<const cx<T>> B, Vec<cx<T>> X,
                  int nslots);
// y = x (type conversion allowed)
template <typename TO, typename TI>
void copy_cast(hipStream_t st, long long N, Vec<const cx<TI>> X, Vec<cx<TO>> Y, int nslots);
// y += alpha x
template <typename T>
void axpy1(hipStream_t st, long long N, T alpha, Vec<const cx<T>> X, Vec<cx<T>> Y, int nslots);
// y = alpha x, alpha real per slot: y = x / div[slot]  (div read on device)
void scale_inv(hipStream_t st, long long N, Vec<const cxd> X, Vec<cxd> Y, const double* div,
               int div_stride, int nslots);
// partial dot products: part[slot][i][blk] = sum_{n in blk} conj(V_i[n]) w[n], i < m
// V_i at Vb.at(slot) + i*N
int multidot_blocks(long long N);
// mlen (nullable, device): per-slot vector count <= m; m sets the layout.
// wpart (nullable): also wpart[slot][blk] = sum_{n in blk} |w[n]|^2.
// flag (nullable, device): slots with flag[slot] == 0 are skipped.
void multidot(hipStream_t st, long long N, int m, const int* mlen, Vec<const cxd> V,
              Vec<const cxd> W, cxd* part, int nslots, double* wpart = nullptr,
              const int* flag = nullptr);
// reduce part over blocks: out[slot*ostride + i] (+)= sum_blk part[slot][i][blk];
// slots with flag[slot] == 0 get 0 (or keep out when accumulating)
void reduce_parts(hipStream_t st, int m, const int* mlen, int nblk, const cxd* part, cxd* out,
                  int ostride, int accumulate, int nslots, const int* flag = nullptr);
// flag[slot] = 1 when |w|^2 - |h|^2 < |w|^2 / 2 (|w|^2 from multidot's wpart,
// h the first Gram-Schmidt pass's coefficients), else 0
void reorth_flag(hipStream_t st, int m, const int* mlen, int nblk, const double* wpart,
                 const cxd* h, int hstride, int* flag, int nslots);
// w -= sum_{i<m} h[slot*hstride + i] V_i; slots with flag[slot] == 0 skipped
void multi_axpy(hipStream_t st, long long N, int m, const int* mlen, Vec<const cxd> V,
                const cxd* h, int hstride, Vec<cxd> W, int nslots, const int* flag = nullptr);
// squared norm partials: part[slot][blk] = sum |w|^2 ; reduced into out[slot*ostride]
void norm2(hipStream_t st, long long N, Vec<const cxd> W, double* part, double* out, int ostride,
           int nslots);
// x += sum_{i<m} y[slot*ystride + i] Z_i  (Z in FP64 or FP32)
template <typename TZ>
void update_solution(hipStream_t st, long long N, int m, const int* mlen, Vec<const cx<TZ>> Z,
                     const cxd* y, int ystride, Vec<cxd> X, int nslots);
// m-step GMRES least squares per slot (Hessenberg hu, norms hn, see
// kernels_vec.hip); y[slot*m + i]; m <= 20
void gmres_lsq(hipStream_t st, int m, cxd* hu, int hs, const double* hn, cxd* y, int nslots);
// b = f (real -> complex)
void real_to_complex(hipStream_t st, long long N, const double* f, cxd* b, int nslots);

}  // namespace helm
