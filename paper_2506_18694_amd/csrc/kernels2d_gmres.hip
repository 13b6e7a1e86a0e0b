// GMRES smoothing of the W-cycle on 2D levels in few launches.
//
// One smoothing is m iterations of Jacobi-left-preconditioned GMRES: an
// Arnoldi process on D^{-1} L from r = D^{-1}(b - L x) with classical
// Gram-Schmidt applied twice, the (m + 1) x m least-squares problem, x += V y.
// Launched one operation at a time it is 56 kernels of 2 to 5 us for m = 5,
// whatever the level.
//
// Levels of up to 2560 nodes run the whole smoothing in one workgroup per
// column (k_gmres_one): the Krylov vectors stay in registers, five nodes per
// thread, one LDS plane serves the stencil and the inner products meet in LDS.
// Larger levels take 3 m + 2 launches (k_gmres_start, per iteration
// k_gmres_apply and two k_gmres_orth, k_gmres_finish): every inner product is
// left as one partial sum per workgroup, which the next launch's workgroups
// add up themselves, so that a reduction costs no launch of its own.  That is
// as many reads as the square of the workgroups, so a column has GMRES_MOST
// workgroups at most, which then take several chunks of nodes each (MANY): with
// one chunk each a smoothing took 3.20 ms at 2048^2 and 38.3 at 4096^2, where
// 56 launches took 1.60 and 6.76; now 1.11 and 5.14 (with at most 256 workgroups
// 1.28 and 7.45, with 512 1.11 and 4.97, with 1024 1.14 and 5.16).  The count
// follows from the nodes alone: a column's sums do not depend on how many
// columns share the launch.  Both forms keep the Krylov vectors unnormalised,
// w_0 = r and w_{j+1} the vector before its division by h_{j+1,j}, with their
// norms beside them: V_i = w_i / |w_i| enters through its scale, and no pass
// normalises.
// Measured per smoothing (m = 5, one column): about 190 us as 56 launches; 19 us
// in one workgroup at 576 nodes, 33 at 2209, and 75 us as 17 launches at 8649
// to 34225, 115 at 512^2 (270 as 56).  The one-workgroup form is a chain of 16
// inner products; summed over the wavefront with LDS shuffles they took 34 and
// 48 us of it.
#include "launch.h"

namespace helm {

namespace {

constexpr int WAVE = 64;

__device__ __forceinline__ cxd zero_c() { return mk(0.0, 0.0); }
__device__ __forceinline__ cxd sel(bool c, cxd a, cxd b) { return mk(c ? a.x : b.x, c ? a.y : b.y); }
// 1 / n, 0 for a zero vector (an invariant Krylov space)
__device__ __forceinline__ double inv_norm(double n) { return n != 0.0 ? 1.0 / n : 0.0; }

// A node's row of the operator with values outside the mesh taken as zero:
// centre, east / west, north / south (the "/" diagonal's weight is the same on
// every node), and its Jacobi factor.
struct Row {
    cxd c, x, y, jf;
};
__device__ __forceinline__ Row row_of(const Op2<double>& op, int i, int j) {
    const int n = op.n;
    const bool cb = (i == 0) | (i == n), rb = (j == 0) | (j == n), lo = (i == 0) == (j == 0);
    const cxd z = zero_c();
    Row r;
    r.c = op.wC + sel(cb, op.dC, z) + sel(rb, op.dC, z) + sel(cb & rb, sel(lo, op.kA, op.kB), z);
    r.y = op.wAx + sel(cb, op.dN, z);
    r.x = op.wAx + sel(rb, op.dN, z);
    r.jf = sel(cb & rb, sel(lo, op.odA, op.odB), sel(cb | rb, op.odE, op.odC));
    return r;
}

// Sums over the wavefront without LDS.  The lane swaps of gfx950 exchange one
// half (or every second row of 16 lanes) of one register with the other half
// of another: adding the two results halves at once the lanes to be summed and
// the values a lane holds.  The last four steps, within a row, are DPP moves.
template <int W>
__device__ __forceinline__ double swap_add(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    unsigned r[2][2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const unsigned p = (unsigned)(x >> (32 * k)), q = (unsigned)(y >> (32 * k));
        if constexpr (W == 32) {
            const auto v = __builtin_amdgcn_permlane32_swap(p, q, false, false);
            r[0][k] = v[0];
            r[1][k] = v[1];
        } else {
            const auto v = __builtin_amdgcn_permlane16_swap(p, q, false, false);
            r[0][k] = v[0];
            r[1][k] = v[1];
        }
    }
    return __builtin_bit_cast(double, ((unsigned long long)r[0][1] << 32) | r[0][0]) +
           __builtin_bit_cast(double, ((unsigned long long)r[1][1] << 32) | r[1][0]);
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double a) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)x, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), CTRL, 0xf, 0xf, true);
    return a + __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double row_sum(double a) {
    a = dpp_add<0xB1>(a);    // quad_perm 1 0 3 2
    a = dpp_add<0x4E>(a);    // quad_perm 2 3 0 1
    a = dpp_add<0x141>(a);   // row_half_mirror
    return dpp_add<0x140>(a);  // row_mirror
}
// The sums over the wavefront of P values per lane (P a power of two >= 2):
// lane l's row then holds the values (l / 32) P / 2 + ... of `value_at`, all of
// its lanes the same.
template <int P>
struct WaveSums {
    static constexpr int H = P >= 4 ? P / 4 : 1;  // values a row holds
    double v[H];
    __device__ __forceinline__ explicit WaveSums(const double (&in)[P]) {
        double t[P / 2];
#pragma unroll
        for (int k = 0; k < P / 2; ++k) t[k] = swap_add<32>(in[k], in[k + P / 2]);
        if constexpr (P >= 4) {
#pragma unroll
            for (int k = 0; k < H; ++k) v[k] = row_sum(swap_add<16>(t[k], t[k + H]));
        } else {
            v[0] = row_sum(swap_add<16>(t[0], t[0]));
        }
    }
    // index of v[k] on this lane
    static __device__ __forceinline__ int value_at(int lane, int k) {
        return (lane >> 5) * (P / 2) + (P >= 4 ? ((lane >> 4) & 1) * (P / 4) : 0) + k;
    }
    // every value once, to out[index]
    __device__ __forceinline__ void write(double* out) const {
        const int lane = (int)threadIdx.x % WAVE;
        if (lane % 16 == 0 && (P >= 4 || (lane & 16) == 0)) {
#pragma unroll
            for (int k = 0; k < H; ++k) out[value_at(lane, k)] = v[k];
        }
    }
};
constexpr int pow2(int c) { return c <= 2 ? 2 : c <= 4 ? 4 : c <= 8 ? 8 : 16; }

// ---- one workgroup per column ------------------------------------------------
constexpr int OT = 512;  // threads

// The sums over the workgroup of C values per thread, in out[0 .. C) for every
// thread after the closing barrier.
template <int C>
__device__ __forceinline__ void block_sums(const double (&in)[C], double* part, double* out) {
    constexpr int P = pow2(C);
    double v[P];
#pragma unroll
    for (int k = 0; k < P; ++k) v[k] = k < C ? in[k] : 0.0;
    WaveSums<P>(v).write(part + (int)threadIdx.x / WAVE * 16);
    __syncthreads();
    if ((int)threadIdx.x < C) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < OT / WAVE; ++w) t += part[w * 16 + threadIdx.x];
        out[threadIdx.x] = t;
    }
    __syncthreads();
}

template <int U>
struct IC {
    static constexpr int value = U;
};
template <int A, int B, typename F>
__device__ __forceinline__ void unrolled(F f) {
    if constexpr (A < B) {
        f(IC<A>{});
        unrolled<A + 1, B>(f);
    }
}

// y of the least-squares problem min |beta e_1 - H y|, times the inverse norms
// (the coefficients of the unnormalised vectors): Givens rotations on the
// columns (column j at hs + j stride), back substitution; a zero pivot gives 0.
// Every lane of one wavefront does the same work in registers.
template <int MM>
__device__ __forceinline__ void least_squares(int m, const cxd* hs, int stride, const double* nrm, cxd* y) {
    cxd g[MM + 1], cs[MM], sn[MM], h[MM][MM];
#pragma unroll
    for (int j = 0; j < MM; ++j)
#pragma unroll
        for (int i = 0; i <= j; ++i) h[j][i] = j < m ? hs[j * stride + i] : zero_c();
    g[0] = mk(nrm[0], 0.0);
    unrolled<0, MM>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (j >= m) return;
#pragma unroll
        for (int i = 0; i < j; ++i) {
            const cxd a = h[j][i], c = h[j][i + 1];
            h[j][i] = cs[i] * a + sn[i] * c;
            h[j][i + 1] = mk(-sn[i].x, sn[i].y) * a + mk(cs[i].x, -cs[i].y) * c;
        }
        const cxd a = h[j][j];
        const double c = nrm[j + 1], den = sqrt(a.x * a.x + a.y * a.y + c * c), inv = inv_norm(den);
        cs[j] = den == 0.0 ? mk(1.0, 0.0) : mk(a.x * inv, -a.y * inv);
        sn[j] = mk(c * inv, 0.0);
        if (den != 0.0) h[j][j] = mk(den, 0.0);
        g[j + 1] = mk(-sn[j].x, sn[j].y) * g[j];
        g[j] = cs[j] * g[j];
    });
    cxd ys[MM];
    unrolled<0, MM>([&](auto ic) {
        constexpr int i = MM - 1 - decltype(ic)::value;
        ys[i] = zero_c();
        if (i >= m) return;
        cxd t = g[i];
#pragma unroll
        for (int q = i + 1; q < MM; ++q)
            if (q < m) t = t - h[q][i] * ys[q];
        const cxd d = h[i][i];
        if (!(d.x == 0.0 && d.y == 0.0)) ys[i] = cdiv(t, d);
        if (threadIdx.x == 0) y[i] = inv_norm(nrm[i]) * ys[i];
    });
}

// NPT nodes per thread; m <= GMRES_ONE_ITS iterations.
template <int NPT>
__global__ __launch_bounds__(OT) void k_gmres_one(Op2<double> L, int m, Vec<const cxd> Bv, Vec<cxd> Xv, int guess) {
    constexpr int MM = GMRES_ONE_ITS;
    extern __shared__ __align__(16) unsigned char raw_lds[];
    const int n = L.n, W = n + 1, S = n + 3, N = W * W;
    cxd* pl = reinterpret_cast<cxd*>(raw_lds);                 // the plane with a rim of zeros
    __shared__ double part[(OT / WAVE) * 16], sums[2 * (MM + 1)];
    // the Hessenberg columns, the norms of the w_i and their inverses
    __shared__ cxd hs[MM * MM], y[MM];
    __shared__ double nrm[MM + 1], sc[MM + 1];
    const int slot = blockIdx.x, tid = threadIdx.x;
    const cxd* b = Bv.at(slot);
    cxd* x = Xv.at(slot);
    cxd w[MM + 1][NPT];
    int pi[NPT], pj[NPT];
    bool on[NPT];
    for (int q = tid; q < S * S; q += OT) pl[q] = zero_c();
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        const int q = tid + u * OT;
        on[u] = q < N;
        pj[u] = on[u] ? q / W : 0;
        pi[u] = on[u] ? q - pj[u] * W : 0;
    }
    __syncthreads();
    auto place = [&](int u) { return (pj[u] + 1) * S + pi[u] + 1; };
    auto put = [&](auto value) {
#pragma unroll
        for (int u = 0; u < NPT; ++u)
            if (on[u]) pl[place(u)] = value(u);
        __syncthreads();
    };
    // L v at this thread's node u, v in the plane
    auto apply = [&](int u, const Row& r) {
        const cxd* q = pl + place(u);
        return cfma(L.wDg, q[S + 1] + q[-S - 1], cfma(r.x, q[1] + q[-1], cfma(r.y, q[S] + q[-S], r.c * q[0])));
    };
    auto norm_of = [&](const cxd (&v)[NPT]) {
        double s[1] = {0.0};
#pragma unroll
        for (int u = 0; u < NPT; ++u) s[0] += v[u].x * v[u].x + v[u].y * v[u].y;
        block_sums<1>(s, part, sums);
    };
    // thread 0 notes |w_i|; read after the next barrier
    auto note = [&](int i) {
        if (tid == 0) {
            nrm[i] = sqrt(sums[0]);
            sc[i] = inv_norm(nrm[i]);
        }
    };
    // r = D^{-1}(b - L x)
    if (guess) put([&](int u) { return x[tid + u * OT]; });
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        const Row r = row_of(L, pi[u], pj[u]);
        cxd v = b[on[u] ? tid + u * OT : 0];
        if (guess) v = v - apply(u, r);
        w[0][u] = on[u] ? r.jf * v : zero_c();
    }
    norm_of(w[0]);
    note(0);
    unrolled<0, MM>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (j >= m) return;
        put([&](int u) { return w[j][u]; });
#pragma unroll
        for (int u = 0; u < NPT; ++u) {
            const Row r = row_of(L, pi[u], pj[u]);
            w[j + 1][u] = on[u] ? sc[j] * (r.jf * apply(u, r)) : zero_c();
        }
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            double d[2 * (j + 1)];
#pragma unroll
            for (int i = 0; i <= j; ++i) {
                cxd a = zero_c();
#pragma unroll
                for (int u = 0; u < NPT; ++u) a = a + cjmul(w[i][u], w[j + 1][u]);
                d[2 * i] = a.x;
                d[2 * i + 1] = a.y;
            }
            block_sums<2 * (j + 1)>(d, part, sums);
#pragma unroll
            for (int i = 0; i <= j; ++i) {
                const cxd hi = sc[i] * mk(sums[2 * i], sums[2 * i + 1]), c = sc[i] * hi;
                if (tid == 0) hs[j * MM + i] = pass == 0 ? hi : hs[j * MM + i] + hi;
#pragma unroll
                for (int u = 0; u < NPT; ++u) w[j + 1][u] = w[j + 1][u] - c * w[i][u];
            }
        }
        norm_of(w[j + 1]);
        note(j + 1);
    });
    __syncthreads();
    if (tid < WAVE) least_squares<MM>(m, hs, MM, nrm, y);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        if (!on[u]) continue;
        cxd v = guess ? x[tid + u * OT] : zero_c();
#pragma unroll
        for (int i = 0; i < MM; ++i)
            if (i < m) v = cfma(y[i], w[i][u], v);
        x[tid + u * OT] = v;
    }
}

// ---- many workgroups per column ----------------------------------------------
constexpr int BS = 256, NPB = 2;  // threads, nodes per thread
constexpr int GROUP = 4;          // inner products per reduction
static_assert(GMRES_BLOCK == BS * NPB, "nodes per workgroup");

// sum of C values per thread over the workgroup, valid in thread 0
template <int C>
__device__ __forceinline__ void block_sum0(double (&v)[C], double* lds) {
    constexpr int P = pow2(C);
    double a[P];
#pragma unroll
    for (int k = 0; k < P; ++k) a[k] = k < C ? v[k] : 0.0;
    const WaveSums<P> s(a);
    __syncthreads();
    s.write(lds + (int)threadIdx.x / WAVE * 16);
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < C; ++k) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < BS / WAVE; ++w) t += lds[w * 16 + k];
            v[k] = t;
        }
    }
}

// |w| from its partial sums of squares, for every thread
__device__ __forceinline__ double norm_from(const double* p, int nblk, double* lds) {
    double v[1] = {0.0};
    for (int q = threadIdx.x; q < nblk; q += BS) v[0] += p[q];
    block_sum0<1>(v, lds);
    if (threadIdx.x == 0) lds[0] = sqrt(v[0]);
    __syncthreads();
    const double r = lds[0];
    __syncthreads();
    return r;
}

// L v at node (i, j), v in memory
__device__ __forceinline__ cxd apply_mem(const Op2<double>& L, const Row& r, const cxd* v, int i, int j) {
    const int n = L.n, W = n + 1, p = j * W + i;
    const bool hE = i < n, hW = i > 0, hN = j < n, hS = j > 0;
    const cxd z = zero_c();
    const cxd c = v[p], e = sel(hE, v[hE ? p + 1 : p], z), w = sel(hW, v[hW ? p - 1 : p], z);
    const cxd nn = sel(hN, v[hN ? p + W : p], z), ss = sel(hS, v[hS ? p - W : p], z);
    const bool hNE = hE & hN, hSW = hW & hS;
    const cxd ne = sel(hNE, v[hNE ? p + W + 1 : p], z), sw = sel(hSW, v[hSW ? p - W - 1 : p], z);
    return cfma(L.wDg, ne + sw, cfma(r.x, e + w, cfma(r.y, nn + ss, r.c * c)));
}

// this thread's nodes of chunk r of the workgroup
__device__ __forceinline__ long long node_at(int chunks, int blk, int r, int u) {
    return (((long long)blk * chunks + r) * NPB + u) * BS + threadIdx.x;
}

// partial sums of conj(w_i) w over this workgroup's nodes, i < cnt, w the
// vector cnt: part[i nblk + blk]; wl: w on the last chunk
__device__ __forceinline__ void dots(const cxd* G, long long N, int cnt, const cxd (&wl)[NPB], cxd* part,
                                     int nblk, int chunks, int blk, double* lds) {
    for (int i0 = 0; i0 < cnt; i0 += GROUP) {
        double d[2 * GROUP];
#pragma unroll
        for (int k = 0; k < 2 * GROUP; ++k) d[k] = 0.0;
        for (int r = 0; r < chunks; ++r) {
            long long t[NPB];
            cxd w[NPB];
#pragma unroll
            for (int u = 0; u < NPB; ++u) {
                t[u] = node_at(chunks, blk, r, u);
                w[u] = wl[u];
                if (r + 1 < chunks) w[u] = t[u] < N ? G[(long long)cnt * N + t[u]] : zero_c();
            }
#pragma unroll
            for (int k = 0; k < GROUP; ++k) {
                if (i0 + k >= cnt) continue;
                const cxd* v = G + (long long)(i0 + k) * N;
#pragma unroll
                for (int u = 0; u < NPB; ++u) {
                    const cxd a = cjmul(v[t[u] < N ? t[u] : 0], w[u]);  // w is zero past the end
                    d[2 * k] += a.x;
                    d[2 * k + 1] += a.y;
                }
            }
        }
        block_sum0<2 * GROUP>(d, lds);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < GROUP; ++k)
                if (i0 + k < cnt) part[(long long)(i0 + k) * nblk + blk] = mk(d[2 * k], d[2 * k + 1]);
        }
    }
}

// w_0 = D^{-1}(b - L x) (x = 0 without a guess) and its partial sums of squares
template <bool MANY>
__global__ __launch_bounds__(BS) void k_gmres_start(Op2<double> L, Vec<const cxd> Bv, Vec<const cxd> Xv, int guess,
                                                    GmresWs g) {
    __shared__ double lds[(BS / WAVE) * 16];
    const int slot = blockIdx.x / g.nblk, blk = blockIdx.x % g.nblk, chunks = MANY ? g.chunks : 1;
    const int W = L.n + 1;
    const long long N = (long long)W * W;
    const cxd *b = Bv.at(slot), *x = Xv.at(slot);
    cxd* G = g.basis + slot * g.bstride;
    double s[1] = {0.0};
    for (int r = 0; r < chunks; ++r) {
#pragma unroll
        for (int u = 0; u < NPB; ++u) {
            const long long t = node_at(chunks, blk, r, u);
            if (t >= N) continue;
            const int j = (int)(t / W), i = (int)(t - (long long)j * W);
            const Row row = row_of(L, i, j);
            cxd v = b[t];
            if (guess) v = v - apply_mem(L, row, x, i, j);
            v = row.jf * v;
            G[t] = v;
            s[0] += v.x * v.x + v.y * v.y;
        }
    }
    block_sum0<1>(s, lds);
    if (threadIdx.x == 0) g.npart[(long long)slot * g.nblk + blk] = s[0];
}

// w_{j+1} = D^{-1} L w_j / |w_j|, the partial inner products with w_0 .. w_j;
// |w_j| is added up from its partial sums
template <bool MANY>
__global__ __launch_bounds__(BS) void k_gmres_apply(Op2<double> L, int j, GmresWs g) {
    __shared__ double lds[(BS / WAVE) * 16];
    const int slot = blockIdx.x / g.nblk, blk = blockIdx.x % g.nblk, chunks = MANY ? g.chunks : 1;
    const int W = L.n + 1;
    const long long N = (long long)W * W;
    cxd* G = g.basis + slot * g.bstride;
    const double nrm = norm_from(g.npart + (long long)slot * g.nblk, g.nblk, lds), sc = inv_norm(nrm);
    if (blk == 0 && threadIdx.x == 0) g.norms[slot * (g.m + 1) + j] = nrm;
    cxd w[NPB];
    for (int r = 0; r < chunks; ++r) {
#pragma unroll
        for (int u = 0; u < NPB; ++u) {
            const long long t = node_at(chunks, blk, r, u);
            w[u] = zero_c();
            if (t >= N) continue;
            const int jj = (int)(t / W), i = (int)(t - (long long)jj * W);
            const Row row = row_of(L, i, jj);
            w[u] = sc * (row.jf * apply_mem(L, row, G + (long long)j * N, i, jj));
            G[(long long)(j + 1) * N + t] = w[u];
        }
    }
    dots(G, N, j + 1, w, g.part[0] + (long long)slot * (g.m + 1) * g.nblk, g.nblk, chunks, blk, lds);
}

// One Gram-Schmidt pass on w_{j+1}: the coefficients from the partial inner
// products, w -= sum V_i h_i; the first pass leaves the inner products of the
// second, the second the partial sums of squares.  C: j + 1, whose vectors are
// then used from registers, those of the first chunk requested before the
// coefficients are added up; 0: any count.
template <int C, bool MANY>
__global__ __launch_bounds__(BS) void k_gmres_orth(long long N, int j, int pass, GmresWs g) {
    __shared__ double lds[(BS / WAVE) * 16];
    __shared__ cxd c[GMRES_MAX_ITS];
    const int slot = blockIdx.x / g.nblk, blk = blockIdx.x % g.nblk, chunks = MANY ? g.chunks : 1;
    cxd* G = g.basis + slot * g.bstride;
    const cxd* part = g.part[pass] + (long long)slot * (g.m + 1) * g.nblk;
    const int lane = (int)threadIdx.x % WAVE, wv = (int)threadIdx.x / WAVE;
    cxd w[NPB], v[C > 0 ? C : 1][NPB];
    long long t[NPB];
    auto load = [&](int r) {
#pragma unroll
        for (int u = 0; u < NPB; ++u) {
            t[u] = node_at(chunks, blk, r, u);
            const long long p = t[u] < N ? t[u] : 0;
            w[u] = G[(long long)(j + 1) * N + p];
#pragma unroll
            for (int i = 0; i < C; ++i) v[i][u] = G[(long long)i * N + p];
        }
    };
    load(0);
    for (int i = wv; i <= j; i += BS / WAVE) {  // a wavefront per coefficient
        double d[2] = {0.0, 0.0};
        for (int q = lane; q < g.nblk; q += WAVE) {
            const cxd a = part[(long long)i * g.nblk + q];
            d[0] += a.x;
            d[1] += a.y;
        }
        const double s = WaveSums<2>(d).v[0], im = __shfl(s, WAVE / 2, WAVE);
        if (lane == 0) {
            const double sc = inv_norm(g.norms[slot * (g.m + 1) + i]);
            const cxd h = sc * mk(s, im);
            c[i] = sc * h;
            if (blk == 0) {
                cxd* hp = g.hess + (long long)slot * g.m * (g.m + 1) + j * (g.m + 1) + i;
                *hp = pass == 0 ? h : *hp + h;
            }
        }
    }
    __syncthreads();
    double s[1] = {0.0}, d[C > 0 ? 2 * C : 1] = {};
    for (int r = 0; r < chunks; ++r) {
        if (r > 0) load(r);
#pragma unroll
        for (int u = 0; u < NPB; ++u) {
            if (t[u] >= N) {
                w[u] = zero_c();
                continue;
            }
            if constexpr (C > 0) {
#pragma unroll
                for (int i = 0; i < C; ++i) w[u] = w[u] - c[i] * v[i][u];
            } else {
                for (int i = 0; i <= j; ++i) w[u] = w[u] - c[i] * G[(long long)i * N + t[u]];
            }
            G[(long long)(j + 1) * N + t[u]] = w[u];
            s[0] += w[u].x * w[u].x + w[u].y * w[u].y;
        }
        if constexpr (C > 0) {
            if (pass == 0) {
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    cxd a = mk(d[2 * i], d[2 * i + 1]);
#pragma unroll
                    for (int u = 0; u < NPB; ++u) a = a + cjmul(v[i][u], w[u]);
                    d[2 * i] = a.x;
                    d[2 * i + 1] = a.y;
                }
            }
        }
    }
    if (pass == 1) {
        block_sum0<1>(s, lds);
        if (threadIdx.x == 0) g.npart[(long long)slot * g.nblk + blk] = s[0];
        return;
    }
    cxd* out = g.part[1] + (long long)slot * (g.m + 1) * g.nblk;
    if constexpr (C > 0) {
        block_sum0<2 * C>(d, lds);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int i = 0; i < C; ++i) out[(long long)i * g.nblk + blk] = mk(d[2 * i], d[2 * i + 1]);
        }
    } else {
        dots(G, N, j + 1, w, out, g.nblk, chunks, blk, lds);
    }
}

// The least-squares problem (every workgroup solves it for itself) and
// x (+)= V y.
template <bool MANY>
__global__ __launch_bounds__(BS) void k_gmres_finish(long long N, int guess, Vec<cxd> Xv, GmresWs g) {
    __shared__ double lds[(BS / WAVE) * 16];
    __shared__ cxd H[GMRES_MAX_ITS * (GMRES_MAX_ITS + 1)], gv[GMRES_MAX_ITS + 1], cs[GMRES_MAX_ITS], sn[GMRES_MAX_ITS];
    __shared__ cxd y[GMRES_MAX_ITS];
    __shared__ double nr[GMRES_MAX_ITS + 1];
    const int slot = blockIdx.x / g.nblk, blk = blockIdx.x % g.nblk, m = g.m, chunks = MANY ? g.chunks : 1;
    const double last = norm_from(g.npart + (long long)slot * g.nblk, g.nblk, lds);
    for (int q = threadIdx.x; q < m * (m + 1); q += BS) H[q] = g.hess[(long long)slot * m * (m + 1) + q];
    for (int q = threadIdx.x; q <= m; q += BS) nr[q] = q < m ? g.norms[slot * (m + 1) + q] : last;
    __syncthreads();
    if (m <= GMRES_ONE_ITS) {
        if ((int)threadIdx.x < WAVE) least_squares<GMRES_ONE_ITS>(m, H, m + 1, nr, y);
    } else if (threadIdx.x == 0) {
        gv[0] = mk(nr[0], 0.0);
        for (int j = 0; j < m; ++j) {
            cxd* col = H + j * (m + 1);
            for (int i = 0; i < j; ++i) {
                const cxd a = col[i], b = col[i + 1];
                col[i] = cs[i] * a + sn[i] * b;
                col[i + 1] = mk(-sn[i].x, sn[i].y) * a + mk(cs[i].x, -cs[i].y) * b;
            }
            const cxd a = col[j];
            const double b = nr[j + 1], den = sqrt(a.x * a.x + a.y * a.y + b * b), inv = inv_norm(den);
            cs[j] = den == 0.0 ? mk(1.0, 0.0) : mk(a.x * inv, -a.y * inv);
            sn[j] = mk(b * inv, 0.0);
            if (den != 0.0) col[j] = mk(den, 0.0);
            gv[j + 1] = mk(-sn[j].x, sn[j].y) * gv[j];
            gv[j] = cs[j] * gv[j];
        }
        for (int i = m - 1; i >= 0; --i) {
            cxd s = gv[i];
            for (int q = i + 1; q < m; ++q) s = s - H[q * (m + 1) + i] * y[q];
            const cxd d = H[i * (m + 1) + i];
            y[i] = (d.x == 0.0 && d.y == 0.0) ? zero_c() : cdiv(s, d);
        }
        for (int i = 0; i < m; ++i) y[i] = inv_norm(nr[i]) * y[i];
    }
    __syncthreads();
    const cxd* G = g.basis + slot * g.bstride;
    cxd* x = Xv.at(slot);
    for (int r = 0; r < chunks; ++r) {
#pragma unroll
        for (int u = 0; u < NPB; ++u) {
            const long long t = node_at(chunks, blk, r, u);
            if (t >= N) continue;
            cxd v = guess ? x[t] : zero_c();
            for (int i = 0; i < m; ++i) v = cfma(y[i], G[(long long)i * N + t], v);
            x[t] = v;
        }
    }
}

}  // namespace

bool gmres_one_2d(hipStream_t st, const Op2<double>& L, int m, Vec<const cxd> B, Vec<cxd> X, bool guess, int ns) {
    const long long N = (long long)(L.n + 1) * (L.n + 1);
    const int S = L.n + 3;
    if (N > 5 * OT || m > GMRES_ONE_ITS) return false;
    const size_t lds = sizeof(cxd) * (size_t)S * S;
    if (N <= 2 * OT) k_gmres_one<2><<<ns, OT, lds, st>>>(L, m, B, X, guess ? 1 : 0);
    else k_gmres_one<5><<<ns, OT, lds, st>>>(L, m, B, X, guess ? 1 : 0);
    return true;
}

template <bool MANY>
static void gmres_launch(hipStream_t st, const Op2<double>& L, Vec<const cxd> B, Vec<cxd> X, bool guess, const GmresWs& g,
                         int ns) {
    const long long N = (long long)(L.n + 1) * (L.n + 1);
    const unsigned nb = (unsigned)(g.nblk * ns);
    const int gs = guess ? 1 : 0;
    k_gmres_start<MANY><<<nb, BS, 0, st>>>(L, B, Vec<const cxd>{X.base, X.cstride, X.off, X.cols}, gs, g);
    for (int j = 0; j < g.m; ++j) {
        k_gmres_apply<MANY><<<nb, BS, 0, st>>>(L, j, g);
        for (int pass = 0; pass < 2; ++pass) {
            switch (j) {
                case 0: k_gmres_orth<1, MANY><<<nb, BS, 0, st>>>(N, j, pass, g); break;
                case 1: k_gmres_orth<2, MANY><<<nb, BS, 0, st>>>(N, j, pass, g); break;
                case 2: k_gmres_orth<3, MANY><<<nb, BS, 0, st>>>(N, j, pass, g); break;
                case 3: k_gmres_orth<4, MANY><<<nb, BS, 0, st>>>(N, j, pass, g); break;
                case 4: k_gmres_orth<5, MANY><<<nb, BS, 0, st>>>(N, j, pass, g); break;
                default: k_gmres_orth<0, MANY><<<nb, BS, 0, st>>>(N, j, pass, g);
            }
        }
    }
    k_gmres_finish<MANY><<<nb, BS, 0, st>>>(N, gs, X, g);
}

void gmres_2d(hipStream_t st, const Op2<double>& L, Vec<const cxd> B, Vec<cxd> X, bool guess, const GmresWs& g, int ns) {
    if (g.chunks > 1) gmres_launch<true>(st, L, B, X, guess, g, ns);
    else gmres_launch<false>(st, L, B, X, guess, g, ns);
}

}  // namespace helm
