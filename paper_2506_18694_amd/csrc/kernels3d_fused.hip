// The z-marching passes (march3d.h) on the 3D levels of any size.
#pragma clang fp contract(off)
#include <type_traits>

#include "march3d.h"

namespace helm {

namespace {

// Two columns a thread on 32 x 32 regions, but one for the FP32 residual, whose
// instructions are then fewer than what the barrier per plane costs: on 32 x 16
// regions up to 4M nodes, whose launches are short of workgroups, above that on
// 32 x 32.  Measured (us, two columns / 32 x 16 / 32 x 32): 96^3 9.9 / 9.1 / 9.7,
// 128^3 12.7 / 12.7 / 13.4, 4 x 128^3 42.0 / 47.6 / 40.5, 256^3 99.3 / 103.8 /
// 93.9.  The other one-stage passes gain nothing from one column a thread: an
// application at 256^3 in FP64 113.5 / 142.8 / 115.9, at 128^3 16.3 / 16.5 / 16.5.
constexpr double RESID_TALL = 4e6;
template <typename T, typename TI, int F, int NJ, bool PRO, int UPD, bool RR>
void launch_pass(hipStream_t st, const Op3F<T>& L, T s, Vec<const cx<TI>> X, Vec<const cx<T>> Bv,
                 Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y, Vec<cx<T>> Bc, int nslots) {
    if constexpr (sizeof(T) == 4 && F == F_RESID) {
        const double nodes = (double)(L.n + 1) * (L.n + 1) * (L.n + 1) * nslots;
        if (nodes < RESID_TALL) launch_d<T, TI, F, NJ, PRO, UPD, RR, 16, 1>(st, L, s, X, Bv, Ec, Rho, Y, Bc, nslots);
        else launch_d<T, TI, F, NJ, PRO, UPD, RR, 32, 1>(st, L, s, X, Bv, Ec, Rho, Y, Bc, nslots);
    } else {
        launch_d<T, TI, F, NJ, PRO, UPD, RR, 32, 2>(st, L, s, X, Bv, Ec, Rho, Y, Bc, nslots);
    }
}

// y = w/D b, the sweep from a zero guess: 16 bytes a thread, gx workgroups a
// plane of the mesh.  The factors come from the table of the number of boundary
// coordinates and a node's place from one 32-bit division: with the division of
// the diagonal and 64-bit ones at every node it took 59 us on 256^3 in FP32,
// now 43.  Nodes a thread, 1 / 2 / 4: FP32 53 / 43 / 43 us, two columns 118 / 94
// / 99; FP64 91 / 96 / 101, where the instructions never counted.
constexpr int J0_BS = 256;
template <typename T>
constexpr int J0_NPT = 16 / (int)sizeof(cx<T>);
template <typename T>
__global__ __launch_bounds__(J0_BS) void k3_jacobi0(Op3F<T> L, Vec<const cx<T>> Bv, Vec<cx<T>> Y, unsigned gx) {
    const unsigned n = (unsigned)L.n, sy = n + 1, sz = sy * sy;
    const unsigned lin = xcd_remap(blockIdx.x, gridDim.x), row = lin / gx, blk = lin - row * gx;
    const unsigned slot = row / sy, l = row - slot * sy;
    const long long base = (long long)l * sz;
    const cx<T>* b = Bv.at((int)slot) + base;
    cx<T>* y = Y.at((int)slot) + base;
    constexpr int NPT = J0_NPT<T>;
    cx<T> v[NPT];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        const unsigned t = (blk * NPT + u) * J0_BS + threadIdx.x;
        v[u] = b[t < sz ? t : 0];
    }
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        const unsigned t = (blk * NPT + u) * J0_BS + threadIdx.x;
        if (t >= sz) continue;
        const unsigned j = t / sy, i = t - j * sy;
        const int q = (int)(i == 0 || i == n) + (int)(j == 0 || j == n) + (int)(l == 0 || l == n);
        const cx<T> od = csel(q < 2, csel(q == 0, L.od[0], L.od[1]), csel(q == 2, L.od[2], L.od[3]));
        y[t] = od * v[u];
    }
}

}  // namespace

template <typename T, typename TI>
bool pass3d(hipStream_t st, const Op3F<T>& L, int first, int nj, bool pro, int upd, T s, Vec<const cx<TI>> X,
            Vec<const cx<T>> Bv, Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y, Vec<cx<T>> Bc, int nslots) {
    const bool rr = Bc.base != nullptr;
#define HELM_P3(F, NJ_, PRO_, UPD_, RR_)                                                      \
    do {                                                                                      \
        launch_pass<T, TI, F, NJ_, PRO_, UPD_, RR_>(st, L, s, X, Bv, Ec, Rho, Y, Bc, nslots); \
        return true;                                                                          \
    } while (0)
    if (!pro && upd == 0 && !rr) {
        if (first == F_APPLY) HELM_P3(F_APPLY, 0, false, 0, false);
        if (first == F_RESID) HELM_P3(F_RESID, 0, false, 0, false);
    }
    if constexpr (std::is_same<T, TI>::value) {
        if (first == F_JAC && !rr) {
            if (nj == 1 && !pro && upd == 0) HELM_P3(F_JAC, 1, false, 0, false);
            if (nj == 2 && !pro && upd == 0) HELM_P3(F_JAC, 2, false, 0, false);
            if (nj == 2 && pro && upd == 0) HELM_P3(F_JAC, 2, true, 0, false);
            if (nj == 2 && pro && upd == 1) HELM_P3(F_JAC, 2, true, 1, false);
        }
        if (!pro && upd == 0 && rr) {
            if (first == F_JAC && nj == 0) HELM_P3(F_JAC, 0, false, 0, true);
            if (first == F_HSS0 && nj == 1) HELM_P3(F_HSS0, 1, false, 0, true);
            if (first == F_JAC0 && nj == 1) HELM_P3(F_JAC0, 1, false, 0, true);
        }
    }
#undef HELM_P3
    return false;
}

template <typename T>
void jacobi0_3d(hipStream_t st, const Op3F<T>& L, Vec<const cx<T>> B, Vec<cx<T>> Y, int ns) {
    const unsigned sz = (unsigned)(L.n + 1) * (unsigned)(L.n + 1), per = J0_BS * J0_NPT<T>;
    const unsigned gx = (sz + per - 1) / per;
    k3_jacobi0<T><<<gx * ((unsigned)L.n + 1) * (unsigned)ns, J0_BS, 0, st>>>(L, B, Y, gx);
}
template void jacobi0_3d<double>(hipStream_t, const Op3F<double>&, Vec<const cxd>, Vec<cxd>, int);
template void jacobi0_3d<float>(hipStream_t, const Op3F<float>&, Vec<const cxf>, Vec<cxf>, int);

#define HELM_INST(T, TI)                                                                               \
    template bool pass3d<T, TI>(hipStream_t, const Op3F<T>&, int, int, bool, int, T, Vec<const cx<TI>>, \
                                Vec<const cx<T>>, Vec<const cx<T>>, Vec<cx<T>>, Vec<cx<T>>,           \
                                Vec<cx<T>>, int);
HELM_INST(double, double)
HELM_INST(double, float)
HELM_INST(float, float)
#undef HELM_INST

}  // namespace helm
