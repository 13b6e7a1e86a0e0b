// The z-marching passes (march3d.h) of a step on the levels that block passes
// serve while their launches are small (kernels3d_block.hip), for launches of
// many columns, with the block passes' roundings: the terms of a row come from
// weights of the column, not from the weights of the interior plus the
// boundary's terms, so that a column's result does not depend on how many
// columns share the launch.
//
// Regions of 32 x 16 columns, one a thread: the column's weights take the
// registers of a second one, and a mesh of 49 to 96 nodes a side leaves less of
// a 16-row region unused than of a 32-row one.
#pragma clang fp contract(off)
#include "march3d.h"

namespace helm {

template <typename T>
bool columns3d(hipStream_t st, const Op3F<T>& L, int first, int nj, bool pro, int upd, T s, Vec<const cx<T>> X,
               Vec<const cx<T>> Bv, Vec<const cx<T>> Ec, Vec<cx<T>> Rho, Vec<cx<T>> Y, Vec<cx<T>> Bc, int ns) {
    const bool rr = Bc.base != nullptr;
#define HELM_C3(F, NJ_, PRO_, UPD_, RR_)                                                             \
    do {                                                                                             \
        launch_d<T, T, F, NJ_, PRO_, UPD_, RR_, 16, 1, true>(st, L, s, X, Bv, Ec, Rho, Y, Bc, ns);   \
        return true;                                                                                 \
    } while (0)
    if (rr) {
        if (pro || upd != 0) return false;
        if (first == F_JAC && nj == 0) HELM_C3(F_JAC, 0, false, 0, true);
        if (first == F_HSS0 && nj == 1) HELM_C3(F_HSS0, 1, false, 0, true);
        if (first == F_JAC0 && nj == 1) HELM_C3(F_JAC0, 1, false, 0, true);
        return false;
    }
    if (first == F_RESID && !pro && upd == 0) HELM_C3(F_RESID, 0, false, 0, false);
    if (first != F_JAC || nj != 2) return false;
    if (!pro && upd == 0) HELM_C3(F_JAC, 2, false, 0, false);
    if (pro && upd == 0) HELM_C3(F_JAC, 2, true, 0, false);
    if (pro && upd == 1) HELM_C3(F_JAC, 2, true, 1, false);
#undef HELM_C3
    return false;
}

template bool columns3d<double>(hipStream_t, const Op3F<double>&, int, int, bool, int, double, Vec<const cxd>,
                                Vec<const cxd>, Vec<const cxd>, Vec<cxd>, Vec<cxd>, Vec<cxd>, int);
template bool columns3d<float>(hipStream_t, const Op3F<float>&, int, int, bool, int, float, Vec<const cxf>,
                               Vec<const cxf>, Vec<const cxf>, Vec<cxf>, Vec<cxf>, Vec<cxf>, int);

}  // namespace helm
