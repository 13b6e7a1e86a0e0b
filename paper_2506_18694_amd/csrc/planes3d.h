// Device helpers of the two kinds of fused 3D pass (kernels3d_fused.hip,
// kernels3d_block.hip): planes read and written through buffer resources, and
// the terms of a node's row, by the weights of the interior and the boundary's
// terms (the marching passes) or by weights of the column (the block passes, and
// the marching passes that take their place for many columns,
// kernels3d_columns.hip).  Passes of one kind use the same formulas term by term,
// and nothing lets the compiler fuse a product into a sum (the files that
// include this switch contraction off before any include), so that a node's
// value does not depend on the form of the pass that computes it: the kind
// follows from the mesh, the form from the size of the launch, and a column's
// result does not depend on how many columns share it.
#pragma once

#include <type_traits>

#include "launch.h"

namespace helm {

namespace {

template <int U>
using IC = std::integral_constant<int, U>;

// Selection between two complex values, one component at a time (a select
// of whole values can be turned into a load through a select of addresses
// of stack copies).
template <typename T>
__device__ __forceinline__ cx<T> csel(bool c, cx<T> a, cx<T> b) {
    return mk(c ? a.x : b.x, c ? a.y : b.y);
}

// Planes are read and written through buffer resources: one per plane, made
// from scalar registers, with the plane's size as its range (0 for a plane
// outside the mesh), and a lane's column as a 32-bit byte offset (OUTSIDE for
// a column outside the mesh, or one that a store leaves to another tile).
// What lies out of range reads as zero and is not written, so no pass tests a
// value or a store, and a step stays one block of straight code.
constexpr unsigned OUTSIDE = 0xFFFFFF00u;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const char* p, unsigned bytes, bool in) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), 0, in ? (int)bytes : 0, 0x00027000);
}
template <typename V>
__device__ __forceinline__ cx<V> bload(__amdgpu_buffer_rsrc_t r, unsigned off) {
    if constexpr (sizeof(V) == 8) {
        return __builtin_bit_cast(cx<V>, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
    } else {
        return __builtin_bit_cast(cx<V>, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
    }
}
template <typename V>
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, unsigned off, cx<V> v) {
    if constexpr (sizeof(V) == 8) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)off, 0, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)off, 0, 0);
    }
}

// a + s t for a real s
template <typename T>
__device__ __forceinline__ cx<T> axpy_real(T s, cx<T> t, cx<T> a) {
    return mk(fmat(s, t.x, a.x), fmat(s, t.y, a.y));
}

// A uniform value as a value of its own in scalar registers (a field of an
// operator record could otherwise be read through an address in a stack copy
// of the record).
__device__ __forceinline__ float scalar(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double scalar(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// The weights of a plane's terms, the same on every lane.
template <typename T>
struct Weights {
    T r1[3], k1, r0[3], k0;
    __device__ __forceinline__ explicit Weights(const Op3F<T>& op) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            r1[q] = scalar(op.r1[q]);
            r0[q] = scalar(op.r0[q]);
        }
        k1 = scalar(op.k1);
        k0 = scalar(op.k0);
    }
};

// T1, T0 of one plane on an interior column (see kernels3d_fused.hip): real
// weights on (a0, s1 = H + V, a2) plus i k times the mass pattern
// m = 16 a0 + 4 s1 + a2 (the imaginary part of every weight is that of its
// mass term).
template <typename T>
__device__ __forceinline__ void plane_terms(const Weights<T>& w, cx<T> a0, cx<T> s1, cx<T> a2, cx<T>& T1,
                                            cx<T>& T0, cx<T>& m) {
    m = mk(fmat((T)4, fmat((T)4, a0.x, s1.x), a2.x), fmat((T)4, fmat((T)4, a0.y, s1.y), a2.y));
    T1 = mk(fmat(w.r1[0], a0.x, fmat(w.r1[1], s1.x, fmat(w.r1[2], a2.x, -w.k1 * m.y))),
            fmat(w.r1[0], a0.y, fmat(w.r1[1], s1.y, fmat(w.r1[2], a2.y, w.k1 * m.x))));
    T0 = mk(fmat(w.r0[0], a0.x, fmat(w.r0[1], s1.x, fmat(w.r0[2], a2.x, -w.k0 * m.y))),
            fmat(w.r0[0], a0.y, fmat(w.r0[1], s1.y, fmat(w.r0[2], a2.y, w.k0 * m.x))));
}

// The same by weights of the column: T = a a0 + h H + v V + d a2, d the same
// on every column, so that boundary columns run the interior ones' code.
template <typename T>
struct ColW {
    cx<T> a, h, v, d;
};
template <typename T>
__device__ __forceinline__ ColW<T> col_weights(const T (&r)[3], T k, const cx<T> (&e)[3], bool bx, bool by) {
    const T fx = bx ? (T)1 : (T)0, fy = by ? (T)1 : (T)0;
    ColW<T> w;
    w.a = axpy_real(fx * fy, e[2], axpy_real(fx + fy, e[0], mk(r[0], (T)16 * k)));
    w.h = axpy_real(fy, e[1], mk(r[1], (T)4 * k));
    w.v = axpy_real(fx, e[1], mk(r[1], (T)4 * k));
    w.d = mk(r[2], k);
    return w;
}
template <typename T>
__device__ __forceinline__ cx<T> col_sum(const ColW<T>& w, cx<T> a0, cx<T> H, cx<T> V, cx<T> a2) {
    return cfma(w.a, a0, cfma(w.h, H, cfma(w.v, V, w.d * a2)));
}
// T0 of an end plane: T0 / 2 + cz times the column's mass pattern
template <typename T>
__device__ __forceinline__ cx<T> end_term(cx<T> cz, bool bx, bool by, cx<T> a0, cx<T> H, cx<T> V, cx<T> a2,
                                          cx<T> t0) {
    const T fx = bx ? (T)1 : (T)0, fy = by ? (T)1 : (T)0;
    const T ma = (T)16 - (T)8 * (fx + fy) + (T)4 * fx * fy, mh = (T)4 - (T)2 * fy, mv = (T)4 - (T)2 * fx;
    const cx<T> m = mk(fmat(ma, a0.x, fmat(mh, H.x, fmat(mv, V.x, a2.x))),
                       fmat(ma, a0.y, fmat(mh, H.y, fmat(mv, V.y, a2.y))));
    return cfma(cz, m, (T)0.5 * t0);
}

// In-plane restriction at the fine centre c of a coarse column, LW values a
// row: weights 1, 1/2, 1/4.
template <typename T, int LW>
__device__ __forceinline__ cx<T> restrict_plane(const cx<T>* c) {
    const cx<T> h = c[-1] + c[1], v = c[-LW] + c[LW];
    const cx<T> d = (c[-LW - 1] + c[-LW + 1]) + (c[LW - 1] + c[LW + 1]);
    return axpy_real((T)0.25, d, axpy_real((T)0.5, h + v, c[0]));
}

}  // namespace

}  // namespace helm
