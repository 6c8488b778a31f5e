// Pieces shared by the kernels that take several steps of a multigrid level in one launch.
#pragma once
#include "launch.hpp"

namespace brd {

namespace {

template <typename T, int VW>
struct RowVec {
    typedef T type __attribute__((ext_vector_type(VW)));
};

// i mod n for any i
__device__ __forceinline__ int modi(int i, int n) {
    i %= n;
    return i < 0 ? i + n : i;
}

// Weight of fine cell 2X - 1 + b for coarse cell X on an axis of n fine cells of a box.
template <typename T>
__device__ __forceinline__ T level_rweight(int b, int X, int n) {
    const int f = 2 * X - 1 + b;
    if (f < 0 || f >= n) return (T)0;
    if (b == 0 || b == 3) return (T)0.125;
    if ((b == 1 && f == 0) || (b == 2 && f == n - 1)) return (T)0.25;
    return (T)0.375;
}

// A fine row's red cells, weighted in x and by wgt, added to coarse cells i0 .. i0 + VW - 1:
// m the row's vector, x its neighbour value (left of it for parity 1, right of it for 0).
template <typename T, int VW, bool BOX>
__device__ __forceinline__ void level_restrict_row(T (&acc)[VW], typename RowVec<T, VW>::type m, T x, int pr, T wgt,
                                                   bool first, bool last) {
    const T w0 = (T)0.125, w1 = (T)0.375;
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        const T l = k ? m[k - 1] : x, n = k + 1 < VW ? m[k + 1] : x;
        T wm = w1;
        if (BOX && (pr ? last && k == VW - 1 : first && k == 0)) wm = (T)0.25;
        acc[k] = fma(wgt, restrict_row(w0, wm, pr, l, m[k], n), acc[k]);
    }
}

// Coarse cells X0 .. X0 + VW - 1 of row Y, plane Z: the values a to the split arrays, with
// the next level's zero-guess red sweep where u0 is set.
template <typename T, int VW, bool BOX>
__device__ __forceinline__ void level_coarse_store(const T (&a)[VW], int X0, int Y, int Z, int cx, int cy, int cz,
                                                   const LevelCoef<T>& c, T* __restrict__ f0, T* __restrict__ f1,
                                                   T* __restrict__ u0) {
    const size_t row = ((size_t)Z * cy + Y) * (cx >> 1);
    const int pc = (Y + Z) & 1;
    auto inv = [&](int X) {
        if (!BOX) return c.invc[0];
        const int f = (X == 0) + (X == cx - 1) + (Y == 0) + (Y == cy - 1) + (Z == 0) + (Z == cz - 1);
        return f == 0 ? c.invc[0] : (f == 1 ? c.invc[1] : (f == 2 ? c.invc[2] : c.invc[3]));
    };
    typedef T H __attribute__((ext_vector_type(VW / 2)));
    const size_t j = row + (X0 >> 1);
    H red, blk, u;
#pragma unroll
    for (int k = 0; k < VW / 2; ++k) {
        red[k] = pc ? a[2 * k + 1] : a[2 * k];
        blk[k] = pc ? a[2 * k] : a[2 * k + 1];
        u[k] = red[k] * inv(X0 + 2 * k + pc);
    }
    *reinterpret_cast<H*>(f0 + j) = red;
    *reinterpret_cast<H*>(f1 + j) = blk;
    if (u0) *reinterpret_cast<H*>(u0 + j) = u;
}

}  // namespace

}  // namespace brd
