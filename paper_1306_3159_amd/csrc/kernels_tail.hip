// The coarse end of the multigrid V-cycle in one work-group: every level from the first
// that fits in LDS down to the coarsest grid, for the periodic operator alpha I - D L and
// for the box with homogeneous faces (arXiv:1306.3159 Sec. III.E, eq. Helmholtz; the box
// of Sec. IV.C). The steps are those of the per-level kernels: zero guess, R B R B
// pre-smoothing, red residual, restriction, the exact coarsest solve, red correction,
// B R B R post-smoothing.
//
// What bounds it is the chain of steps (about ten per level, each a barrier, an LDS round
// trip and a few dependent sums), not bytes, so the work per step is kept short:
//  * Levels are held red/black split (cell (x, y, z) of colour (x+y+z)&1 at index x/2 of
//    row (y, z) of its colour). The two cells of one index are each other's x-neighbour, so
//    a thread that owns an index keeps both values, both right-hand sides and its
//    neighbours' LDS offsets in registers: a half-sweep reads five values and writes one.
//    The first level's indices (up to eight per thread) stay in registers across the whole
//    kernel; the lower levels have at most one index per thread and keep theirs in LDS.
//  * The coarsest (pseudo-)inverse is applied in FP64: up to 64 cells as a dense matrix that
//    is loaded into registers at the start, behind the first level's loads; beyond, in the
//    eigenvector bases of the axes (the operator is a sum of three one-dimensional ones),
//    2 (nx + ny + nz) products per cell from LDS instead of nx ny nz from L2.
//  * Transfers: four threads to a coarse cell of the restriction, a plane each; coordinates
//    by reciprocals and 24-bit products (a 32-bit product takes four issue slots).
//  * The descriptor is copied to LDS at once and planes are padded against bank conflicts.
// Measured, one application (kernel trace): FP64 from 16^3 11.4 us (12.4 with a thread to a
// coarse cell, spectral coarsest solve and the descriptor in kernel arguments), FP32 box from
// 16^3 16.6 us (19.5), FP32 from 18 x 14 x 10 9.4 us (9.3; its 315 coarsest cells stay
// spectral). The first kernel, all arrays in LDS, coordinates divided out at every step and
// the dense inverse read from L2: 28 to 36 us.
#include "launch.hpp"

namespace brd {

namespace {

constexpr int kTailThreads = kFinBlock;

// Quotients by a fixed divisor of whole numbers below 2^13: (i + 1/2) / n is at least
// 1 / (2 n) from every whole number, and the rounding of the product far smaller.
struct Div {
    float r;
    int n;
    __device__ __forceinline__ explicit Div(int d) : r(1.0f / (float)d), n(d) {}
    __device__ __forceinline__ int operator()(int i) const { return (int)(((float)i + 0.5f) * r); }
};
// i -> (a, b, c) of row-major dims (na, nb, *)
struct Dec {
    Div a, b;
    __device__ __forceinline__ Dec(int na, int nb) : a(na), b(nb) {}
    __device__ __forceinline__ void operator()(int i, int& x, int& y, int& z) const {
        const int t = a(i);
        x = i - __mul24(t, a.n);
        z = b(t);
        y = t - __mul24(z, b.n);
    }
};

// The coarsest solve by eigenvectors: in and out are m doubles in LDS (natural order), b another
// m. spec (LDS): row-major eigenvector matrices (row = mode) of the x, y and z axes, then the
// inverse eigenvalue of every mode (natural order; zero for the constant mode when it is
// the null space). The result is left in `a`.
__device__ __forceinline__ double spec_dot(const double* v, int vs, const double* a, int as, int n) {
    double s = 0.0;
    for (int k0 = 0; k0 < n; k0 += 4) {  // four products' operands in flight
        double x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = min(k0 + u, n - 1);
            x[u] = v[__mul24(k, vs)];
            y[u] = k0 + u < n ? a[__mul24(k, as)] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) s += x[u] * y[u];
    }
    return s;
}
__device__ __forceinline__ void spectral_solve(double* a, double* b, const double* spec, int nx, int ny, int nz) {
    const int m = nx * ny * nz, j = threadIdx.x, pl = nx * ny;
    const double* vx = spec;
    const double* vy = vx + nx * nx;
    const double* vz = vy + ny * ny;
    const double* w = vz + nz * nz;
    const bool on = j < m;
    int x = 0, y = 0, z = 0;
    if (on) Dec(nx, ny)(j, x, y, z);
    const int row = j - x, col = j - y * nx, pil = j - z * pl;
    if (on) b[j] = spec_dot(vx + x * nx, 1, a + row, 1, nx);
    lds_barrier();
    if (on) a[j] = spec_dot(vy + y * ny, 1, b + col, nx, ny);
    lds_barrier();
    if (on) b[j] = spec_dot(vz + z * nz, 1, a + pil, pl, nz) * w[j];
    lds_barrier();
    if (on) a[j] = spec_dot(vz + z, nz, b + pil, pl, nz);
    lds_barrier();
    if (on) b[j] = spec_dot(vy + y, ny, a + col, nx, ny);
    lds_barrier();
    if (on) a[j] = spec_dot(vx + x, nx, b + row, 1, nx);
    lds_barrier();
}

// The coarsest solve as a dense matrix (rows and columns padded to kDenseCells): 16 threads to a
// row, four columns each, loaded by dense_load into c; the result is left in a.
constexpr int kDenseCells = 64;
static_assert(kDenseCells * 16 == kTailThreads && kDenseCells == kTailDense, "a row of lanes to a row");
__device__ __forceinline__ void dense_load(double (&c)[4], const double* __restrict__ dense) {
    typedef double D2 __attribute__((ext_vector_type(2)));
    const D2* p = reinterpret_cast<const D2*>(dense + 4 * threadIdx.x);
    const D2 u = p[0], v = p[1];
    c[0] = u[0], c[1] = u[1], c[2] = v[0], c[3] = v[1];
}
__device__ __forceinline__ void dense_solve(double* a, const double (&c)[4]) {
    const double* f = a + 4 * (threadIdx.x & 15);
    double s = (c[0] * f[0] + c[1] * f[1]) + (c[2] * f[2] + c[3] * f[3]);
    s = row_sum(s);
    lds_barrier();  // every thread has read a
    if ((threadIdx.x & 15) == 15) a[threadIdx.x >> 4] = s;
    lds_barrier();
}

// One index of a split level: byte offsets within a colour array of the other colour's values
// that its red (xr) and its black cell (xb) read besides the one at its own index, and of the
// y and z neighbours of both, two to a register (the LDS budget keeps a colour array below
// 64 KiB); beyond a box face the offset is that of a stored zero (`zero`). pos holds the
// index's (i, y, z) and the faces its red and black cells touch in a box.
struct TailCell {
    unsigned x, y, z, pos, own;  // own: the index's offset in elements
    __device__ __forceinline__ unsigned xr() const { return x & 0xffffu; }
    __device__ __forceinline__ unsigned xb() const { return x >> 16; }
    __device__ __forceinline__ int pi() const { return pos & 255; }
    __device__ __forceinline__ int py() const { return (pos >> 8) & 511; }
    __device__ __forceinline__ int pz() const { return (pos >> 17) & 511; }
    __device__ __forceinline__ int fr() const { return (pos >> 26) & 3; }
    __device__ __forceinline__ int fb() const { return (pos >> 28) & 3; }
};

template <typename T, bool BOX>
__device__ __forceinline__ TailCell tail_cell(int i, int y, int z, int hx, int ny, int nz, int plane, int zero) {
    const int row = __mul24(z, plane) + __mul24(y, hx), own = row + i, wrap = __mul24(ny - 1, hx);
    const int up = (y + z) & 1;  // red cell x = 2i + up, black cell x = 2i + (1 - up)
    const int r = i + 1, l = i - 1;
    int right, left, ym, yp, zm, zp, fr = 0, fb = 0;
    if (BOX) {
        right = r < hx ? row + r : zero;
        left = l >= 0 ? row + l : zero;
        ym = y > 0 ? own - hx : zero;
        yp = y + 1 < ny ? own + hx : zero;
        zm = z > 0 ? own - plane : zero;
        zp = z + 1 < nz ? own + plane : zero;
        const int fyz = (y == 0) + (y + 1 == ny) + (z == 0) + (z + 1 == nz);
        fr = fyz + (up ? r == hx : i == 0);
        fb = fyz + (up ? i == 0 : r == hx);
    } else {
        right = row + (r < hx ? r : 0);
        left = row + (l >= 0 ? l : hx - 1);
        ym = y > 0 ? own - hx : own + wrap;
        yp = y + 1 < ny ? own + hx : own - wrap;
        zm = z > 0 ? own - plane : own + __mul24(nz - 1, plane);
        zp = z + 1 < nz ? own + plane : own - __mul24(nz - 1, plane);
    }
    constexpr unsigned S = sizeof(T);
    TailCell c;
    c.x = (unsigned)(up ? right : left) * S | ((unsigned)(up ? left : right) * S << 16);
    c.y = (unsigned)ym * S | ((unsigned)yp * S << 16);
    c.z = (unsigned)zm * S | ((unsigned)zp * S << 16);
    c.own = (unsigned)own;
    c.pos = (unsigned)i | ((unsigned)y << 8) | ((unsigned)z << 17) | ((unsigned)fr << 26) | ((unsigned)fb << 28);
    return c;
}

// Coefficients of one level; box: diagonal diag + f s of a cell touching f faces and its
// inverse, selected without a runtime-indexed array.
template <typename T, bool BOX>
struct TailCoef {
    T s, diag, i0, i1, i2, i3;
    __device__ __forceinline__ TailCoef(const TailDesc& d, int l)
        : s((T)d.s[l]), diag((T)d.diag[l]), i0((T)d.inv_diag[l][0]), i1(BOX ? (T)d.inv_diag[l][1] : (T)0),
          i2(BOX ? (T)d.inv_diag[l][2] : (T)0), i3(BOX ? (T)d.inv_diag[l][3] : (T)0) {}
    __device__ __forceinline__ T inv(int f) const {
        if (!BOX) return i0;
        return f == 0 ? i0 : (f == 1 ? i1 : (f == 2 ? i2 : i3));
    }
    __device__ __forceinline__ T dg(int f) const { return BOX ? diag + (T)f * s : diag; }
};

// Neighbour sum of a cell: its x-neighbour at the same index (own), the other x-neighbour,
// then the y and z pairs, in the order of the per-level kernels.
template <typename T>
__device__ __forceinline__ T tail_sum(const T* o, T own, unsigned xo, const TailCell& c) {
    const char* b = reinterpret_cast<const char*>(o);
    auto at = [&](unsigned off) { return *reinterpret_cast<const T*>(b + off); };
    return ((own + at(xo)) + (at(c.y & 0xffffu) + at(c.y >> 16))) + (at(c.z & 0xffffu) + at(c.z >> 16));
}

// Plane c (fine z = 2Z - 1 + c) of the restriction of the split red residual R (black zero) to
// coarse cell (X, Y, Z): the red cells of a fine row of parity p among 2X-1 .. 2X+2 are those at
// index X-1 and X (p = 1) or X and X+1 (p = 0).
template <typename T, bool BOX>
__device__ __forceinline__ T tail_restrict_plane(const T* R, int X, int Y, int Z, int c, int hx, int ny, int nz,
                                                 int pstr) {
    const T w0 = (T)0.125, w1 = (T)0.375;
    const int xl = X == 0 ? hx - 1 : X - 1, xr = X + 1 == hx ? 0 : X + 1;
    const T* plane = R + __mul24(wrapi(2 * Z - 1 + c, nz), pstr);
    T accb = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        int y = 2 * Y - 1 + b;
        T wy = (b == 0 || b == 3) ? w0 : w1;
        if (BOX) {
            if (y < 0 || y >= ny) wy = (T)0;
            else if ((b == 1 && y == 0) || (b == 2 && y == ny - 1)) wy = (T)0.25;
        }
        const T* row = plane + __mul24(wrapi(y, ny), hx);
        const int p = (b + c) & 1;  // parity of the row (dims are even)
        const T m = row[X];
        T e = row[p ? xl : xr];
        T wm = w1;
        if (BOX) {
            if (p ? X == 0 : X + 1 == hx) e = (T)0;
            if (p ? X + 1 == hx : X == 0) wm = (T)0.25;  // the boundary fine cell of a boundary coarse cell
        }
        accb = fma(wy, restrict_row(w0, wm, p, e, m, e), accb);
    }
    return accb;
}

// The weighted sum of the four planes' values held by the lanes of a quad, in every lane of it.
template <typename T, bool BOX>
__device__ __forceinline__ T tail_restrict_sum(T v, int Z, int nz) {
    const T p[4] = {quad_value<0>(v), quad_value<1>(v), quad_value<2>(v), quad_value<3>(v)};
    T acc = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        T w = (c == 0 || c == 3) ? (T)0.125 : (T)0.375;
        if (BOX) {
            const int z = 2 * Z - 1 + c;
            if (z < 0 || z >= nz) w = (T)0;
            else if ((c == 1 && z == 0) || (c == 2 && z == nz - 1)) w = (T)0.25;
        }
        acc = fma(w, p[c], acc);
    }
    return acc;
}

// u plus the trilinear correction of the red fine cell (2i + up, y, z) from the coarse
// values C in natural order.
template <typename T, bool BOX>
__device__ __forceinline__ T tail_correct(T u, const T* C, int i, int y, int z, int cx, int cy, int cz) {
    const int up = (y + z) & 1;
    const int I0 = i, J0 = y >> 1, K0 = z >> 1;
    int I1 = up ? I0 + 1 : I0 - 1, J1 = (y & 1) ? J0 + 1 : J0 - 1, K1 = (z & 1) ? K0 + 1 : K0 - 1;
    if (BOX) {
        // beyond a face the coarse ghost is -u of the parent, which then takes 1/2
        T a0 = (T)0.75, a1 = (T)0.25, b0 = a0, b1 = a1, c0 = a0, c1 = a1;
        if (I1 < 0 || I1 >= cx) I1 = I0, a0 = (T)0.5, a1 = (T)0;
        if (J1 < 0 || J1 >= cy) J1 = J0, b0 = (T)0.5, b1 = (T)0;
        if (K1 < 0 || K1 >= cz) K1 = K0, c0 = (T)0.5, c1 = (T)0;
        const int pl = __mul24(cx, cy), j0 = __mul24(J0, cx), j1 = __mul24(J1, cx);
        const T *p0 = C + __mul24(K0, pl), *p1 = C + __mul24(K1, pl);
        const T *r00 = p0 + j0, *r10 = p0 + j1, *r01 = p1 + j0, *r11 = p1 + j1;
        const T v00 = a0 * r00[I0] + a1 * r00[I1], v10 = a0 * r10[I0] + a1 * r10[I1];
        const T v01 = a0 * r01[I0] + a1 * r01[I1], v11 = a0 * r11[I0] + a1 * r11[I1];
        return u + (c0 * (b0 * v00 + b1 * v10) + c1 * (b0 * v01 + b1 * v11));
    }
    I1 = wrapi(I1, cx);
    J1 = wrapi(J1, cy);
    K1 = wrapi(K1, cz);
    const int pl = __mul24(cx, cy), j0 = __mul24(J0, cx), j1 = __mul24(J1, cx);
    const T *p0 = C + __mul24(K0, pl), *p1 = C + __mul24(K1, pl);
    const T *r00 = p0 + j0, *r10 = p0 + j1, *r01 = p1 + j0, *r11 = p1 + j1;
    return tri_add(u, r00[I0], r00[I1], r10[I0], r10[I1], r01[I0], r01[I1], r11[I0], r11[I1]);
}

// K indices of the first level per thread (index j = threadIdx.x + k * kTailThreads). dg: the
// descriptor where the caller has it (kernel arguments or device memory); its words go to LDS
// first, all at once: read where they are used, each of its cache lines would stall a step.
template <typename T, int K, bool BOX>
__device__ __forceinline__ void tail_run(const T* __restrict__ f0g, const T* __restrict__ f1g, T* __restrict__ u0g,
                                         T* __restrict__ u1g, const TailDesc& dg, const double* __restrict__ specg,
                                         unsigned char* smem) {
    TailDesc& d = *reinterpret_cast<TailDesc*>(smem);
    const int tid = threadIdx.x;
    static_assert(sizeof(TailDesc) % 4 == 0 && sizeof(TailDesc) / 4 <= kTailThreads, "a word a thread");
    if (tid < (int)(sizeof(TailDesc) / 4)) reinterpret_cast<int*>(&d)[tid] = reinterpret_cast<const int*>(&dg)[tid];
    const int nx0 = dg.nx[0], ny0 = dg.ny[0], nz0 = dg.nz[0], hx0 = nx0 >> 1, nh0 = hx0 * ny0 * nz0;
    T f0[K], f1[K], u0[K], u1[K];
    TailCell cell[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = tid + k * kTailThreads;
        f0[k] = f1[k] = u0[k] = u1[k] = (T)0;
        cell[k] = TailCell{};
        if (j < nh0) {
            f0[k] = f0g[j];
            f1[k] = f1g[j];
        }
    }
    const int L = dg.nlev - 1, nspec = dg.nspec;
    const int mc = dg.nx[L] * dg.ny[L] * dg.nz[L];
    const bool dense = mc <= kDenseCells;
    double dc[4];
    if (dense) dense_load(dc, specg + nspec);
    // planes are padded by 8 values: rows of neighbouring planes fall into different banks
    const int ps0 = __mul24(hx0, ny0) + kTailPad, zero0 = __mul24(nz0, ps0);
    {
        const Dec dec(hx0, ny0);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = tid + k * kTailThreads;
            if (j < nh0) {
                int i, y, z;
                dec(j, i, y, z);
                cell[k] = tail_cell<T, BOX>(i, y, z, hx0, ny0, nz0, ps0, zero0);
            }
        }
    }
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    auto at = [&](int off) { return smem + uni(off); };
    lds_barrier();
    T* const A0 = reinterpret_cast<T*>(at(d.off_u[0]));  // red values, then a zero
    T* const A1 = A0 + zero0 + 1;                        // black values, then a zero
    double* const spec = reinterpret_cast<double*>(at(d.off_spec));
    double* const ab = reinterpret_cast<double*>(at(d.off_ab));
    const TailCoef<T, BOX> c0(d, 0);
    if (dense) {
        if (tid < kDenseCells) ab[tid] = 0.0;  // padding of the solve
    } else {
        for (int j = tid; j < nspec; j += kTailThreads) spec[j] = specg[j];
    }
    if (BOX && tid == 0) A0[zero0] = A1[zero0] = (T)0;
    // half-sweeps of the first level; the barrier orders the written colour before its readers
    auto red = [&]() {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (tid + k * kTailThreads < nh0) {
                u0[k] = relax(f0[k], c0.s, tail_sum(A1, u1[k], cell[k].xr(), cell[k]), c0.inv(cell[k].fr()));
                A0[cell[k].own] = u0[k];
            }
        lds_barrier();
    };
    auto black = [&]() {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (tid + k * kTailThreads < nh0) {
                u1[k] = relax(f1[k], c0.s, tail_sum(A0, u0[k], cell[k].xb(), cell[k]), c0.inv(cell[k].fb()));
                A1[cell[k].own] = u1[k];
            }
        lds_barrier();
    };
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tid + k * kTailThreads < nh0) {
            u0[k] = relax_zero(f0[k], c0.inv(cell[k].fr()));  // red sweep from zero
            A0[cell[k].own] = u0[k];
        }
    lds_barrier();
    black();
    red();
    black();
    // red residual, over the red values (every owner keeps its own)
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tid + k * kTailThreads < nh0)
            A0[cell[k].own] =
                red_resid(f0[k], c0.dg(cell[k].fr()), u0[k], c0.s, tail_sum(A1, u1[k], cell[k].xr(), cell[k]));
    lds_barrier();
    // lower levels, down: u0 | 0 | u1 | 0 | r (padded planes) | f0 | f1 of the level, then its
    // values in natural order
    const T* R = A0;
    int fhx = hx0, fny = ny0, fnz = nz0, fps = ps0;
    for (int l = 1; l <= L; ++l) {
        const int nx = uni(d.nx[l]), ny = uni(d.ny[l]), nz = uni(d.nz[l]), n = nx * ny * nz;
        const int hx = nx >> 1, nh = hx * ny * nz, ps = hx * ny + kTailPad, zero = nz * ps;
        const bool last = l == L;
        T* B0 = reinterpret_cast<T*>(at(d.off_u[last ? 0 : l]));
        T* B1 = B0 + zero + 1;
        T* RR = B1 + zero + 1;
        T* F0 = RR + zero;
        T* F1 = F0 + nh;
        {
            const Dec dec(nx, ny);
            for (int q = tid; q < 4 * n; q += kTailThreads) {  // whole quads: 4 n and the stride are multiples of 4
                int X, Y, Z;
                dec(q >> 2, X, Y, Z);
                T v = tail_restrict_plane<T, BOX>(R, X, Y, Z, q & 3, fhx, fny, fnz, fps);
                v = tail_restrict_sum<T, BOX>(v, Z, fnz);
                if ((q & 3) == 0) {
                    // rounded to T on the coarsest grid too, as a stored level would be
                    if (last) ab[q >> 2] = (double)v;
                    else (((X + Y + Z) & 1) ? F1 : F0)[__mul24(__mul24(Z, ny) + Y, hx) + (X >> 1)] = v;
                }
            }
        }
        if (last) {
            lds_barrier();
            break;
        }
        if (BOX && tid == 0) B0[zero] = B1[zero] = (T)0;
        const TailCoef<T, BOX> c(d, l);
        const bool on = tid < nh;
        T a = 0, b = 0, fa = 0, fb = 0;
        TailCell ce{};
        if (on) {
            int i, y, z;
            Dec(hx, ny)(tid, i, y, z);
            ce = tail_cell<T, BOX>(i, y, z, hx, ny, nz, ps, zero);
        }
        lds_barrier();
        if (on) {
            fa = F0[tid];
            fb = F1[tid];
            a = relax_zero(fa, c.inv(ce.fr()));
            B0[ce.own] = a;
        }
        lds_barrier();
        if (on) B1[ce.own] = b = relax(fb, c.s, tail_sum(B0, a, ce.xb(), ce), c.inv(ce.fb()));
        lds_barrier();
        if (on) B0[ce.own] = a = relax(fa, c.s, tail_sum(B1, b, ce.xr(), ce), c.inv(ce.fr()));
        lds_barrier();
        if (on) B1[ce.own] = b = relax(fb, c.s, tail_sum(B0, a, ce.xb(), ce), c.inv(ce.fb()));
        lds_barrier();
        if (on) RR[ce.own] = red_resid(fa, c.dg(ce.fr()), a, c.s, tail_sum(B1, b, ce.xr(), ce));
        lds_barrier();
        R = RR;
        fhx = hx;
        fny = ny;
        fnz = nz;
        fps = ps;
    }
    // coarsest grid
    {
        const int nx = uni(d.nx[L]), ny = uni(d.ny[L]), nz = uni(d.nz[L]), m = nx * ny * nz;
        if (dense) dense_solve(ab, dc);
        else spectral_solve(ab, ab + m, spec, nx, ny, nz);
        T* C = reinterpret_cast<T*>(at(d.off_nat[L]));
        for (int j = tid; j < m; j += kTailThreads) C[j] = (T)ab[j];
        lds_barrier();
    }
    // lower levels, up
    for (int l = L - 1; l >= 1; --l) {
        const int nx = uni(d.nx[l]), ny = uni(d.ny[l]), nz = uni(d.nz[l]);
        const int hx = nx >> 1, nh = hx * ny * nz, ps = hx * ny + kTailPad, zero = nz * ps;
        T* B0 = reinterpret_cast<T*>(at(d.off_u[l]));
        T* B1 = B0 + zero + 1;
        const T* F0 = B1 + zero + 1 + zero;
        const T* F1 = F0 + nh;
        T* N = reinterpret_cast<T*>(at(d.off_nat[l]));
        const T* C = reinterpret_cast<const T*>(at(d.off_nat[l + 1]));
        const TailCoef<T, BOX> c(d, l);
        const bool on = tid < nh;
        T a = 0, b = 0, fa = 0, fb = 0;
        TailCell ce{};
        int i = 0, y = 0, z = 0;
        if (on) {
            Dec(hx, ny)(tid, i, y, z);
            ce = tail_cell<T, BOX>(i, y, z, hx, ny, nz, ps, zero);
            fa = F0[tid];
            fb = F1[tid];
            a = tail_correct<T, BOX>(B0[ce.own], C, i, y, z, hx, ny >> 1, nz >> 1);
            B0[ce.own] = a;
        }
        lds_barrier();
        if (on) B1[ce.own] = b = relax(fb, c.s, tail_sum(B0, a, ce.xb(), ce), c.inv(ce.fb()));
        lds_barrier();
        if (on) B0[ce.own] = a = relax(fa, c.s, tail_sum(B1, b, ce.xr(), ce), c.inv(ce.fr()));
        lds_barrier();
        if (on) B1[ce.own] = b = relax(fb, c.s, tail_sum(B0, a, ce.xb(), ce), c.inv(ce.fb()));
        lds_barrier();
        if (on) {
            a = relax(fa, c.s, tail_sum(B1, b, ce.xr(), ce), c.inv(ce.fr()));
            const int row = __mul24(__mul24(z, ny) + y, nx), up = (y + z) & 1;
            N[row + 2 * i + up] = a;
            N[row + 2 * i + (up ^ 1)] = b;
        }
        lds_barrier();
    }
    // first level, up
    const T* C = reinterpret_cast<const T*>(at(d.off_nat[1]));
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tid + k * kTailThreads < nh0) {
            u0[k] = tail_correct<T, BOX>(u0[k], C, cell[k].pi(), cell[k].py(), cell[k].pz(), hx0, ny0 >> 1, nz0 >> 1);
            A0[cell[k].own] = u0[k];
        }
    lds_barrier();
    black();
    red();
    black();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = tid + k * kTailThreads;
        if (j < nh0) {
            u0g[j] = relax(f0[k], c0.s, tail_sum(A1, u1[k], cell[k].xr(), cell[k]), c0.inv(cell[k].fr()));
            u1g[j] = u1[k];
        }
    }
}

}  // namespace

template <typename T, int K, bool BOX>
__global__ void __launch_bounds__(kTailThreads) k_tail(const T* __restrict__ f0g, const T* __restrict__ f1g,
                                                       T* __restrict__ u0g, T* __restrict__ u1g, TailDesc d,
                                                       const double* __restrict__ spec, const Scalars* sc) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (sc && sc->done) return;
    tail_run<T, K, BOX>(f0g, f1g, u0g, u1g, d, spec, smem);
}

// Indices of the first level per thread, rounded up to an instantiated count: the LDS budget
// that the levels were chosen for keeps FP32 ones within 8 and FP64 ones within 4.
static int tail_k(const TailDesc& d) {
    const int nh = (d.nx[0] >> 1) * d.ny[0] * d.nz[0];
    return nh <= kTailThreads ? 1 : (nh <= 2 * kTailThreads ? 2 : (nh <= 4 * kTailThreads ? 4 : 8));
}

template <typename T, int K>
static void tail_go(hipStream_t st, const T* f0, const T* f1, T* u0, T* u1, const TailDesc& d, const double* spec,
                    bool box, const Scalars* sc) {
    if (box)
        hipLaunchKernelGGL((k_tail<T, K, true>), dim3(1), dim3(kTailThreads), d.lds_bytes, st, f0, f1, u0, u1, d,
                           spec, sc);
    else
        hipLaunchKernelGGL((k_tail<T, K, false>), dim3(1), dim3(kTailThreads), d.lds_bytes, st, f0, f1, u0, u1, d,
                           spec, sc);
}

template <typename T>
void launch_tail(hipStream_t st, const T* f0, const T* f1, T* u0, T* u1, const TailDesc& d, const double* spec,
                 bool box, const Scalars* sc) {
    switch (tail_k(d)) {
        case 1: tail_go<T, 1>(st, f0, f1, u0, u1, d, spec, box, sc); break;
        case 2: tail_go<T, 2>(st, f0, f1, u0, u1, d, spec, box, sc); break;
        case 4: tail_go<T, 4>(st, f0, f1, u0, u1, d, spec, box, sc); break;
        default: tail_go<T, 32 / (int)sizeof(T)>(st, f0, f1, u0, u1, d, spec, box, sc); break;
    }
}

// One work-group per instance of a batch (periodic): the tail from the instance's level t.
template <typename T>
__global__ void __launch_bounds__(kTailThreads) kb_tail(const InstDev* inst, const int* gate, int ninst) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int i = blockIdx.x;
    if (i >= ninst || !gate[i]) return;
    const InstDev* I = inst + i;
    if (I->sc->done) return;
    T* const* a = reinterpret_cast<T* const*>(I->lv[I->t]);
    const TailDesc& d = I->tail;
    const int nh = (d.nx[0] >> 1) * d.ny[0] * d.nz[0];
    if (nh <= kTailThreads) tail_run<T, 1, false>(a[2], a[3], a[0], a[1], d, I->spec, smem);
    else if (nh <= 2 * kTailThreads) tail_run<T, 2, false>(a[2], a[3], a[0], a[1], d, I->spec, smem);
    else if (nh <= 4 * kTailThreads) tail_run<T, 4, false>(a[2], a[3], a[0], a[1], d, I->spec, smem);
    else tail_run<T, 32 / (int)sizeof(T), false>(a[2], a[3], a[0], a[1], d, I->spec, smem);
}

template <typename T>
void launchb_tail(hipStream_t st, const InstDev* inst, const int* gate, int ninst, unsigned lds) {
    hipLaunchKernelGGL(kb_tail<T>, dim3(ninst), dim3(kTailThreads), lds, st, inst, gate, ninst);
}

// LDS limit of the tail kernels, raised once to the budget the levels were chosen for.
template <typename T>
hipError_t tail_set_lds(size_t bytes) {
    constexpr int KM = 32 / (int)sizeof(T);
    const void* fn[] = {(const void*)k_tail<T, 1, false>, (const void*)k_tail<T, 1, true>,
                        (const void*)k_tail<T, 2, false>, (const void*)k_tail<T, 2, true>,
                        (const void*)k_tail<T, 4, false>, (const void*)k_tail<T, 4, true>,
                        (const void*)k_tail<T, KM, false>, (const void*)k_tail<T, KM, true>,
                        (const void*)kb_tail<T>};
    for (const void* f : fn) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

#define BRD_TAIL_INST(T)                                                                                            \
    template void launch_tail<T>(hipStream_t, const T*, const T*, T*, T*, const TailDesc&, const double*, bool,     \
                                 const Scalars*);                                                                   \
    template void launchb_tail<T>(hipStream_t, const InstDev*, const int*, int, unsigned);                          \
    template hipError_t tail_set_lds<T>(size_t);
BRD_TAIL_INST(float)
BRD_TAIL_INST(double)
#undef BRD_TAIL_INST

}  // namespace brd
