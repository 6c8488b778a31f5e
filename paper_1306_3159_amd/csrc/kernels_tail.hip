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
//  * The coarsest operator is a sum of three one-dimensional ones, so its (pseudo-)inverse
//    is applied in their eigenvector bases: 2 (nx + ny + nz) products per cell in FP64 from
//    LDS instead of the dense inverse's nx ny nz from L2.
// Measured, one application (kernel trace): 16^3 -> 8^3 -> 4^3 in FP32 29.9 -> 12.8 us, in
// FP64 31.8 -> 14.1 us, in a box (FP32) 35.6 -> 19.5 us; 18 x 14 x 10 -> 9 x 7 x 5 36.4 -> 9.3
// us. Before: all arrays in LDS, cell coordinates divided out at every step, dense inverse.
#include "launch.hpp"

namespace brd {

namespace {

constexpr int kTailThreads = kFinBlock;

// The coarsest solve: in and out are m doubles in LDS (natural order), tmp another m.
// spec (LDS): row-major eigenvector matrices (row = mode) of the x, y and z axes, then the
// inverse eigenvalue of every mode (natural order; zero for the constant mode when it is
// the null space). The result is left in `a`.
__device__ __forceinline__ void spectral_solve(double* a, double* b, const double* spec, int nx, int ny, int nz) {
    const int m = nx * ny * nz, j = threadIdx.x;
    const double* vx = spec;
    const double* vy = vx + nx * nx;
    const double* vz = vy + ny * ny;
    const double* w = vz + nz * nz;
    const bool on = j < m;
    const int x = on ? j % nx : 0, t = on ? j / nx : 0, y = t % ny, z = t / ny;
    const int row = j - x, col = j - y * nx, pil = j - z * nx * ny;
    if (on) {
        double s = 0.0;
        for (int k = 0; k < nx; ++k) s += vx[x * nx + k] * a[row + k];
        b[j] = s;
    }
    __syncthreads();
    if (on) {
        double s = 0.0;
        for (int k = 0; k < ny; ++k) s += vy[y * ny + k] * b[col + k * nx];
        a[j] = s;
    }
    __syncthreads();
    if (on) {
        double s = 0.0;
        for (int k = 0; k < nz; ++k) s += vz[z * nz + k] * a[pil + k * nx * ny];
        b[j] = s * w[j];
    }
    __syncthreads();
    if (on) {
        double s = 0.0;
        for (int k = 0; k < nz; ++k) s += vz[k * nz + z] * b[pil + k * nx * ny];
        a[j] = s;
    }
    __syncthreads();
    if (on) {
        double s = 0.0;
        for (int k = 0; k < ny; ++k) s += vy[k * ny + y] * a[col + k * nx];
        b[j] = s;
    }
    __syncthreads();
    if (on) {
        double s = 0.0;
        for (int k = 0; k < nx; ++k) s += vx[k * nx + x] * b[row + k];
        a[j] = s;
    }
    __syncthreads();
}

// One index of a split level: byte offsets within a colour array of the other colour's values
// that its red (xr) and its black cell (xb) read besides the one at its own index, and of the
// y and z neighbours of both, two to a register (the LDS budget keeps a colour array below
// 64 KiB); beyond a box face the offset is that of a stored zero (`zero`). pos holds the
// index's (i, y, z) and the faces its red and black cells touch in a box.
struct TailCell {
    unsigned x, y, z, pos;
    __device__ __forceinline__ unsigned xr() const { return x & 0xffffu; }
    __device__ __forceinline__ unsigned xb() const { return x >> 16; }
    __device__ __forceinline__ int pi() const { return pos & 255; }
    __device__ __forceinline__ int py() const { return (pos >> 8) & 511; }
    __device__ __forceinline__ int pz() const { return (pos >> 17) & 511; }
    __device__ __forceinline__ int fr() const { return (pos >> 26) & 3; }
    __device__ __forceinline__ int fb() const { return (pos >> 28) & 3; }
};

template <typename T, bool BOX>
__device__ __forceinline__ TailCell tail_cell(int i, int y, int z, int hx, int ny, int nz, int zero) {
    const int row = (z * ny + y) * hx, plane = ny * hx, own = row + i;
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
        ym = y > 0 ? own - hx : own + plane - hx;
        yp = y + 1 < ny ? own + hx : own - (plane - hx);
        zm = z > 0 ? own - plane : own + (nz - 1) * plane;
        zp = z + 1 < nz ? own + plane : own - (nz - 1) * plane;
    }
    constexpr unsigned S = sizeof(T);
    TailCell c;
    c.x = (unsigned)(up ? right : left) * S | ((unsigned)(up ? left : right) * S << 16);
    c.y = (unsigned)ym * S | ((unsigned)yp * S << 16);
    c.z = (unsigned)zm * S | ((unsigned)zp * S << 16);
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

// Restriction of the split red residual R (black zero) to coarse cell (X, Y, Z): the red
// cells of a fine row of parity p among 2X-1 .. 2X+2 are those at index X-1 and X (p = 1)
// or X and X+1 (p = 0).
template <typename T, bool BOX>
__device__ __forceinline__ T tail_restrict(const T* R, int X, int Y, int Z, int hx, int ny, int nz) {
    const T w0 = (T)0.125, w1 = (T)0.375;
    const int xl = X == 0 ? hx - 1 : X - 1, xr = X + 1 == hx ? 0 : X + 1;
    T acc = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        int z = 2 * Z - 1 + c;
        T wz = (c == 0 || c == 3) ? w0 : w1;
        if (BOX) {
            if (z < 0 || z >= nz) wz = (T)0;
            else if ((c == 1 && z == 0) || (c == 2 && z == nz - 1)) wz = (T)0.25;
        }
        z = wrapi(z, nz);
        T accb = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            int y = 2 * Y - 1 + b;
            T wy = (b == 0 || b == 3) ? w0 : w1;
            if (BOX) {
                if (y < 0 || y >= ny) wy = (T)0;
                else if ((b == 1 && y == 0) || (b == 2 && y == ny - 1)) wy = (T)0.25;
            }
            y = wrapi(y, ny);
            const T* row = R + (z * ny + y) * hx;
            const int p = (y + z) & 1;
            const T m = row[X];
            T e = row[p ? xl : xr];
            T wm = w1;
            if (BOX) {
                if (p ? X == 0 : X + 1 == hx) e = (T)0;
                if (p ? X + 1 == hx : X == 0) wm = (T)0.25;  // the boundary fine cell of a boundary coarse cell
            }
            accb = fma(wy, restrict_row(w0, wm, p, e, m, e), accb);
        }
        acc = fma(wz, accb, acc);
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
        const T* r00 = C + (K0 * cy + J0) * cx;
        const T* r10 = C + (K0 * cy + J1) * cx;
        const T* r01 = C + (K1 * cy + J0) * cx;
        const T* r11 = C + (K1 * cy + J1) * cx;
        const T v00 = a0 * r00[I0] + a1 * r00[I1], v10 = a0 * r10[I0] + a1 * r10[I1];
        const T v01 = a0 * r01[I0] + a1 * r01[I1], v11 = a0 * r11[I0] + a1 * r11[I1];
        return u + (c0 * (b0 * v00 + b1 * v10) + c1 * (b0 * v01 + b1 * v11));
    }
    I1 = wrapi(I1, cx);
    J1 = wrapi(J1, cy);
    K1 = wrapi(K1, cz);
    const T* r00 = C + (K0 * cy + J0) * cx;
    const T* r10 = C + (K0 * cy + J1) * cx;
    const T* r01 = C + (K1 * cy + J0) * cx;
    const T* r11 = C + (K1 * cy + J1) * cx;
    return tri_add(u, r00[I0], r00[I1], r10[I0], r10[I1], r01[I0], r01[I1], r11[I0], r11[I1]);
}

// K indices of the first level per thread (index j = threadIdx.x + k * kTailThreads).
template <typename T, int K, bool BOX>
__device__ __forceinline__ void tail_run(const T* __restrict__ f0g, const T* __restrict__ f1g, T* __restrict__ u0g,
                                         T* __restrict__ u1g, const TailDesc& d, const double* __restrict__ specg,
                                         unsigned char* smem) {
    const int tid = threadIdx.x, L = d.nlev - 1;
    const int nx0 = d.nx[0], ny0 = d.ny[0], nz0 = d.nz[0], hx0 = nx0 >> 1, nh0 = hx0 * ny0 * nz0;
    T* const A0 = reinterpret_cast<T*>(smem + d.off_u[0]);  // red values, then a zero
    T* const A1 = A0 + nh0 + 1;                             // black values, then a zero
    double* const spec = reinterpret_cast<double*>(smem + d.off_spec);
    const TailCoef<T, BOX> c0(d, 0);
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
    for (int j = tid; j < d.nspec; j += kTailThreads) spec[j] = specg[j];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = tid + k * kTailThreads;
        if (j < nh0) {
            const int i = j % hx0, t = j / hx0, y = t % ny0, z = t / ny0;
            cell[k] = tail_cell<T, BOX>(i, y, z, hx0, ny0, nz0, nh0);
        }
    }
    if (BOX && tid == 0) A0[nh0] = A1[nh0] = (T)0;
    // half-sweeps of the first level; the barrier orders the written colour before its readers
    auto red = [&]() {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = tid + k * kTailThreads;
            if (j < nh0) {
                u0[k] = relax(f0[k], c0.s, tail_sum(A1, u1[k], cell[k].xr(), cell[k]), c0.inv(cell[k].fr()));
                A0[j] = u0[k];
            }
        }
        __syncthreads();
    };
    auto black = [&]() {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = tid + k * kTailThreads;
            if (j < nh0) {
                u1[k] = relax(f1[k], c0.s, tail_sum(A0, u0[k], cell[k].xb(), cell[k]), c0.inv(cell[k].fb()));
                A1[j] = u1[k];
            }
        }
        __syncthreads();
    };
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = tid + k * kTailThreads;
        if (j < nh0) {
            u0[k] = relax_zero(f0[k], c0.inv(cell[k].fr()));  // red sweep from zero
            A0[j] = u0[k];
        }
    }
    __syncthreads();
    black();
    red();
    black();
    // red residual, over the red values (every owner keeps its own)
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = tid + k * kTailThreads;
        if (j < nh0)
            A0[j] = red_resid(f0[k], c0.dg(cell[k].fr()), u0[k], c0.s, tail_sum(A1, u1[k], cell[k].xr(), cell[k]));
    }
    __syncthreads();
    // lower levels, down: u0 | 0 | u1 | 0 | f0 | f1 | r of the level, then its values in natural order
    const T* R = A0;
    int fhx = hx0, fny = ny0, fnz = nz0;
    for (int l = 1; l <= L; ++l) {
        const int nx = d.nx[l], ny = d.ny[l], nz = d.nz[l], n = nx * ny * nz;
        if (l == L) {
            double* a = reinterpret_cast<double*>(smem + d.off_ab);
            for (int j = tid; j < n; j += kTailThreads) {
                const int X = j % nx, t = j / nx;
                // the right-hand side is rounded to T, as the stored coarse level would be
                a[j] = (double)tail_restrict<T, BOX>(R, X, t % ny, t / ny, fhx, fny, fnz);
            }
            __syncthreads();
            break;
        }
        const int hx = nx >> 1, nh = hx * ny * nz;
        T* B0 = reinterpret_cast<T*>(smem + d.off_u[l]);
        T* B1 = B0 + nh + 1;
        T* F0 = B1 + nh + 1;
        T* F1 = F0 + nh;
        T* RR = F1 + nh;
        for (int j = tid; j < n; j += kTailThreads) {
            const int X = j % nx, t = j / nx, Y = t % ny, Z = t / ny;
            const T v = tail_restrict<T, BOX>(R, X, Y, Z, fhx, fny, fnz);
            (((X + Y + Z) & 1) ? F1 : F0)[(Z * ny + Y) * hx + (X >> 1)] = v;
        }
        if (BOX && tid == 0) B0[nh] = B1[nh] = (T)0;
        __syncthreads();
        const TailCoef<T, BOX> c(d, l);
        const bool on = tid < nh;
        T a = 0, b = 0, fa = 0, fb = 0;
        TailCell ce{};
        if (on) {
            const int i = tid % hx, t = tid / hx;
            ce = tail_cell<T, BOX>(i, t % ny, t / ny, hx, ny, nz, nh);
            fa = F0[tid];
            fb = F1[tid];
            a = relax_zero(fa, c.inv(ce.fr()));
            B0[tid] = a;
        }
        __syncthreads();
        if (on) B1[tid] = b = relax(fb, c.s, tail_sum(B0, a, ce.xb(), ce), c.inv(ce.fb()));
        __syncthreads();
        if (on) B0[tid] = a = relax(fa, c.s, tail_sum(B1, b, ce.xr(), ce), c.inv(ce.fr()));
        __syncthreads();
        if (on) B1[tid] = b = relax(fb, c.s, tail_sum(B0, a, ce.xb(), ce), c.inv(ce.fb()));
        __syncthreads();
        if (on) RR[tid] = red_resid(fa, c.dg(ce.fr()), a, c.s, tail_sum(B1, b, ce.xr(), ce));
        __syncthreads();
        R = RR;
        fhx = hx;
        fny = ny;
        fnz = nz;
    }
    // coarsest grid
    {
        const int nx = d.nx[L], ny = d.ny[L], nz = d.nz[L], m = nx * ny * nz;
        double* a = reinterpret_cast<double*>(smem + d.off_ab);
        spectral_solve(a, a + m, spec, nx, ny, nz);
        T* C = reinterpret_cast<T*>(smem + d.off_nat[L]);
        for (int j = tid; j < m; j += kTailThreads) C[j] = (T)a[j];
        __syncthreads();
    }
    // lower levels, up
    for (int l = L - 1; l >= 1; --l) {
        const int nx = d.nx[l], ny = d.ny[l], nz = d.nz[l], hx = nx >> 1, nh = hx * ny * nz;
        T* B0 = reinterpret_cast<T*>(smem + d.off_u[l]);
        T* B1 = B0 + nh + 1;
        const T* F0 = B1 + nh + 1;
        const T* F1 = F0 + nh;
        T* N = reinterpret_cast<T*>(smem + d.off_nat[l]);
        const T* C = reinterpret_cast<const T*>(smem + d.off_nat[l + 1]);
        const TailCoef<T, BOX> c(d, l);
        const bool on = tid < nh;
        T a = 0, b = 0, fa = 0, fb = 0;
        TailCell ce{};
        int i = 0, y = 0, z = 0;
        if (on) {
            i = tid % hx;
            const int t = tid / hx;
            y = t % ny;
            z = t / ny;
            ce = tail_cell<T, BOX>(i, y, z, hx, ny, nz, nh);
            fa = F0[tid];
            fb = F1[tid];
            a = tail_correct<T, BOX>(B0[tid], C, i, y, z, hx, ny >> 1, nz >> 1);
            B0[tid] = a;
        }
        __syncthreads();
        if (on) B1[tid] = b = relax(fb, c.s, tail_sum(B0, a, ce.xb(), ce), c.inv(ce.fb()));
        __syncthreads();
        if (on) B0[tid] = a = relax(fa, c.s, tail_sum(B1, b, ce.xr(), ce), c.inv(ce.fr()));
        __syncthreads();
        if (on) B1[tid] = b = relax(fb, c.s, tail_sum(B0, a, ce.xb(), ce), c.inv(ce.fb()));
        __syncthreads();
        if (on) {
            a = relax(fa, c.s, tail_sum(B1, b, ce.xr(), ce), c.inv(ce.fr()));
            const int row = (z * ny + y) * nx, up = (y + z) & 1;
            N[row + 2 * i + up] = a;
            N[row + 2 * i + (up ^ 1)] = b;
        }
        __syncthreads();
    }
    // first level, up
    const T* C = reinterpret_cast<const T*>(smem + d.off_nat[1]);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = tid + k * kTailThreads;
        if (j < nh0) {
            u0[k] = tail_correct<T, BOX>(u0[k], C, cell[k].pi(), cell[k].py(), cell[k].pz(), hx0, ny0 >> 1, nz0 >> 1);
            A0[j] = u0[k];
        }
    }
    __syncthreads();
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

// A grid that is itself the coarsest level: u = A^{-1} f (natural order, m <= 512 cells).
template <typename T>
__global__ void __launch_bounds__(kMaxCoarse) k_coarse(const T* __restrict__ f, T* __restrict__ u,
                                                       const double* __restrict__ specg, int nx, int ny, int nz,
                                                       int nspec, const Scalars* sc) {
    if (sc && sc->done) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int m = nx * ny * nz;
    double* a = reinterpret_cast<double*>(smem);
    double* spec = a + 2 * m;
    for (int j = threadIdx.x; j < m; j += blockDim.x) a[j] = (double)f[j];
    for (int j = threadIdx.x; j < nspec; j += blockDim.x) spec[j] = specg[j];
    __syncthreads();
    spectral_solve(a, a + m, spec, nx, ny, nz);
    for (int j = threadIdx.x; j < m; j += blockDim.x) u[j] = (T)a[j];
}

template <typename T>
void launch_coarse(hipStream_t st, const T* f, T* u, const double* spec, int nx, int ny, int nz, const Scalars* sc) {
    const int m = nx * ny * nz, nspec = nx * nx + ny * ny + nz * nz + m;
    hipLaunchKernelGGL(k_coarse<T>, dim3(1), dim3(kMaxCoarse), (2 * m + nspec) * sizeof(double), st, f, u, spec, nx,
                       ny, nz, nspec, sc);
}

#define BRD_TAIL_INST(T)                                                                                            \
    template void launch_tail<T>(hipStream_t, const T*, const T*, T*, T*, const TailDesc&, const double*, bool,     \
                                 const Scalars*);                                                                   \
    template void launchb_tail<T>(hipStream_t, const InstDev*, const int*, int, unsigned);                          \
    template hipError_t tail_set_lds<T>(size_t);                                                                    \
    template void launch_coarse<T>(hipStream_t, const T*, T*, const double*, int, int, int, const Scalars*);
BRD_TAIL_INST(float)
BRD_TAIL_INST(double)
#undef BRD_TAIL_INST

}  // namespace brd
