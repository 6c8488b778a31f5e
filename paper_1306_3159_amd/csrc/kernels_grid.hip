// Natural-layout FP64 grid kernels and the one-work-group finalize kernels.
//
// Operators (arXiv:1306.3159 Sec. III.A-III.B): A = alpha I - D L with L the
// periodic 7-point Laplacian; the CG vector updates of the multigrid-
// preconditioned Krylov solves of Sec. III.E.
#include "launch.hpp"

#include <cmath>

namespace brd {

// y = alpha x - s (sum of 6 neighbours - 6 x), s = D / h^2. BOX: a box with
// homogeneous faces, where the neighbour beyond a face is the ghost -x.
template <bool BOX>
__device__ __forceinline__ double stencil_A(const double* __restrict__ x, int X, int Y, int Z, int nx, int ny, int nz,
                                            double alpha, double s, size_t idx, double* center) {
    const long long sxy = (long long)nx * ny;
    const long long i = (long long)idx;
    const double c = x[i];
    double xm, xp, ym, yp, zm, zp;
    if (BOX) {
        xm = X > 0 ? x[i - 1] : -c;
        xp = X + 1 < nx ? x[i + 1] : -c;
        ym = Y > 0 ? x[i - nx] : -c;
        yp = Y + 1 < ny ? x[i + nx] : -c;
        zm = Z > 0 ? x[i - sxy] : -c;
        zp = Z + 1 < nz ? x[i + sxy] : -c;
    } else {
        xm = x[i - X + wrapi(X - 1, nx)];
        xp = x[i - X + wrapi(X + 1, nx)];
        ym = x[i + (long long)(wrapi(Y - 1, ny) - Y) * nx];
        yp = x[i + (long long)(wrapi(Y + 1, ny) - Y) * nx];
        zm = x[i + (long long)(wrapi(Z - 1, nz) - Z) * sxy];
        zp = x[i + (long long)(wrapi(Z + 1, nz) - Z) * sxy];
    }
    *center = c;
    return alpha * c - s * ((xm + xp) + (ym + yp) + (zm + zp) - 6.0 * c);
}

template <bool BOX>
__global__ void __launch_bounds__(kBlock) k_applyA(const double* __restrict__ p, double* __restrict__ q,
                                                   double alpha, double s, int nx, int ny, int nz, unsigned ncell,
                                                   double* part, const Scalars* sc) {
    if (sc && sc->done) return;
    unsigned lo, hi;
    chunk_of(xcd_block(blockIdx.x, gridDim.x), gridDim.x, ncell, &lo, &hi);
    double v[2] = {0.0, 0.0};
    for (unsigned idx = lo + threadIdx.x; idx < hi; idx += blockDim.x) {
        const int X = idx % nx;
        const unsigned t = idx / nx;
        const int Y = t % ny, Z = t / ny;
        double c;
        const double y = stencil_A<BOX>(p, X, Y, Z, nx, ny, nz, alpha, s, idx, &c);
        q[idx] = y;
        v[0] += c * y;
        v[1] += y;
    }
    if (part) block_partials<2>(v, part, gridDim.x, blockIdx.x);
}

typedef double double2_t __attribute__((ext_vector_type(2)));

// Sums of K values per index i < n (at(i, v) adds index i's to v) by kBlock threads, in the order
// of the finalize kernel's kFinBlock: each wave stands for four of its waves.
template <int K, typename At>
__device__ __forceinline__ void fold_sums(unsigned n, At at, double (&s)[K]) {
    __shared__ double sh[K][kFinBlock / 64];
    constexpr int J = kFinBlock / kBlock;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    double v[J][K] = {};
    for (unsigned i0 = 0; i0 < n; i0 += kFinBlock)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const unsigned i = i0 + (wid + j * (kBlock / 64)) * 64 + lane;
            if (i < n) at(i, v[j]);
        }
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double t = wave_sum(v[j][k]);
            if (lane == 0) sh[k][wid + j * (kBlock / 64)] = t;
        }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = lane_value(row_sum(lane < kFinBlock / 64 ? sh[k][lane & 15] : 0.0), 15);
    lds_barrier();
}
template <int K>
__device__ __forceinline__ void fold_partials(const CgFold& f, double (&s)[K]) {
    const double* p = f.in;
    const unsigned np = f.np;
    fold_sums<K>(np, [=](unsigned i, double (&v)[K]) {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] += p[(size_t)k * np + i];
    }, s);
}

// alpha p - D L p of the cells (x even, x + 1) whose row holds xl, c[0], c[1], xr, with its
// roundings fixed: every kernel that applies the operator to a vector gives the same bits.
__device__ __forceinline__ double2_t stencil_pair(double2_t c, double xl, double xr, double2_t ym, double2_t yp,
                                                  double2_t zm, double2_t zp, double alpha, double s) {
#pragma clang fp contract(off)
    const double a = ((xl + c[1]) + (ym[0] + yp[0])) + (zm[0] + zp[0]);
    const double b = ((c[0] + xr) + (ym[1] + yp[1])) + (zm[1] + zp[1]);
    return double2_t{fma(-s, fma(-6.0, c[0], a), alpha * c[0]), fma(-s, fma(-6.0, c[1], b), alpha * c[1])};
}

// Two cells per thread (x even, x + 1) with 16-byte loads: q = alpha p - D L p,
// partials (p.q, sum q).
template <bool BOX>
__device__ __forceinline__ void applyA2_body(const double* __restrict__ p, double* __restrict__ q, double alpha,
                                             double s, int nx, int ny, int nz, unsigned npair, double* part, Blk blk,
                                             const double* __restrict__ base = nullptr) {
    unsigned lo, hi;
    chunk_of(xcd_block(blk.b, blk.nb), blk.nb, npair, &lo, &hi);
    double v[2] = {0.0, 0.0};
    const int hx = nx >> 1;
    const long long sxy = (long long)nx * ny;
    // kU pairs per pass: every load of the pass is issued before any of its pairs is
    // computed (a chunk of several pairs per thread then keeps kU x 7 loads in flight);
    // pairs are computed and summed in the chunk's order, as one at a time would be
    constexpr int kU = 4;
    const unsigned bd = blockDim.x;
    for (unsigned k0 = lo + threadIdx.x; k0 < hi; k0 += kU * bd) {
        long long i[kU];
        int X[kU];
        double2_t c[kU], ym[kU], yp[kU], zm[kU], zp[kU], b[kU];
        double xl[kU], xr[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const unsigned k = k0 + u * bd;
            if (k >= hi) continue;
            X[u] = 2 * (int)(k % hx);
            const unsigned t = k / hx;
            const int Y = t % ny, Z = t / ny;
            i[u] = ((long long)Z * ny + Y) * nx + X[u];
            c[u] = *reinterpret_cast<const double2_t*>(p + i[u]);
            if (BOX) {
                xl[u] = X[u] > 0 ? p[i[u] - 1] : -c[u][0];
                xr[u] = X[u] + 2 < nx ? p[i[u] + 2] : -c[u][1];
                ym[u] = Y > 0 ? *reinterpret_cast<const double2_t*>(p + i[u] - nx) : -c[u];
                yp[u] = Y + 1 < ny ? *reinterpret_cast<const double2_t*>(p + i[u] + nx) : -c[u];
                zm[u] = Z > 0 ? *reinterpret_cast<const double2_t*>(p + i[u] - sxy) : -c[u];
                zp[u] = Z + 1 < nz ? *reinterpret_cast<const double2_t*>(p + i[u] + sxy) : -c[u];
            } else {
                xl[u] = p[i[u] - X[u] + (X[u] == 0 ? nx - 1 : X[u] - 1)];
                xr[u] = p[i[u] - X[u] + (X[u] + 2 == nx ? 0 : X[u] + 2)];
                ym[u] = *reinterpret_cast<const double2_t*>(p + i[u] + (long long)(wrapi(Y - 1, ny) - Y) * nx);
                yp[u] = *reinterpret_cast<const double2_t*>(p + i[u] + (long long)(wrapi(Y + 1, ny) - Y) * nx);
                zm[u] = *reinterpret_cast<const double2_t*>(p + i[u] + (long long)(wrapi(Z - 1, nz) - Z) * sxy);
                zp[u] = *reinterpret_cast<const double2_t*>(p + i[u] + (long long)(wrapi(Z + 1, nz) - Z) * sxy);
            }
            if (base) b[u] = *reinterpret_cast<const double2_t*>(base + i[u]);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (k0 + u * bd >= hi) continue;
            double2_t y = stencil_pair(c[u], xl[u], xr[u], ym[u], yp[u], zm[u], zp[u], alpha, s);
            if (base) {  // residual form q = base - A p
                y[0] = b[u][0] - y[0];
                y[1] = b[u][1] - y[1];
            }
            *reinterpret_cast<double2_t*>(q + i[u]) = y;
            v[0] += c[u][0] * y[0] + c[u][1] * y[1];
            v[1] += y[0] + y[1];
        }
    }
    if (part) block_partials<2>(v, part, blk.nb, blk.b);
}

template <bool BOX>
__global__ void __launch_bounds__(kBlock) k_applyA2(const double* __restrict__ p, double* __restrict__ q,
                                                    double alpha, double s, int nx, int ny, int nz, unsigned npair,
                                                    double* part, const Scalars* sc) {
    if (sc && sc->done) return;
    applyA2_body<BOX>(p, q, alpha, s, nx, ny, nz, npair, part, Blk{blockIdx.x, gridDim.x});
}

// q = base - (alpha p - D L p), two cells per thread (no partials)
template <bool BOX>
__global__ void __launch_bounds__(kBlock) k_residA2(const double* __restrict__ base, const double* __restrict__ p,
                                                    double* __restrict__ q, double alpha, double s, int nx, int ny,
                                                    int nz, unsigned npair) {
    applyA2_body<BOX>(p, q, alpha, s, nx, ny, nz, npair, nullptr, Blk{blockIdx.x, gridDim.x}, base);
}

void launch_applyA2(hipStream_t st, const double* p, double* q, double alpha, double s, int nx, int ny, int nz,
                    double* part, const Scalars* sc, unsigned* np, bool box) {
    const unsigned npair = (unsigned)(nx / 2) * ny * nz;
    const unsigned nb = red_blocks(npair);
    hipLaunchKernelGGL(box ? k_applyA2<true> : k_applyA2<false>, dim3(nb), dim3(kBlock), 0, st, p, q, alpha, s, nx,
                       ny, nz, npair, part, sc);
    *np = nb;
}

// Steps of x that iteration k = sc->iters applies before its direction: none at odd k (and
// k = 0), those of the two iterations before at even k. 1: x starts at zero and is not read.
__device__ __forceinline__ int cg_steps(const Scalars* sc) {
    return (sc->iters & 1) || sc->iters == 0 ? 0 : (sc->xzero && sc->iters == 2 ? 1 : 2);
}

// One CG direction and its product in one pass, two cells per thread:
//   pn = z + shift + beta po
//   q  = alpha pn - D L pn, partials (pn.q, sum q)
//   x += step[0] pn_old + step[1] po   (every second iteration: the steps of the last two, whose
//                                       directions are in the two buffers)
// Bound by bytes on large grids, by launches on small ones. Apart, the direction (reads z, po;
// writes pn), the stencil (reads pn; writes q) and the step of x in the update (reads po, x;
// writes x) move 8 words of 8 bytes and z per cell; here the neighbours' directions are formed
// again from z and po, which the caches hold, and 4.5 words and z move. pn and po are two
// buffers: a block reads neighbours of po that another block would have replaced.
// Measured per iteration, FP32 z: at 256^3 149 us and 75 us for the update (direction 57,
// stencil 58 and update 177 apart, in 4096 blocks; 4.5 TB/s here, which writes as many bytes as
// it reads); at 128^3 13.1 + 9.8 us (6.4 + 9.4 + 14.0) and a launch less.
template <typename T, bool BOX>
__device__ __forceinline__ void cg_dir_body(const T* __restrict__ z0, const T* __restrict__ z1,
                                            const double* __restrict__ po, double* __restrict__ pn,
                                            double* __restrict__ q, double* __restrict__ x, double alpha, double s,
                                            int nx, int ny, int nz, unsigned npair, double beta, double shift,
                                            double step0, double step1, int steps, bool old, double* part,
                                            Blk blk) {
    unsigned lo, hi;
    chunk_of(xcd_block(blk.b, blk.nb), blk.nb, npair, &lo, &hi);
    double v[2] = {0.0, 0.0};
    const int hx = nx >> 1, plane = hx * ny;
    const double2_t* po2 = reinterpret_cast<const double2_t*>(po);
    // kU pairs per pass: the loads of all are issued before any is computed
    constexpr int kU = 2;
    const unsigned bd = blockDim.x;
    for (unsigned k0 = lo + threadIdx.x; k0 < hi; k0 += kU * bd) {
        int X[kU], Y[kU], Z[kU];
        double2_t c[kU], ym[kU], yp[kU], zm[kU], zp[kU], xv[kU], pv[kU];
        T wc[kU][2], wl[kU], wr[kU], wy[kU][4], wz[kU][4];
        double xl[kU], xr[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const unsigned k = k0 + u * bd;
            if (k >= hi) continue;
            X[u] = (int)(k % hx);
            const unsigned t = k / hx;
            Y[u] = t % ny;
            Z[u] = t / ny;
            const int par = (Y[u] + Z[u]) & 1;  // colour of the row's even cells
            const T* ze = par ? z1 : z0;
            const T* zo = par ? z0 : z1;
            // neighbour pairs (out of the box: the pair itself, its value is not used)
            const int kl = (int)k + (X[u] > 0 ? -1 : (BOX ? 0 : hx - 1));
            const int kr = (int)k + (X[u] + 1 < hx ? 1 : (BOX ? 0 : 1 - hx));
            const int kym = (int)k + (Y[u] > 0 ? -hx : (BOX ? 0 : plane - hx));
            const int kyp = (int)k + (Y[u] + 1 < ny ? hx : (BOX ? 0 : hx - plane));
            const int kzm = (int)k + (Z[u] > 0 ? -plane : (BOX ? 0 : (nz - 1) * plane));
            const int kzp = (int)k + (Z[u] + 1 < nz ? plane : (BOX ? 0 : -(nz - 1) * plane));
            wc[u][0] = ze[k];
            wc[u][1] = zo[k];
            wl[u] = zo[kl];
            wr[u] = ze[kr];
            wy[u][0] = zo[kym];  // rows of the other parity: even cells in zo
            wy[u][1] = ze[kym];
            wy[u][2] = zo[kyp];
            wy[u][3] = ze[kyp];
            wz[u][0] = zo[kzm];
            wz[u][1] = ze[kzm];
            wz[u][2] = zo[kzp];
            wz[u][3] = ze[kzp];
            c[u] = ym[u] = yp[u] = zm[u] = zp[u] = xv[u] = pv[u] = double2_t{0.0, 0.0};
            xl[u] = xr[u] = 0.0;
            if (old) {
                c[u] = po2[k];
                xl[u] = po[2 * (size_t)kl + 1];
                xr[u] = po[2 * (size_t)kr];
                ym[u] = po2[kym];
                yp[u] = po2[kyp];
                zm[u] = po2[kzm];
                zp[u] = po2[kzp];
            }
            if (steps) pv[u] = reinterpret_cast<const double2_t*>(pn)[k];
            if (steps == 2) xv[u] = reinterpret_cast<const double2_t*>(x)[k];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const unsigned k = k0 + u * bd;
            if (k >= hi) continue;
            if (steps)
                reinterpret_cast<double2_t*>(x)[k] =
                    double2_t{fma(step1, c[u][0], fma(step0, pv[u][0], xv[u][0])),
                              fma(step1, c[u][1], fma(step0, pv[u][1], xv[u][1]))};
            auto dir = [&](T w, double o) { return fma(beta, o, (double)w + shift); };
            double2_t cn{dir(wc[u][0], c[u][0]), dir(wc[u][1], c[u][1])};
            double l = dir(wl[u], xl[u]), r = dir(wr[u], xr[u]);
            double2_t a{dir(wy[u][0], ym[u][0]), dir(wy[u][1], ym[u][1])};
            double2_t b{dir(wy[u][2], yp[u][0]), dir(wy[u][3], yp[u][1])};
            double2_t d{dir(wz[u][0], zm[u][0]), dir(wz[u][1], zm[u][1])};
            double2_t e{dir(wz[u][2], zp[u][0]), dir(wz[u][3], zp[u][1])};
            if (BOX) {
                if (X[u] == 0) l = -cn[0];
                if (X[u] + 1 == hx) r = -cn[1];
                if (Y[u] == 0) a = -cn;
                if (Y[u] + 1 == ny) b = -cn;
                if (Z[u] == 0) d = -cn;
                if (Z[u] + 1 == nz) e = -cn;
            }
            const double2_t y = stencil_pair(cn, l, r, a, b, d, e, alpha, s);
            reinterpret_cast<double2_t*>(pn)[k] = cn;
            reinterpret_cast<double2_t*>(q)[k] = y;
            v[0] += cn[0] * y[0] + cn[1] * y[1];
            v[1] += y[0] + y[1];
        }
    }
    block_partials<2>(v, part, blk.nb, blk.b);
}

template <typename T, bool BOX, bool FOLD>
__global__ void __launch_bounds__(kBlock) k_cg_dir(const T* __restrict__ z0, const T* __restrict__ z1,
                                                   const double* __restrict__ po, double* __restrict__ pn,
                                                   double* __restrict__ q, double* __restrict__ x, double alpha,
                                                   double s, int nx, int ny, int nz, unsigned npair, double* part,
                                                   Scalars* sc, CgFold fold) {
    if (!cg_dir_runs(sc)) return;
    double beta = 0.0, shift = 0.0;
    if (FOLD) {
        // every block forms beta; the first stores it, in fields that no block of this launch reads
        // (rz of this iteration beside that of the last; a breakdown in halt, not in done)
        double t[3];
        fold_partials<3>(fold, t);
        const CgBeta c = cg_beta(t[0], t[1], t[2], sc);
        if (blockIdx.x == 0 && threadIdx.x == 0) cg_beta_store(c, sc, true);
        if (c.bad) return;
        beta = c.beta;
        shift = c.shift;
    } else {
        beta = sc->beta;
        shift = sc->shift;
    }
    cg_dir_body<T, BOX>(z0, z1, po, pn, q, x, alpha, s, nx, ny, nz, npair, beta, shift, sc->step[0], sc->step[1],
                        cg_steps(sc), sc->iters > 0, part, Blk{blockIdx.x, gridDim.x});
}

template <typename T>
__global__ void __launch_bounds__(kBlock) kb_cg_dir(const InstDev* inst, const int* gate, const BatchTab* tab) {
    const BatchEntry* ent = tab_entries(tab);
    for (unsigned g = blockIdx.x; g < tab->total; g += gridDim.x) {
        Blk blk;
        const InstDev* I = batch_slot(inst, gate, ent, tab->n, g, blk);
        if (!I) continue;
        const Scalars* sc = I->sc;
        const int cur = sc->iters & 1;
        cg_dir_body<T, false>(static_cast<const T*>(I->lv[0][0]), static_cast<const T*>(I->lv[0][1]), I->p[cur ^ 1],
                              I->p[cur], I->q, I->x, I->alpha, I->ls[0], I->nx, I->ny, I->nz,
                              (unsigned)(I->nx / 2) * I->ny * I->nz, sc->beta, sc->shift, sc->step[0], sc->step[1],
                              cg_steps(sc), sc->iters > 0, I->part, blk);
        __syncthreads();  // partial-sum scratch is reused by the next virtual block
    }
}

template <typename T>
void launch_cg_dir(hipStream_t st, const T* z0, const T* z1, const double* po, double* pn, double* q, double* x,
                   double alpha, double s, int nx, int ny, int nz, double* part, Scalars* sc, unsigned* np, bool box,
                   const CgFold& fold) {
    const unsigned npair = (unsigned)(nx / 2) * ny * nz;
    const unsigned nb = cg_blocks(npair);
    const auto k = box ? (fold.np ? k_cg_dir<T, true, true> : k_cg_dir<T, true, false>)
                       : (fold.np ? k_cg_dir<T, false, true> : k_cg_dir<T, false, false>);
    hipLaunchKernelGGL(k, dim3(nb), dim3(kBlock), 0, st, z0, z1, po, pn, q, x, alpha, s, nx, ny, nz, npair, part, sc,
                       fold);
    *np = nb;
}
template void launch_cg_dir<float>(hipStream_t, const float*, const float*, const double*, double*, double*, double*,
                                   double, double, int, int, int, double*, Scalars*, unsigned*, bool, const CgFold&);
template void launch_cg_dir<double>(hipStream_t, const double*, const double*, const double*, double*, double*,
                                    double*, double, double, int, int, int, double*, Scalars*, unsigned*, bool,
                                    const CgFold&);

// The steps of x that no further direction applies: iterations sc->xsteps .. sc->iters - 1
// (at most two).
__global__ void __launch_bounds__(kBlock) k_cg_last(double* __restrict__ x, const double* __restrict__ p0,
                                                    const double* __restrict__ p1, unsigned npair,
                                                    const Scalars* sc) {
    const int first = sc->xsteps, n = sc->iters - first;
    const unsigned k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= npair || n <= 0) return;
    const int a = first & 1;
    const double2_t pv = reinterpret_cast<const double2_t*>(a ? p1 : p0)[k];
    double2_t xv = sc->xzero && first == 0 ? double2_t{0.0, 0.0} : reinterpret_cast<const double2_t*>(x)[k];
    xv = double2_t{fma(sc->step[a], pv[0], xv[0]), fma(sc->step[a], pv[1], xv[1])};
    if (n > 1) {
        const double2_t pw = reinterpret_cast<const double2_t*>(a ? p0 : p1)[k];
        xv = double2_t{fma(sc->step[a ^ 1], pw[0], xv[0]), fma(sc->step[a ^ 1], pw[1], xv[1])};
    }
    reinterpret_cast<double2_t*>(x)[k] = xv;
}
void launch_cg_last(hipStream_t st, double* x, const double* p0, const double* p1, size_t ncell, const Scalars* sc) {
    const unsigned npair = (unsigned)(ncell / 2);
    hipLaunchKernelGGL(k_cg_last, dim3(nblocks(npair)), dim3(kBlock), 0, st, x, p0, p1, npair, sc);
}

// r -= alpha q with partials (r.r, sum r), and the V-cycle
// entry for the new r in the same pass: f = r - mean (the mean predicted from
// sum r and sum q) into the split level-0 arrays, and the first red
// half-sweep from a zero guess, u_red = f_red / diag (as k_enter computes it).
// BOX: the diagonal of a box with fixed faces, per red cell from its face count.
template <typename T, bool BOX = false>
__device__ __forceinline__ void update2_enter_body(double* __restrict__ r, const double* __restrict__ q,
                                                   T* __restrict__ f0, T* __restrict__ f1, T* __restrict__ u0, int nx,
                                                   int ny, unsigned npair, double inv_diag, double a, double m,
                                                   double* part, Blk blk, int nz = 0, BoxCoef binv = BoxCoef{}) {
    unsigned lo, hi;
    chunk_of(xcd_block(blk.b, blk.nb), blk.nb, npair, &lo, &hi);
    double v[2] = {0.0, 0.0};
    const int hx = nx >> 1;
    for (unsigned k = lo + threadIdx.x; k < hi; k += blockDim.x) {
        double2_t rv = reinterpret_cast<double2_t*>(r)[k];
        const double2_t qv = reinterpret_cast<const double2_t*>(q)[k];
        rv[0] -= a * qv[0];
        rv[1] -= a * qv[1];
        reinterpret_cast<double2_t*>(r)[k] = rv;
        v[0] += rv[0] * rv[0] + rv[1] * rv[1];
        v[1] += rv[0] + rv[1];
        const unsigned t = k / hx;
        const int par = ((int)(t % ny) + (int)(t / ny)) & 1;  // colour of the even cell
        const double fa = rv[0] - m, fb = rv[1] - m;
        const double fr = par ? fb : fa, fk = par ? fa : fb;
        f0[k] = (T)fr;
        f1[k] = (T)fk;
        if (!u0) continue;  // the cycle opens from f
        if (BOX) {
            const int xr = 2 * (int)(k % hx) + par;  // the red cell of the pair
            u0[k] = (T)((T)fr * (T)binv.v[box_faces(xr, (int)(t % ny), (int)(t / ny), nx, ny, nz)]);
        } else {
            u0[k] = (T)((T)fr * (T)inv_diag);
        }
    }
    block_partials<2>(v, part, blk.nb, blk.b);
}

// alpha and the removed mean for an update (false: CG has broken down): folded as in k_cg_dir.
template <bool FOLD>
__device__ __forceinline__ bool cg_fold_alpha(const CgFold& fold, Scalars* sc, double& alpha, double& mean) {
    if (!FOLD) {
        alpha = sc->alpha;
        mean = sc->mean_next;
        return true;
    }
    double t[2];
    fold_partials<2>(fold, t);
    if (fold.na) {
        const double *na = fold.na, *nb = fold.nb;
        double b[2];
        fold_sums<2>((unsigned)fold.n, [=](unsigned i, double (&v)[2]) {
            const double y = nb[i];
            v[0] = fma(na[i], y, v[0]);
            v[1] += y;
        }, b);
        t[0] = fma(fold.inv_h3, b[0], t[0]);
        t[1] = fma(fold.inv_h3, b[1], t[1]);
    }
    const CgAlpha c = cg_alpha(t[0], t[1], sc);
    if (blockIdx.x == 0 && threadIdx.x == 0) cg_alpha_store(c, t[0], t[1], sc, true);
    alpha = c.alpha;
    mean = c.mean;
    return !c.bad;
}

template <typename T, bool FOLD>
__global__ void __launch_bounds__(kBlock) k_update2_enter(double* __restrict__ r, const double* __restrict__ q,
                                                          T* __restrict__ f0, T* __restrict__ f1, T* __restrict__ u0,
                                                          int nx, int ny, unsigned npair, double inv_diag,
                                                          double* part, Scalars* sc, CgFold fold) {
    if (!cg_update_runs(sc)) return;
    double a, m;
    if (!cg_fold_alpha<FOLD>(fold, sc, a, m)) return;
    update2_enter_body<T>(r, q, f0, f1, u0, nx, ny, npair, inv_diag, a, m, part, Blk{blockIdx.x, gridDim.x});
}

template <typename T, bool FOLD>
__global__ void __launch_bounds__(kBlock) k_update2_enter_box(double* __restrict__ r, const double* __restrict__ q,
                                                              T* __restrict__ f0,
                                                              T* __restrict__ f1, T* __restrict__ u0, int nx, int ny,
                                                              int nz, unsigned npair, BoxCoef binv, double* part,
                                                              Scalars* sc, CgFold fold) {
    if (!cg_update_runs(sc)) return;
    double a, m;
    if (!cg_fold_alpha<FOLD>(fold, sc, a, m)) return;
    update2_enter_body<T, true>(r, q, f0, f1, u0, nx, ny, npair, 0.0, a, m,
                                part, Blk{blockIdx.x, gridDim.x}, nz, binv);
}

template <typename T>
__global__ void __launch_bounds__(kBlock) kb_update2_enter(const InstDev* inst, const int* gate, const BatchTab* tab) {
    const BatchEntry* ent = tab_entries(tab);
    for (unsigned g = blockIdx.x; g < tab->total; g += gridDim.x) {
        Blk blk;
        const InstDev* I = batch_slot(inst, gate, ent, tab->n, g, blk);
        if (!I) continue;
        update2_enter_body<T>(I->r, I->q, static_cast<T*>(I->lv[0][2]), static_cast<T*>(I->lv[0][3]),
                              static_cast<T*>(I->lv[0][0]), I->nx, I->ny, (unsigned)(I->nx / 2) * I->ny * I->nz,
                              1.0 / I->ldiag[0], I->sc->alpha, I->sc->mean_next, I->part, blk);
        __syncthreads();  // partial-sum scratch is reused by the next virtual block
    }
}

template <typename T>
void launch_update2_enter(hipStream_t st, double* r, const double* q, T* f0, T* f1, T* u0,
                          int nx, int ny, int nz, double inv_diag, double* part, Scalars* sc, unsigned* np,
                          const BoxCoef* box_inv, const CgFold& fold) {
    const unsigned npair = (unsigned)(nx / 2) * ny * nz;
    const unsigned nb = cg_blocks(npair);
    if (box_inv) {
        const auto k = fold.np ? k_update2_enter_box<T, true> : k_update2_enter_box<T, false>;
        hipLaunchKernelGGL(k, dim3(nb), dim3(kBlock), 0, st, r, q, f0, f1, u0, nx, ny, nz, npair, *box_inv, part, sc,
                           fold);
    } else {
        const auto k = fold.np ? k_update2_enter<T, true> : k_update2_enter<T, false>;
        hipLaunchKernelGGL(k, dim3(nb), dim3(kBlock), 0, st, r, q, f0, f1, u0, nx, ny, npair, inv_diag, part, sc, fold);
    }
    *np = nb;
}
template void launch_update2_enter<float>(hipStream_t, double*, const double*, float*, float*,
                                          float*, int, int, int, double, double*, Scalars*, unsigned*,
                                          const BoxCoef*, const CgFold&);
template void launch_update2_enter<double>(hipStream_t, double*, const double*, double*,
                                           double*, double*, int, int, int, double, double*, Scalars*,
                                           unsigned*, const BoxCoef*, const CgFold&);

// partials (sum z, z.r, z.q), two cells per thread
template <typename T>
__global__ void __launch_bounds__(kBlock) k_zdots2(const T* __restrict__ z0, const T* __restrict__ z1,
                                                   const double* __restrict__ r, const double* __restrict__ q,
                                                   int nx, int ny, unsigned npair, double* part, const Scalars* sc) {
    if (sc->done) return;
    unsigned lo, hi;
    chunk_of(xcd_block(blockIdx.x, gridDim.x), gridDim.x, npair, &lo, &hi);
    double v[3] = {0.0, 0.0, 0.0};
    const int hx = nx >> 1;
    for (unsigned k = lo + threadIdx.x; k < hi; k += blockDim.x) {
        const unsigned t = k / hx;
        const int par = ((int)(t % ny) + (int)(t / ny)) & 1;
        const double za = (double)(par ? z1[k] : z0[k]);
        const double zb = (double)(par ? z0[k] : z1[k]);
        const double2_t rv = reinterpret_cast<const double2_t*>(r)[k];
        const double2_t qv = reinterpret_cast<const double2_t*>(q)[k];
        v[0] += za + zb;
        v[1] += za * rv[0] + zb * rv[1];
        v[2] += za * qv[0] + zb * qv[1];
    }
    block_partials<3>(v, part, gridDim.x, blockIdx.x);
}

template <typename T>
void launch_zdots2(hipStream_t st, const T* z0, const T* z1, const double* r, const double* q, int nx, int ny, int nz,
                   double* part, const Scalars* sc, unsigned* np) {
    const unsigned npair = (unsigned)(nx / 2) * ny * nz;
    const unsigned nb = red_blocks(npair);
    hipLaunchKernelGGL(k_zdots2<T>, dim3(nb), dim3(kBlock), 0, st, z0, z1, r, q, nx, ny, npair, part, sc);
    *np = nb;
}
template void launch_zdots2<float>(hipStream_t, const float*, const float*, const double*, const double*, int, int,
                                   int, double*, const Scalars*, unsigned*);
template void launch_zdots2<double>(hipStream_t, const double*, const double*, const double*, const double*, int,
                                    int, int, double*, const Scalars*, unsigned*);

// pairs of cells per thread of the plain stencil launches (BLOB_RD_STENCIL_PAIRS, default 2:
// at 256^3 38 us warm and 71 us cold against 50 and 77 with one pair per thread)
unsigned stencil_pairs() {
    static const unsigned v = [] {
        const char* e = std::getenv("BLOB_RD_STENCIL_PAIRS");
        const int k = e ? std::atoi(e) : 2;
        return (unsigned)(k >= 1 && k <= 16 ? k : 2);
    }();
    return v;
}

void launch_applyA_plain(hipStream_t st, const double* x, double* y, double alpha, double s, int nx, int ny,
                         int nz, bool box) {
    const unsigned n = (unsigned)nx * ny * nz;
    if (nx % 2 == 0) {  // two cells per thread, the same arithmetic
        const unsigned npair = n / 2;
        hipLaunchKernelGGL(box ? k_applyA2<true> : k_applyA2<false>, dim3(nblocks(npair, kBlock * stencil_pairs())),
                           dim3(kBlock), 0, st, x, y, alpha, s, nx, ny, nz, npair, (double*)nullptr,
                           (const Scalars*)nullptr);
        return;
    }
    hipLaunchKernelGGL(box ? k_applyA<true> : k_applyA<false>, dim3(nblocks(n)), dim3(kBlock), 0, st, x, y, alpha,
                       s, nx, ny, nz, n, (double*)nullptr, (const Scalars*)nullptr);
}

void launch_residA_plain(hipStream_t st, const double* base, const double* x, double* q, double alpha, double s,
                         int nx, int ny, int nz, bool box) {
    const unsigned n = (unsigned)nx * ny * nz;
    if (nx % 2 == 0) {
        const unsigned npair = n / 2;
        hipLaunchKernelGGL(box ? k_residA2<true> : k_residA2<false>, dim3(nblocks(npair, kBlock * stencil_pairs())),
                           dim3(kBlock), 0, st, base, x, q, alpha, s, nx, ny, nz, npair);
        return;
    }
    launch_applyA_plain(st, x, q, alpha, s, nx, ny, nz, box);
    launch_axpby(st, q, base, n, -1.0, 1.0);
}

// r = g - (alpha x - D L x) or, with x == nullptr, r = g - q0 (q0 may be null: r = g).
__global__ void __launch_bounds__(kBlock) k_residual64(const double* __restrict__ g, const double* __restrict__ x,
                                                       const double* __restrict__ q0, double* __restrict__ r,
                                                       double alpha, double s, int nx, int ny, int nz,
                                                       unsigned ncell, double* part) {
    unsigned lo, hi;
    chunk_of(xcd_block(blockIdx.x, gridDim.x), gridDim.x, ncell, &lo, &hi);
    double v[3] = {0.0, 0.0, 0.0};
    for (unsigned idx = lo + threadIdx.x; idx < hi; idx += blockDim.x) {
        double ax = 0.0;
        if (x) {
            const int X = idx % nx;
            const unsigned t = idx / nx;
            double c;
            ax = stencil_A<false>(x, X, (int)(t % ny), (int)(t / ny), nx, ny, nz, alpha, s, idx, &c);
        } else if (q0) {
            ax = q0[idx];
        }
        const double gv = g[idx];
        const double rv = gv - ax;
        r[idx] = rv;
        v[0] += rv * rv;
        v[1] += rv;
        v[2] += gv * gv;
    }
    block_partials<3>(v, part, gridDim.x, blockIdx.x);
}

// The partials of launch_residual_from_q(g, null, r) when r already holds g:
// (g.g, sum g, g.g), same chunks and order.
__global__ void __launch_bounds__(kBlock) k_self_partials(const double* __restrict__ g, unsigned n, double* part) {
    unsigned lo, hi;
    chunk_of(xcd_block(blockIdx.x, gridDim.x), gridDim.x, n, &lo, &hi);
    double v[3] = {0.0, 0.0, 0.0};
    for (unsigned idx = lo + threadIdx.x; idx < hi; idx += blockDim.x) {
        const double gv = g[idx];
        const double rv = gv - 0.0;
        v[0] += rv * rv;
        v[1] += rv;
        v[2] += gv * gv;
    }
    block_partials<3>(v, part, gridDim.x, blockIdx.x);
}

void launch_self_partials(hipStream_t st, const double* g, size_t n, double* part, unsigned* np) {
    const unsigned nb = red_blocks(n);
    hipLaunchKernelGGL(k_self_partials, dim3(nb), dim3(kBlock), 0, st, g, (unsigned)n, part);
    *np = nb;
}

void launch_residual_from_q(hipStream_t st, const double* g, const double* q0, double* r, size_t n, double* part,
                            unsigned* np) {
    const unsigned nb = red_blocks(n);
    hipLaunchKernelGGL(k_residual64, dim3(nb), dim3(kBlock), 0, st, g, (const double*)nullptr, q0, r, 0.0, 0.0, 1,
                       1, 1, (unsigned)n, part);
    *np = nb;
}

// Split-layout value at natural (X, Y, Z) of level 0.

// out = scale * out + z (+ shift_scale * *shift_dev)   (z split -> natural)
template <typename T>
__global__ void __launch_bounds__(kBlock) k_split_to_nat(const T* __restrict__ z0, const T* __restrict__ z1,
                                                         double* __restrict__ out, int nx, int ny, unsigned ncell,
                                                         double scale, const double* __restrict__ shift_dev,
                                                         double shift_scale) {
    const unsigned idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= ncell) return;
    const int X = idx % nx;
    const unsigned t = idx / nx;
    const double zv = split_at(z0, z1, X, (int)(t % ny), (int)(t / ny), nx >> 1, ny);
    double v = scale == 0.0 ? zv : scale * out[idx] + zv;
    if (shift_dev) v += shift_scale * shift_dev[0];
    out[idx] = v;
}

// Pair form: the element j of each colour array per thread, i.e. the natural cells
// x = 2i and 2i + 1 of a row (x = 2i has colour (y + z) & 1, x = 2i + 1 the other), which
// sit at 2j and 2j + 1 of the natural vector; each computed as in the one-cell form.
template <typename T>
__global__ void __launch_bounds__(kBlock) k_split_to_nat2(const T* __restrict__ z0, const T* __restrict__ z1,
                                                          double* __restrict__ out, int hx, int ny, unsigned nh,
                                                          double scale, const double* __restrict__ shift_dev,
                                                          double shift_scale) {
    typedef double D2 __attribute__((ext_vector_type(2)));
    const unsigned idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nh) return;
    const unsigned t = idx / hx;  // row z * ny + y
    const int p = ((int)(t % ny) + (int)(t / ny)) & 1;
    const double a = (double)z0[idx], b = (double)z1[idx];
    const double e0 = p ? b : a, e1 = p ? a : b;
    D2* o = reinterpret_cast<D2*>(out) + idx;
    double v0, v1;
    if (scale == 0.0) {
        v0 = e0;
        v1 = e1;
    } else {
        const D2 prev = *o;
        v0 = scale * prev[0] + e0;
        v1 = scale * prev[1] + e1;
    }
    if (shift_dev) {
        v0 += shift_scale * shift_dev[0];
        v1 += shift_scale * shift_dev[0];
    }
    *o = D2{v0, v1};
}

template <typename T>
void launch_split_to_nat(hipStream_t st, const T* z0, const T* z1, double* out, int nx, int ny, int nz,
                         double scale, const double* shift_dev, double shift_scale) {
    if (nx % 2 == 0) {
        const unsigned nh = (unsigned)(nx / 2) * ny * nz;
        hipLaunchKernelGGL(k_split_to_nat2<T>, dim3(nblocks(nh)), dim3(kBlock), 0, st, z0, z1, out, nx / 2, ny, nh,
                           scale, shift_dev, shift_scale);
        return;
    }
    const unsigned n = (unsigned)nx * ny * nz;
    hipLaunchKernelGGL(k_split_to_nat<T>, dim3(nblocks(n)), dim3(kBlock), 0, st, z0, z1, out, nx, ny, n, scale,
                       shift_dev, shift_scale);
}
template void launch_split_to_nat<float>(hipStream_t, const float*, const float*, double*, int, int, int, double,
                                         const double*, double);
template void launch_split_to_nat<double>(hipStream_t, const double*, const double*, double*, int, int, int, double,
                                          const double*, double);

// out = (b + z) + shift_scale * *shift_dev with b and z in the split layout (pair form, nx
// even): what k_split_to_nat2 with scale 1 writes when out holds the natural copy of b.
template <typename T>
__global__ void __launch_bounds__(kBlock) k_split_add_to_nat2(const T* __restrict__ b0, const T* __restrict__ b1,
                                                              const T* __restrict__ z0, const T* __restrict__ z1,
                                                              double* __restrict__ out, int hx, int ny, unsigned nh,
                                                              const double* __restrict__ shift_dev,
                                                              double shift_scale) {
    typedef double D2 __attribute__((ext_vector_type(2)));
    const unsigned idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nh) return;
    const unsigned t = idx / hx;  // row z * ny + y
    const int p = ((int)(t % ny) + (int)(t / ny)) & 1;
    const double a = (double)z0[idx], b = (double)z1[idx];
    const double ba = (double)b0[idx], bb = (double)b1[idx];
    double v0 = (p ? bb : ba) + (p ? b : a);
    double v1 = (p ? ba : bb) + (p ? a : b);
    if (shift_dev) {
        v0 += shift_scale * shift_dev[0];
        v1 += shift_scale * shift_dev[0];
    }
    reinterpret_cast<D2*>(out)[idx] = D2{v0, v1};
}

template <typename T>
void launch_split_add_to_nat(hipStream_t st, const T* b0, const T* b1, const T* z0, const T* z1, double* out, int nx,
                             int ny, int nz, const double* shift_dev, double shift_scale) {
    const unsigned nh = (unsigned)(nx / 2) * ny * nz;
    hipLaunchKernelGGL(k_split_add_to_nat2<T>, dim3(nblocks(nh)), dim3(kBlock), 0, st, b0, b1, z0, z1, out, nx / 2,
                       ny, nh, shift_dev, shift_scale);
}
template void launch_split_add_to_nat<float>(hipStream_t, const float*, const float*, const float*, const float*,
                                             double*, int, int, int, const double*, double);
template void launch_split_add_to_nat<double>(hipStream_t, const double*, const double*, const double*,
                                              const double*, double*, int, int, int, const double*, double);

__global__ void __launch_bounds__(kBlock) k_norm_partials(const double* __restrict__ v, unsigned n, double* part) {
    unsigned lo, hi;
    chunk_of(blockIdx.x, gridDim.x, n, &lo, &hi);
    double a[2] = {0.0, 0.0};
    for (unsigned idx = lo + threadIdx.x; idx < hi; idx += blockDim.x) {
        a[0] += v[idx];
        a[1] += v[idx] * v[idx];
    }
    block_partials<2>(a, part, gridDim.x, blockIdx.x);
}

void launch_norm_partials(hipStream_t st, const double* v, size_t n, double* part, unsigned* np) {
    const unsigned nb = red_blocks(n);
    hipLaunchKernelGGL(k_norm_partials, dim3(nb), dim3(kBlock), 0, st, v, (unsigned)n, part);
    *np = nb;
}

// Measurement probe: out = a + b over n16 16-byte vectors, the launch shape of the vector
// half-sweep (one vector per thread, XCD-mapped blocks): the bandwidth a plain streaming
// launch of the sweep's size reaches, the ceiling its roofline fraction is read against.
__global__ void __launch_bounds__(kBlock) k_stream_add(const float4* __restrict__ a, const float4* __restrict__ b,
                                                       float4* __restrict__ out, unsigned n16) {
    const unsigned idx = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (idx >= n16) return;
    const float4 x = a[idx], y = b[idx];
    out[idx] = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
}
void launch_stream_add(hipStream_t st, const void* a, const void* b, void* out, size_t bytes) {
    const unsigned n16 = (unsigned)(bytes / 16);
    hipLaunchKernelGGL(k_stream_add, dim3(nblocks(n16)), dim3(kBlock), 0, st, (const float4*)a, (const float4*)b,
                       (float4*)out, n16);
}

__global__ void k_fill(double* v, unsigned n, double value) {
    const unsigned idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < n) v[idx] = value;
}
void launch_fill(hipStream_t st, double* v, size_t n, double value) {
    hipLaunchKernelGGL(k_fill, dim3(nblocks(n)), dim3(kBlock), 0, st, v, (unsigned)n, value);
}

__global__ void k_axpby(double* y, const double* x, unsigned n, double a, double b) {
    const unsigned idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < n) y[idx] = (a == 0.0 ? 0.0 : a * y[idx]) + b * x[idx];
}
void launch_axpby(hipStream_t st, double* y, const double* x, size_t n, double a, double b) {
    hipLaunchKernelGGL(k_axpby, dim3(nblocks(n)), dim3(kBlock), 0, st, y, x, (unsigned)n, a, b);
}

__global__ void k_add_shift(double* v, unsigned n, const double* shift, double sign) {
    const unsigned idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < n) v[idx] += sign * shift[0];
}
void launch_add_shift(hipStream_t st, double* v, size_t n, const double* shift_dev, double sign) {
    hipLaunchKernelGGL(k_add_shift, dim3(nblocks(n)), dim3(kBlock), 0, st, v, (unsigned)n, shift_dev, sign);
}

// ---------------------------------------------------------------------------
// Finalize: one work-group of kFinBlock threads reduces block partials in a
// fixed order and advances the CG scalars.
// ---------------------------------------------------------------------------
// Sums of K sets of n partials each (set k at p + k n): every load of four strides of every
// set is issued before the first is added, then one reduction for all.
template <int K>
__device__ __forceinline__ void fin_sums(const double* __restrict__ p, unsigned n, double (&s)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = 0.0;
    for (unsigned i0 = threadIdx.x; i0 < n; i0 += 4 * blockDim.x) {
        double v[K][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned i = i0 + u * blockDim.x;
#pragma unroll
            for (int k = 0; k < K; ++k) v[k][u] = i < n ? p[(size_t)k * n + i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) s[k] += v[k][u];
    }
    wg_sums<K>(s);
}
__device__ __forceinline__ double fin_sum(const double* __restrict__ p, unsigned n) {
    double s[1];
    fin_sums<1>(p, n, s);
    return s[0];
}

__device__ __forceinline__ void fin_body(int kind, const double* __restrict__ part, unsigned np, Scalars* sc,
                                         const double* __restrict__ na, const double* __restrict__ nb, int nblob,
                                         double inv_h3) {
    if (kind == FIN_INIT) {
        double t[3];
        fin_sums<3>(part, np, t);
        const double rr = t[0], rs = t[1], gg = t[2];
        if (threadIdx.x == 0) {
            // On entry tol2 holds rtol^2 and rr0 holds an absolute floor^2.
            const double t2 = fmax(sc->tol2 * gg, sc->rr0);
            sc->rr = rr;
            sc->rr0 = rr;
            sc->rsum = rs;
            sc->gg = gg;
            sc->tol2 = t2;
            sc->iters = 0;
            sc->xsteps = 0;
            sc->beta = 0.0;
            sc->status = is_finite_d(rr) ? 0 : 1;
            sc->done = (rr <= t2 || !is_finite_d(rr)) ? 1 : 0;
            sc->mean_r = sc->project ? rs * sc->inv_ncell : 0.0;
        }
    } else if (kind == FIN_ALPHA) {
        double t[2];
        fin_sums<2>(part, np, t);
        double pq = t[0], qs = t[1];
        if (na && nb) {
            // blob term of B: p.(S mu) = h^-3 (J p).mu, sum(S mu) = h^-3 sum(mu)
            double b[2] = {0.0, 0.0};
            for (int i0 = threadIdx.x; i0 < nblob; i0 += 4 * blockDim.x) {
                double x[4], y[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u * (int)blockDim.x;
                    x[u] = i < nblob ? na[i] : 0.0;
                    y[u] = i < nblob ? nb[i] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    b[0] = fma(x[u], y[u], b[0]);
                    b[1] += y[u];
                }
            }
            wg_sums<2>(b);
            const double ta = b[0], tc = b[1];
            pq = fma(inv_h3, ta, pq);
            qs = fma(inv_h3, tc, qs);
        }
        if (threadIdx.x == 0) cg_alpha_store(cg_alpha(pq, qs, sc), pq, qs, sc, false);
    } else if (kind == FIN_UPDATE) {
        double t[2];
        fin_sums<2>(part, np, t);
        const double rr = t[0], rs = t[1];
        if (threadIdx.x == 0) {
            sc->rr = rr;
            sc->rsum = rs;
            sc->iters += 1;
            sc->mean_r = sc->project ? rs * sc->inv_ncell : 0.0;
            if (!is_finite_d(rr)) {
                sc->status = 1;
                sc->done = 1;
            } else if (rr <= sc->tol2) {
                sc->done = 1;
            }
        }
    } else {  // FIN_BETA
        double t[3];
        fin_sums<3>(part, np, t);
        if (threadIdx.x == 0) cg_beta_store(cg_beta(t[0], t[1], t[2], sc), sc, false);
    }
}

__global__ void __launch_bounds__(kFinBlock) k_fin(int kind, const double* __restrict__ part, unsigned np,
                                                   Scalars* sc, const double* __restrict__ na,
                                                   const double* __restrict__ nb, int nblob, double inv_h3) {
    if (kind != FIN_INIT) {
        if (sc->done) return;
        if (cg_halted(sc)) {
            if (threadIdx.x == 0) cg_stop(sc);  // waves that see done set return as well
            return;
        }
    }
    fin_body(kind, part, np, sc, na, nb, nblob, inv_h3);
}

void launch_fin(hipStream_t st, int kind, const double* part, unsigned np, Scalars* sc, const double* na,
                const double* nb, int nblob, double inv_h3) {
    hipLaunchKernelGGL(k_fin, dim3(1), dim3(kFinBlock), 0, st, kind, part, np, sc, na, nb, nblob, inv_h3);
}

// One work-group per instance: FIN_ALPHA (with the blob sums of blob
// instances), FIN_UPDATE or FIN_BETA of every gated, unfinished instance.
__global__ void __launch_bounds__(kFinBlock) kb_fin(int kind, const InstDev* inst, const int* gate, int ninst) {
    const int i = blockIdx.x;
    if (i >= ninst || !gate[i]) return;
    const InstDev* I = inst + i;
    if (I->sc->done) return;
    const unsigned np = kind == FIN_ALPHA ? I->np_apply : kind == FIN_UPDATE ? I->np_update : I->np_dots;
    const bool blob = kind == FIN_ALPHA && I->blobs;
    fin_body(kind, I->part, np, I->sc, blob ? I->jx : nullptr, blob ? I->mu : nullptr, blob ? I->N : 0, I->inv_h3);
}

template <typename T>
void launchb_cg(hipStream_t st, int what, const InstDev* inst, const int* gate, const BatchTab* tab, unsigned grid,
                int ninst) {
    const dim3 g(grid), b(kBlock);
    switch (what) {
        case BCG_DIR: hipLaunchKernelGGL(kb_cg_dir<T>, g, b, 0, st, inst, gate, tab); break;
        case BCG_UPDATE: hipLaunchKernelGGL(kb_update2_enter<T>, g, b, 0, st, inst, gate, tab); break;
        default:
            hipLaunchKernelGGL(kb_fin, dim3(ninst), dim3(kFinBlock), 0, st,
                               what == BCG_FIN_ALPHA ? FIN_ALPHA : what == BCG_FIN_UPDATE ? FIN_UPDATE : FIN_BETA,
                               inst, gate, ninst);
    }
}
template void launchb_cg<float>(hipStream_t, int, const InstDev*, const int*, const BatchTab*, unsigned, int);
template void launchb_cg<double>(hipStream_t, int, const InstDev*, const int*, const BatchTab*, unsigned, int);

__global__ void __launch_bounds__(kFinBlock) k_reduce_parts(const double* __restrict__ part, unsigned np, int k,
                                                            double* out) {
    for (int j = 0; j < k; ++j) {
        const double s = fin_sum(part + (size_t)j * np, np);
        if (threadIdx.x == 0) out[j] = s;
    }
}

void launch_reduce_parts(hipStream_t st, const double* part, unsigned np, int k, double* out) {
    hipLaunchKernelGGL(k_reduce_parts, dim3(1), dim3(kFinBlock), 0, st, part, np, k, out);
}

// ---------------------------------------------------------------------------
// Long vectors of the flexible GMRES on the block saddle system: a grid part of
// ncell values followed by N blob values, n = ncell + N doubles, each vector
// 16-byte aligned. Two values per thread (16-byte loads), one scalar tail.
// ---------------------------------------------------------------------------

// One modified Gram-Schmidt pass: w -= (*hprev) vprev when vprev is set, then
// partials of w.vnext (of w.w when vnext is null) into part[block].
__global__ void __launch_bounds__(kBlock) k_fg_mgs(double* __restrict__ w, const double* __restrict__ vprev,
                                                   const double* __restrict__ hprev, const double* __restrict__ vnext,
                                                   unsigned n, double* part) {
    const unsigned n2 = n >> 1;
    unsigned lo, hi;
    chunk_of(blockIdx.x, gridDim.x, n2, &lo, &hi);
    const double hp = vprev ? *hprev : 0.0;
    double a[1] = {0.0};
    double2* w2 = reinterpret_cast<double2*>(w);
    for (unsigned p = lo + threadIdx.x; p < hi; p += blockDim.x) {
        double2 x = w2[p];
        if (vprev) {
            const double2 v = reinterpret_cast<const double2*>(vprev)[p];
            x.x -= hp * v.x;
            x.y -= hp * v.y;
            w2[p] = x;
        }
        if (vnext) {
            const double2 v = reinterpret_cast<const double2*>(vnext)[p];
            a[0] += x.x * v.x + x.y * v.y;
        } else {
            a[0] += x.x * x.x + x.y * x.y;
        }
    }
    if ((n & 1u) && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        double x = w[n - 1];
        if (vprev) {
            x -= hp * vprev[n - 1];
            w[n - 1] = x;
        }
        a[0] += x * (vnext ? vnext[n - 1] : x);
    }
    block_partials<1>(a, part, gridDim.x, blockIdx.x);
}

void launch_fg_mgs(hipStream_t st, double* w, const double* vprev, const double* hprev, const double* vnext,
                   size_t n, double* part, unsigned* np) {
    const unsigned nb = red_blocks(n / 2 + 1);
    hipLaunchKernelGGL(k_fg_mgs, dim3(nb), dim3(kBlock), 0, st, w, vprev, hprev, vnext, (unsigned)n, part);
    *np = nb;
}

// ---- classical Gram-Schmidt passes of the flexible GMRES --------------------------------
// Dots of w with the NV basis vectors V0 + v * stride (block partials, value v at part[v * nb]),
// and w.w after them with WN. A set gate that reads 0 turns the launch into a no-op.
// A basis vector's 16-byte load; NT marks it streaming (non-temporal): a basis of
// 256^3 grid vectors is read once per pass and is far larger than the caches, and
// keeping it out of them leaves the last-level cache to the vectors that are reused
// (measured: the block solve 35.8 -> 35.2 ms, bitwise the same results).
typedef double FgD2 __attribute__((ext_vector_type(2)));
template <bool NT>
__device__ __forceinline__ double2 fg_basis_load(const double* base, unsigned p) {
    const FgD2* q = reinterpret_cast<const FgD2*>(base) + p;
    FgD2 v;
    if (NT) v = __builtin_nontemporal_load(q);
    else v = *q;
    return double2{v.x, v.y};
}

template <int NV, bool WN, bool NT>
__global__ void __launch_bounds__(kBlock) k_fg_mdot(const double* __restrict__ w, const double* __restrict__ V0,
                                                    size_t stride, unsigned n, double* part, const int* gate) {
    if (gate && !*gate) return;
    constexpr int K = NV + (WN ? 1 : 0);
    const unsigned n2 = n >> 1;
    unsigned lo, hi;
    chunk_of(blockIdx.x, gridDim.x, n2, &lo, &hi);
    double a[K];
#pragma unroll
    for (int k = 0; k < K; ++k) a[k] = 0.0;
    const double2* w2 = reinterpret_cast<const double2*>(w);
    for (unsigned p = lo + threadIdx.x; p < hi; p += blockDim.x) {
        const double2 x = w2[p];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double2 y = fg_basis_load<NT>(V0 + (size_t)v * stride, p);
            a[v] += x.x * y.x + x.y * y.y;
        }
        if (WN) a[K - 1] += x.x * x.x + x.y * x.y;
    }
    if ((n & 1u) && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const double x = w[n - 1];
#pragma unroll
        for (int v = 0; v < NV; ++v) a[v] += x * V0[(size_t)v * stride + n - 1];
        if (WN) a[K - 1] += x * x;
    }
    block_partials<K>(a, part, gridDim.x, blockIdx.x);
}

// out[v] the sum of value v's partials, v < K (v < K - 1 with wn, which takes the last value's).
template <int K>
__global__ void __launch_bounds__(kFinBlock) k_fg_mfin(const double* __restrict__ part, unsigned np, double* out,
                                                      double* wn, const int* gate) {
    if (gate && !*gate) return;
    double t[K];
    fin_sums<K>(part, np, t);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int v = 0; v < K; ++v) {
            if (wn && v == K - 1) *wn = t[v];
            else out[v] = t[v];
        }
    }
}

// w -= sum_v h[v] v_v over the m basis vectors (in order), partials of the new w.w.
template <bool NT>
__global__ void __launch_bounds__(kBlock) k_fg_mupdate(double* __restrict__ w, const double* __restrict__ V0,
                                                       size_t stride, unsigned n, const double* __restrict__ h,
                                                       int m, double* part, const int* gate) {
    if (gate && !*gate) return;
    __shared__ double hs[kFgMaxRestart];
    for (int k = threadIdx.x; k < m; k += blockDim.x) hs[k] = h[k];
    __syncthreads();
    const unsigned n2 = n >> 1;
    unsigned lo, hi;
    chunk_of(blockIdx.x, gridDim.x, n2, &lo, &hi);
    double a[1] = {0.0};
    double2* w2 = reinterpret_cast<double2*>(w);
    for (unsigned p = lo + threadIdx.x; p < hi; p += blockDim.x) {
        double2 x = w2[p];
        for (int v = 0; v < m; ++v) {
            const double2 y = fg_basis_load<NT>(V0 + (size_t)v * stride, p);
            x.x -= hs[v] * y.x;
            x.y -= hs[v] * y.y;
        }
        w2[p] = x;
        a[0] += x.x * x.x + x.y * x.y;
    }
    if ((n & 1u) && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        double x = w[n - 1];
        for (int v = 0; v < m; ++v) x -= hs[v] * V0[(size_t)v * stride + n - 1];
        w[n - 1] = x;
        a[0] += x * x;
    }
    block_partials<1>(a, part, gridDim.x, blockIdx.x);
}

// *hout = |w| from the update's partials. First pass (add == null): *redo = 1 when |w|^2 fell
// below eta2 * *pre2 (w lost most of its length to the projection, so the rounding left in
// it is relatively large). Second pass (gated by redo): col[v] += add[v], v < m.
__global__ void __launch_bounds__(kFinBlock) k_fg_norm(const double* __restrict__ part, unsigned np, double* hout,
                                                      const double* pre2, double eta2, int* redo, double* col,
                                                      const double* add, int m, const int* gate) {
    if (gate && !*gate) return;
    const double s = fin_sum(part, np);
    if (threadIdx.x == 0) {
        *hout = sqrt(s);
        if (!add) *redo = s < eta2 * *pre2 ? 1 : 0;
    }
    if (add)
        for (int v = threadIdx.x; v < m; v += blockDim.x) col[v] += add[v];
}

namespace {
template <int NV>
void mdot_launch(hipStream_t st, bool wn, unsigned nb, const double* w, const double* V0, size_t stride, unsigned n,
                 double* part, const int* gate) {
    if (wn) hipLaunchKernelGGL((k_fg_mdot<NV, true, true>), dim3(nb), dim3(kBlock), 0, st, w, V0, stride, n, part, gate);
    else hipLaunchKernelGGL((k_fg_mdot<NV, false, true>), dim3(nb), dim3(kBlock), 0, st, w, V0, stride, n, part, gate);
}
template <int K = 1>
void mfin_launch(hipStream_t st, int k, const double* part, unsigned np, double* out, double* wn, const int* gate) {
    if constexpr (K < 9) {
        if (k > K) return mfin_launch<K + 1>(st, k, part, np, out, wn, gate);
    }
    hipLaunchKernelGGL(k_fg_mfin<K>, dim3(1), dim3(kFinBlock), 0, st, part, np, out, wn, gate);
}
}  // namespace

unsigned fg_cgs_blocks(size_t n) { return red_blocks(n / 2 + 1); }

void launch_fg_cgs_dots(hipStream_t st, const double* w, const double* V, size_t stride, size_t n, int m, int group,
                        double* out, double* wn2, double* part, const int* gate) {
    const unsigned nb = fg_cgs_blocks(n);
    for (int g0 = 0; g0 < m; g0 += group) {
        const int nv = m - g0 < group ? m - g0 : group;
        const bool wn = g0 == 0 && wn2;
        const double* V0 = V + (size_t)g0 * stride;
        switch (nv) {
            case 1: mdot_launch<1>(st, wn, nb, w, V0, stride, (unsigned)n, part, gate); break;
            case 2: mdot_launch<2>(st, wn, nb, w, V0, stride, (unsigned)n, part, gate); break;
            case 3: mdot_launch<3>(st, wn, nb, w, V0, stride, (unsigned)n, part, gate); break;
            case 4: mdot_launch<4>(st, wn, nb, w, V0, stride, (unsigned)n, part, gate); break;
            case 5: mdot_launch<5>(st, wn, nb, w, V0, stride, (unsigned)n, part, gate); break;
            case 6: mdot_launch<6>(st, wn, nb, w, V0, stride, (unsigned)n, part, gate); break;
            case 7: mdot_launch<7>(st, wn, nb, w, V0, stride, (unsigned)n, part, gate); break;
            default: mdot_launch<8>(st, wn, nb, w, V0, stride, (unsigned)n, part, gate); break;
        }
        mfin_launch(st, nv + (wn ? 1 : 0), part, nb, out + g0, wn ? wn2 : nullptr, gate);
    }
}

void launch_fg_cgs_update(hipStream_t st, double* w, const double* V, size_t stride, size_t n, const double* h, int m,
                          double* part, const int* gate, double* hout, const double* pre2, double eta2, int* redo,
                          double* col, const double* add) {
    const unsigned nb = fg_cgs_blocks(n);
    hipLaunchKernelGGL(k_fg_mupdate<true>, dim3(nb), dim3(kBlock), 0, st, w, V, stride, (unsigned)n, h, m, part, gate);
    hipLaunchKernelGGL(k_fg_norm, dim3(1), dim3(kFinBlock), 0, st, part, nb, hout, pre2, eta2, redo, col, add, m,
                       gate);
}

// out = sum of the partials (its square root with take_sqrt)
__global__ void __launch_bounds__(kFinBlock) k_fg_fin(const double* __restrict__ part, unsigned np, double* out,
                                                      int take_sqrt) {
    const double s = fin_sum(part, np);
    if (threadIdx.x == 0) *out = take_sqrt ? sqrt(s) : s;
}

void launch_fg_fin(hipStream_t st, const double* part, unsigned np, double* out, int take_sqrt) {
    hipLaunchKernelGGL(k_fg_fin, dim3(1), dim3(kFinBlock), 0, st, part, np, out, take_sqrt);
}

// w /= *h (w = 0 when *h is 0: an exact breakdown)
__global__ void __launch_bounds__(kBlock) k_fg_scale(double* __restrict__ w, const double* __restrict__ h,
                                                     unsigned n) {
    const double hv = *h;
    const double inv = hv > 0.0 ? 1.0 / hv : 0.0;
    const unsigned p = blockIdx.x * blockDim.x + threadIdx.x;
    if (2 * p + 1 < n) {
        double2 x = reinterpret_cast<double2*>(w)[p];
        x.x *= inv;
        x.y *= inv;
        reinterpret_cast<double2*>(w)[p] = x;
    } else if (2 * p < n) {
        w[2 * p] *= inv;
    }
}

void launch_fg_scale(hipStream_t st, double* w, const double* h, size_t n) {
    hipLaunchKernelGGL(k_fg_scale, dim3(nblocks((n + 1) / 2)), dim3(kBlock), 0, st, w, h, (unsigned)n);
}

// w *= 1 / *h over the n entries, and block partial sums of the scaled grid part (the
// first ncell entries) into part[block], as k_norm_partials' first component: the sum the
// preconditioner's mean step reads next, without its own pass over w.
__global__ void __launch_bounds__(kBlock) k_fg_scale_sum(double* __restrict__ w, const double* __restrict__ h,
                                                         unsigned n, unsigned ncell, double* part) {
    const double hv = *h;
    const double inv = hv > 0.0 ? 1.0 / hv : 0.0;
    unsigned lo, hi;
    chunk_of(blockIdx.x, gridDim.x, n, &lo, &hi);
    double a[1] = {0.0};
    for (unsigned idx = lo + threadIdx.x; idx < hi; idx += blockDim.x) {
        const double v = w[idx] * inv;
        w[idx] = v;
        if (idx < ncell) a[0] += v;
    }
    block_partials<1>(a, part, gridDim.x, blockIdx.x);
}

void launch_fg_scale_sum(hipStream_t st, double* w, const double* h, size_t n, size_t ncell, double* part,
                         unsigned* np) {
    const unsigned nb = red_blocks(n);
    hipLaunchKernelGGL(k_fg_scale_sum, dim3(nb), dim3(kBlock), 0, st, w, h, (unsigned)n, (unsigned)ncell, part);
    *np = nb;
}

// r = b - r (sub) or r = b, with b = [bg; 0]; partials of r.r
__global__ void __launch_bounds__(kBlock) k_fg_resid(double* __restrict__ r, const double* __restrict__ bg,
                                                     unsigned ncell, unsigned n, int sub, double* part, double phi) {
    unsigned lo, hi;
    chunk_of(blockIdx.x, gridDim.x, n, &lo, &hi);
    double a[1] = {0.0};
    for (unsigned i = lo + threadIdx.x; i < hi; i += blockDim.x) {
        const double b = i < ncell ? bg[i] : phi;
        const double v = sub ? b - r[i] : b;
        r[i] = v;
        a[0] += v * v;
    }
    block_partials<1>(a, part, gridDim.x, blockIdx.x);
}

void launch_fg_resid(hipStream_t st, double* r, const double* bg, size_t ncell, size_t n, int sub, double* part,
                     unsigned* np, double phi) {
    const unsigned nb = red_blocks(n);
    hipLaunchKernelGGL(k_fg_resid, dim3(nb), dim3(kBlock), 0, st, r, bg, (unsigned)ncell, (unsigned)n, sub, part,
                       phi);
    *np = nb;
}

// x[i] += sum_j y_j Z_j[off + i] for i < n (Z_j = Z + j * stride, y on the device)
__global__ void __launch_bounds__(kBlock) k_fg_update(double* __restrict__ x, const double* __restrict__ Z,
                                                      size_t stride, size_t off, unsigned n, int k,
                                                      const double* __restrict__ y) {
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double acc = x[i];
    for (int j = 0; j < k; ++j) acc += y[j] * Z[(size_t)j * stride + off + i];
    x[i] = acc;
}

void launch_fg_update(hipStream_t st, double* x, const double* Z, size_t stride, size_t off, size_t n, int k,
                      const double* y) {
    if (n == 0 || k == 0) return;
    hipLaunchKernelGGL(k_fg_update, dim3(nblocks(n)), dim3(kBlock), 0, st, x, Z, stride, off, (unsigned)n, k, y);
}

// Column j of the Hessenberg matrix (column-major, leading dimension ld) is
// complete: apply the previous Givens rotations, form rotation j, advance the
// right-hand side g; out[0] = |g[j+1]| (the residual estimate), out[1] = the
// subdiagonal entry before rotation.
__global__ void __launch_bounds__(64) k_fg_givens(double* Hd, int ld, double* cs, double* sn, double* g, int j,
                                                  double* out) {
    // the chain runs over registers: entries and rotations are loaded by the wave, 64 at a time
    double* col = Hd + (size_t)j * ld;
    const int t = threadIdx.x;
    double a = col[0];
    for (int i0 = 0; i0 < j; i0 += 64) {
        const int i = i0 + t, n = min(64, j - i0);
        const double b_ = i < j ? col[i + 1] : 0.0, c_ = i < j ? cs[i] : 0.0, s_ = i < j ? sn[i] : 0.0;
        double mine = 0.0;
        for (int k = 0; k < n; ++k) {
            const double b = __shfl(b_, k, 64), c = __shfl(c_, k, 64), s = __shfl(s_, k, 64);
            const double r = c * a + s * b;
            if (t == k) mine = r;
            a = -s * a + c * b;
        }
        if (i < j) col[i] = mine;
    }
    if (t != 0) return;
    const double b = col[j + 1], gj = g[j];
    const double den = sqrt(a * a + b * b);
    const double c = den == 0.0 ? 1.0 : a / den, s = den == 0.0 ? 0.0 : b / den;
    cs[j] = c;
    sn[j] = s;
    out[1] = b;
    col[j] = den;
    col[j + 1] = 0.0;
    g[j + 1] = -s * gj;
    g[j] = c * gj;
    out[0] = fabs(-s * gj);
}

void launch_fg_givens(hipStream_t st, double* Hd, int ld, double* cs, double* sn, double* g, int j, double* out) {
    hipLaunchKernelGGL(k_fg_givens, dim3(1), dim3(64), 0, st, Hd, ld, cs, sn, g, j, out);
}

// g[0] = *beta, g[1..] = 0
__global__ void k_fg_gstart(double* g, int len, const double* beta) {
    for (int i = threadIdx.x; i < len; i += blockDim.x) g[i] = i == 0 ? *beta : 0.0;
}

void launch_fg_gstart(hipStream_t st, double* g, int len, const double* beta) {
    hipLaunchKernelGGL(k_fg_gstart, dim3(1), dim3(256), 0, st, g, len, beta);
}

// y = R^{-1} g for the leading k x k upper triangle R of the rotated Hessenberg matrix
__global__ void __launch_bounds__(kFgMaxRestart) k_fg_backsolve(const double* __restrict__ Hd, int ld,
                                                                const double* __restrict__ g, double* y, int k) {
    // by columns: once y_j is known every row above takes its share of it
    __shared__ double yj;
    const int t = threadIdx.x;
    double r = t < k ? g[t] : 0.0;
    for (int j = k - 1; j >= 0; --j) {
        const double h = t <= j ? Hd[(size_t)j * ld + t] : 0.0;
        if (t == j) {
            yj = h != 0.0 ? r / h : 0.0;
            y[j] = yj;
        }
        lds_barrier();
        if (t < j) r -= h * yj;
        lds_barrier();
    }
}

void launch_fg_backsolve(hipStream_t st, const double* Hd, int ld, const double* g, double* y, int k) {
    hipLaunchKernelGGL(k_fg_backsolve, dim3(1), dim3(k > 0 ? (k + 63) / 64 * 64 : 64), 0, st, Hd, ld, g, y,
                       k);
}

}  // namespace brd
