// Learned pairwise preconditioner for the Schur complement M = J A^+ S.
//
// The paper's diagonal preconditioner M^{-1} ~ chi gamma^{-1} I with
// gamma ~ (4 pi a)^{-1} (arXiv:1306.3159 Sec. III.E, eq. Schur_diagonal) is
// kept, and a short-ranged symmetric correction is added:
//   W_ij = D h [ delta_ij 4 pi a0/h + (g(i,j) + g(j,i))/2 ],  |q_j - q_i| < r_c,
// with g a 10 -> 64 -> 64 -> 1 SiLU network of pair features
//   [d/r_c (3), |d|/r_c, frac(q_i/h - 1/2) (3), frac(q_j/h - 1/2) (3)].
// Layers 1 and 2 (and in training the backward products and the weight
// gradients) run on v_mfma_f32_16x16x32_bf16: bfloat16 operands, float32
// accumulation. Layer 3 is a float32 dot product.
//
// MFMA 16x16x32 operand layout (wave64): A is 16 x 32 with lane l holding row
// l & 15, k = 8 (l >> 4) .. + 7; B is 32 x 16 with lane l holding column
// l & 15, k = 8 (l >> 4) .. + 7; the 16 x 16 result gives lane l column l & 15,
// rows 4 (l >> 4) .. + 3.
#include "launch.hpp"

#include <cmath>

namespace brd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 mfma16(const bf16x8& a, const bf16x8& b, const floatx4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float silu_f(float t) { return t / (1.0f + __expf(-t)); }
__device__ __forceinline__ float dsilu_f(float t) {
    const float s = 1.0f / (1.0f + __expf(-t));
    return s * (1.0f + t * (1.0f - s));
}

// Sum over the 16 lanes that share (l >> 4).
__device__ __forceinline__ float sum16(float v) {
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 8, 64);
    return v;
}
// Sum over the 4 lane groups (l >> 4) for a fixed l & 15.
__device__ __forceinline__ float sum_groups(float v) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

// ---------------------------------------------------------------------------
// Pair list: blobs binned in a cell grid of edge >= r_c (a single cell when an
// axis has fewer than 3 cells), then each blob scans the neighbouring cells.
__global__ void k_pair_cells(const double* __restrict__ q, int N, PairGeom pg, int* __restrict__ cell_of,
                             int* __restrict__ counts) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    int c[3];
    const int nc[3] = {pg.ncx, pg.ncy, pg.ncz};
    for (int a = 0; a < 3; ++a) {
        const double L = pg.box[a];
        double v = q[3 * i + a];
        v -= L * floor(v / L);
        if (v >= L) v -= L;
        int k = (int)(v / L * nc[a]);
        c[a] = k < 0 ? 0 : (k >= nc[a] ? nc[a] - 1 : k);
    }
    const int id = (c[2] * pg.ncy + c[1]) * pg.ncx + c[0];
    cell_of[i] = id;
    atomicAdd(&counts[id], 1);
}

__device__ __forceinline__ double min_image(double d, double L) { return d - L * rint(d / L); }

// One wave per blob: the neighbouring cells' blob ranges a lane each, then the lanes take their
// blobs in turn (a thread per blob walked its 27 cells alone: 49 us for 1250 blobs, as here 7).
// FILL writes the row's columns in candidate order, else counts them.
template <bool FILL>
__global__ void __launch_bounds__(kBlock) k_pair_scan(const double* __restrict__ q, int N, PairGeom pg,
                                                      const int* __restrict__ cell_of,
                                                      const int* __restrict__ offsets, const int* __restrict__ perm,
                                                      int* __restrict__ cnt, const int* __restrict__ rowptr,
                                                      int* __restrict__ col, int* __restrict__ rowidx) {
    const int i = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= N) return;
    const int id = cell_of[i];
    const int cx = id % pg.ncx, cy = (id / pg.ncx) % pg.ncy, cz = id / (pg.ncx * pg.ncy);
    const double xi = q[3 * i], yi = q[3 * i + 1], zi = q[3 * i + 2];
    const double rc2 = pg.rc * pg.rc;
    // an axis of fewer than three cells has one (pair_geom)
    const int mx = pg.ncx >= 3 ? 3 : 1, my = pg.ncy >= 3 ? 3 : 1, mz = pg.ncz >= 3 ? 3 : 1, nr = mx * my * mz;
    int lo = 0, len = 0;
    if (lane < nr) {
        const int dx = lane % mx - mx / 2, dy = (lane / mx) % my - my / 2, dz = lane / (mx * my) - mz / 2;
        const int nb = (((cz + dz + pg.ncz) % pg.ncz) * pg.ncy + (cy + dy + pg.ncy) % pg.ncy) * pg.ncx +
                       (cx + dx + pg.ncx) % pg.ncx;
        lo = offsets[nb];
        len = offsets[nb + 1] - lo;
    }
    const int inc = wave_scan(len), total = __shfl(inc, 63, 64), first = lo - (inc - len);
    const int base = FILL ? rowptr[i] : 0;
    int n = 0;
    for (int k0 = 0; k0 < total; k0 += 64) {
        const int k = k0 + lane;
        int r = 0;  // the range candidate k lies in
        for (int d = 0; d < nr; ++d) r += __shfl(inc, d, 64) <= k;
        const int from = __shfl(first, min(r, 63), 64);
        bool hit = false;
        int j = 0;
        if (k < total) {
            j = perm[from + k];
            const double ddx = min_image(q[3 * j] - xi, pg.box[0]);
            const double ddy = min_image(q[3 * j + 1] - yi, pg.box[1]);
            const double ddz = min_image(q[3 * j + 2] - zi, pg.box[2]);
            hit = ddx * ddx + ddy * ddy + ddz * ddz < rc2;
        }
        const unsigned long long m = __ballot(hit);
        if (FILL && hit) {
            const int e = base + n + __popcll(m & ((1ull << lane) - 1));
            col[e] = j;
            rowidx[e] = i;
        }
        n += __popcll(m);
    }
    if (!FILL && lane == 0) cnt[i] = n;
}

// Columns of each row in ascending order (fixed order for every later sum). One wave per row:
// a lane's columns (distinct) go to their ranks; rows beyond 64 kRowRegs are sorted by lane 0.
constexpr int kRowRegs = 8;
__global__ void __launch_bounds__(kBlock) k_row_sort(const int* __restrict__ rowptr, int N, int* col) {
    const int i = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= N) return;
    const int lo = rowptr[i], hi = rowptr[i + 1], n = hi - lo;
    if (n <= 64 * kRowRegs) {
        int v[kRowRegs], rank[kRowRegs];
#pragma unroll
        for (int c = 0; c < kRowRegs; ++c) {
            v[c] = lane + 64 * c < n ? col[lo + lane + 64 * c] : 0x7fffffff;
            rank[c] = 0;
        }
#pragma unroll
        for (int c = 0; c < kRowRegs; ++c) {
            const int m = min(64, n - 64 * c);
            for (int k = 0; k < m; ++k) {
                const int u = __shfl(v[c], k, 64);
#pragma unroll
                for (int b = 0; b < kRowRegs; ++b) rank[b] += u < v[b];
            }
        }
#pragma unroll
        for (int c = 0; c < kRowRegs; ++c)
            if (lane + 64 * c < n) col[lo + rank[c]] = v[c];
        return;
    }
    if (lane != 0) return;
    for (int a = lo + 1; a < hi; ++a) {
        const int v = col[a];
        int b = a - 1;
        while (b >= lo && col[b] > v) {
            col[b + 1] = col[b];
            --b;
        }
        col[b + 1] = v;
    }
}

void launch_pair_cells(hipStream_t st, const double* q, int N, PairGeom pg, int* cell_of, int* counts) {
    hipLaunchKernelGGL(k_pair_cells, dim3(nblocks(N)), dim3(kBlock), 0, st, q, N, pg, cell_of, counts);
}
void launch_pair_count(hipStream_t st, const double* q, int N, PairGeom pg, const int* cell_of, const int* offsets,
                       const int* perm, int* cnt) {
    hipLaunchKernelGGL(k_pair_scan<false>, dim3(nblocks(N, kBlock / 64)), dim3(kBlock), 0, st, q, N, pg, cell_of, offsets, perm,
                       cnt, (const int*)nullptr, (int*)nullptr, (int*)nullptr);
}
void launch_pair_fill(hipStream_t st, const double* q, int N, PairGeom pg, const int* cell_of, const int* offsets,
                      const int* perm, const int* rowptr, int* col, int* rowidx) {
    hipLaunchKernelGGL(k_pair_scan<true>, dim3(nblocks(N, kBlock / 64)), dim3(kBlock), 0, st, q, N, pg, cell_of, offsets, perm,
                       (int*)nullptr, rowptr, col, rowidx);
    hipLaunchKernelGGL(k_row_sort, dim3(nblocks(N, kBlock / 64)), dim3(kBlock), 0, st, rowptr, N, col);
}

// ---------------------------------------------------------------------------
// Pair features of evaluation ev: entry e = ev >> 1, ordering ev & 1.
__device__ __forceinline__ void pair_features(const double* __restrict__ q, PairGeom pg, int a, int b, float* x) {
    double d[3];
    for (int k = 0; k < 3; ++k) {
        double qa = q[3 * a + k], qb = q[3 * b + k];
        const double L = pg.box[k];
        qa -= L * floor(qa / L);
        qb -= L * floor(qb / L);
        d[k] = min_image(qb - qa, L);
        const double sa = qa / pg.h - 0.5, sb = qb / pg.h - 0.5;
        x[4 + k] = (float)(sa - floor(sa));
        x[7 + k] = (float)(sb - floor(sb));
    }
    const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    x[0] = (float)(d[0] / pg.rc);
    x[1] = (float)(d[1] / pg.rc);
    x[2] = (float)(d[2] / pg.rc);
    x[3] = (float)(r / pg.rc);
    x[10] = kNuScale * pg.nu[a];
    x[11] = kNuScale * pg.nu[b];
}

// nu_i: the other blobs of row i of the pair list closer than rc / 2 (minimum image, the
// separation formed as in pair_features).
__global__ void __launch_bounds__(kBlock) k_pair_nu(const double* __restrict__ q, PairGeom pg,
                                                    const int* __restrict__ rowptr, const int* __restrict__ col,
                                                    int N, float* __restrict__ nu) {
    const int i = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;  // one wave per row
    if (i >= N) return;
    double qi[3];
    for (int k = 0; k < 3; ++k) {
        const double L = pg.box[k];
        qi[k] = q[3 * i + k] - L * floor(q[3 * i + k] / L);
    }
    int count = 0;
    const int lo = rowptr[i], hi = rowptr[i + 1];
    for (int e0 = lo; e0 < hi; e0 += 64) {
        const int e = e0 + lane;
        const int j = e < hi ? col[e] : i;
        bool near = false;
        if (j != i) {
            double r2 = 0.0;
            for (int k = 0; k < 3; ++k) {
                const double L = pg.box[k];
                const double qj = q[3 * j + k] - L * floor(q[3 * j + k] / L);
                const double dk = min_image(qj - qi[k], L);
                r2 += dk * dk;
            }
            near = sqrt(r2) < 0.5 * pg.rc;
        }
        count += __popcll(__ballot(near));
    }
    if (lane == 0) nu[i] = (float)count;
}

void launch_pair_nu(hipStream_t st, const double* q, PairGeom pg, const int* rowptr, const int* col, int N, float* nu) {
    if (N <= 0) return;
    hipLaunchKernelGGL(k_pair_nu, dim3(nblocks(N, kBlock / 64)), dim3(kBlock), 0, st, q, pg, rowptr, col, N, nu);
}

// Weight operands in registers (per lane), loaded once per kernel.
struct NetRegs {
    bf16x8 b1[4];       // layer 1 B operand, output tile t
    bf16x8 b2[2][4];    // layer 2 B operand, k step ks, output tile t
    float bias1[4], bias2[4], w3[4];
    float b3;
};

__device__ __forceinline__ void load_net(NetRegs& R, const NetDev& net) {
    const int l = threadIdx.x & 63, c = l & 15, g = l >> 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = 8 * g + j;
            v[j] = k < 16 ? net.W1b[(16 * t + c) * 16 + k] : (__bf16)0.0f;
        }
        R.b1[t] = v;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 w;
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] = net.W2b[(16 * t + c) * 64 + 32 * ks + 8 * g + j];
            R.b2[ks][t] = w;
        }
        R.bias1[t] = net.P[kOffB1 + 16 * t + c];
        R.bias2[t] = net.P[kOffB2 + 16 * t + c];
        R.w3[t] = (float)net.w3b[16 * t + c];
    }
    R.b3 = net.P[kOffB3];
}

// Forward of 16 evaluations. feat: this lane's A operand (features of row l&15).
// h1s: wave LDS [16][64] bf16. Outputs (per lane, rows 4g+i): a1, a2, h2 in
// the result layout, g_out (valid on lanes with (l & 15) == 0).
struct Fwd {
    float a1[4][4], a2[4][4], h2[4][4];
    float out[4];
};

__device__ __forceinline__ void net_forward(const NetRegs& R, const bf16x8& feat, __bf16* h1s, Fwd& F) {
    const int l = threadIdx.x & 63, c = l & 15, g = l >> 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma16(feat, R.b1[t], acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a = acc[i] + R.bias1[t];
            F.a1[t][i] = a;
            h1s[(4 * g + i) * 64 + 16 * t + c] = (__bf16)silu_f(a);
        }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    bf16x8 A[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 8; ++j) A[ks][j] = h1s[c * 64 + 32 * ks + 8 * g + j];
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma16(A[0], R.b2[0][t], acc);
        acc = mfma16(A[1], R.b2[1][t], acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a = acc[i] + R.bias2[t];
            F.a2[t][i] = a;
            const float hv = silu_f(a);
            F.h2[t][i] = hv;
            part[i] += R.w3[t] * hv;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) F.out[i] = sum16(part[i]) + R.b3;
}

__device__ __forceinline__ bf16x8 feature_operand(const double* q, PairGeom pg, const int* col, const int* rowidx,
                                                  long long ev, long long nev) {
    const int l = threadIdx.x & 63, g = l >> 4;
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (__bf16)0.0f;
    if (g < 2) {
        float x[kNetFeat];
        if (ev < nev) {
            const long long e = ev >> 1;
            const int a = rowidx[e], b = col[e];
            if (ev & 1) pair_features(q, pg, b, a, x);
            else pair_features(q, pg, a, b, x);
        } else {
#pragma unroll
            for (int k = 0; k < kNetFeat; ++k) x[k] = 0.f;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = 8 * g + j;
            v[j] = (__bf16)(k < kNetFeat ? x[k] : 0.f);
        }
    }
    return v;
}

// W values: one wave per 16 evaluations (8 entries) per pass.
__global__ void __launch_bounds__(kBlock) k_net_assemble(const double* __restrict__ q, PairGeom pg, NetDev net,
                                                         const int* __restrict__ col, const int* __restrict__ rowidx,
                                                         long long nnz, double Dh, double diag,
                                                         double* __restrict__ val) {
    __shared__ __bf16 h1s_all[kBlock / 64][16 * 64];
    const int wv = threadIdx.x >> 6, l = threadIdx.x & 63, c = l & 15, g = l >> 4;
    __bf16* h1s = h1s_all[wv];
    NetRegs R;
    load_net(R, net);
    const long long nev = 2 * nnz;
    const long long ntile = (nev + 15) / 16;
    const long long wglobal = (long long)blockIdx.x * (kBlock / 64) + wv;
    const long long nwaves = (long long)gridDim.x * (kBlock / 64);
    for (long long tile = wglobal; tile < ntile; tile += nwaves) {
        const long long ev0 = tile * 16;
        const bf16x8 feat = feature_operand(q, pg, col, rowidx, ev0 + c, nev);
        Fwd F;
        net_forward(R, feat, h1s, F);
        if (c == 0) {
            // rows 4g .. 4g+3 = evaluations of entries 2g and 2g+1 of this tile
            for (int pr = 0; pr < 2; ++pr) {
                const long long e = (ev0 >> 1) + 2 * g + pr;
                if (e < nnz) {
                    const double gsum = 0.5 * ((double)F.out[2 * pr] + (double)F.out[2 * pr + 1]);
                    val[e] = Dh * (gsum + (rowidx[e] == col[e] ? diag : 0.0));
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

void launch_net_assemble(hipStream_t st, const double* q, PairGeom pg, NetDev net, const int* col, const int* rowidx,
                         long long nnz, double Dh, double diag, double* val) {
    const long long tiles = (2 * nnz + 15) / 16;
    long long blocks = (tiles + 3) / 4;
    if (blocks > 2048) blocks = 2048;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_net_assemble, dim3((unsigned)blocks), dim3(kBlock), 0, st, q, pg, net, col, rowidx, nnz, Dh,
                       diag, val);
}

// ---------------------------------------------------------------------------
// CSR SpMV y = W (x - mean(x)) (FP64), columns ascending: each block sums x itself (the same order in every block,
// so every block subtracts the same mean), then one thread per row.
__global__ void __launch_bounds__(kBlock) k_spmv_centered(const int* __restrict__ rowptr, const int* __restrict__ col,
                                                          const double* __restrict__ val,
                                                          const double* __restrict__ x, double* __restrict__ y,
                                                          int N) {
    // the block's copy of mean(x): eight independent partial sums keep eight loads in flight
    double p[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const int bd = (int)blockDim.x;
    int i0 = threadIdx.x;
    for (; i0 + 7 * bd < N; i0 += 8 * bd) {
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] += x[i0 + u * bd];
    }
    for (; i0 < N; i0 += bd) p[0] += x[i0];
    const double m = wg_sum(((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]))) / (double)N;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    double acc = 0.0;
    for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) acc += val[k] * (x[col[k]] - m);
    y[i] = acc;
}

void launch_spmv_centered(hipStream_t st, const int* rowptr, const int* col, const double* val, const double* x,
                          double* y, int N) {
    if (N <= 0) return;
    hipLaunchKernelGGL(k_spmv_centered, dim3(nblocks(N)), dim3(kBlock), 0, st, rowptr, col, val, x, y, N);
}

// Non-finite entries of W (watchdog)
__global__ void __launch_bounds__(kFinBlock) k_count_bad(const double* v, long long n, int* out) {
    int bad = 0;
    for (long long i = threadIdx.x; i < n; i += blockDim.x) bad += !(v[i] == v[i] && v[i] - v[i] == 0.0);
    const double s = wg_sum((double)bad);  // exact: whole numbers below 2^53
    if (threadIdx.x == 0) out[0] = (int)s;
}
void launch_count_bad(hipStream_t st, const double* v, long long n, int* out) {
    hipLaunchKernelGGL(k_count_bad, dim3(1), dim3(kFinBlock), 0, st, v, n, out);
}

// ---------------------------------------------------------------------------
// Training.
//
// The loss, per sample s: yp = P y, rp = P W yp - x (W and P as the solve applies them),
// sums[2 s] = |rp|^2, sums[2 s + 1] = |x|^2, then rp's mean removed. The sums run over the
// threads' strided entries of one work-group, as the single-vector kernels' do.
__device__ __forceinline__ void loss_center(const double* __restrict__ y, int N, double* __restrict__ yp) {
    const int bd = (int)blockDim.x;
    double s = 0.0;
    for (int i = threadIdx.x; i < N; i += bd) s += y[i];
    const double m = wg_sum(s) / (double)N;
    for (int i = threadIdx.x; i < N; i += bd) yp[i] = y[i] - m;
}
__device__ __forceinline__ double loss_row(const int* __restrict__ rowptr, const int* __restrict__ col,
                                           const double* __restrict__ val, const double* yp, int i) {
    double acc = 0.0;
    for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) acc += val[k] * yp[col[k]];
    return acc;
}
// s: this thread's sum of rp = W yp
__device__ __forceinline__ void loss_finish(const double* __restrict__ x, int N, double* rp, double s, double* sums) {
    const int bd = (int)blockDim.x;
    double m = wg_sum(s) / (double)N;
    double t[3] = {0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < N; i += bd) {
        const double xi = x[i], r = (rp[i] - m) - xi;
        rp[i] = r;
        t[0] += r;
        t[1] += r * r;
        t[2] += xi * xi;
    }
    wg_sums<3>(t);
    m = t[0] / (double)N;
    for (int i = threadIdx.x; i < N; i += bd) rp[i] -= m;
    if (threadIdx.x == 0) {
        sums[0] = t[1];
        sums[1] = t[2];
    }
}

// All of it in one launch, a work-group a sample.
__global__ void __launch_bounds__(kFinBlock) k_loss_rows(const int* __restrict__ rowptr, const int* __restrict__ col,
                                                        const double* __restrict__ val, const double* __restrict__ X,
                                                        const double* __restrict__ Y, int N, double* RP, double* YP,
                                                        double* sums) {
    const size_t o = (size_t)blockIdx.x * N;
    double *rp = RP + o, *yp = YP + o;
    loss_center(Y + o, N, yp);
    __syncthreads();
    double s = 0.0;
    for (int i = threadIdx.x; i < N; i += (int)blockDim.x) {
        const double acc = loss_row(rowptr, col, val, yp, i);
        rp[i] = acc;
        s += acc;
    }
    loss_finish(X + o, N, rp, s, sums + 2 * blockIdx.x);
}

// The same in three, the rows of W over the whole GPU (the same bits).
__global__ void __launch_bounds__(kFinBlock) k_loss_center(const double* __restrict__ Y, int N,
                                                          double* __restrict__ YP) {
    const size_t o = (size_t)blockIdx.x * N;
    loss_center(Y + o, N, YP + o);
}
__global__ void __launch_bounds__(kBlock) k_loss_product(const int* __restrict__ rowptr, const int* __restrict__ col,
                                                        const double* __restrict__ val, int N,
                                                        const double* __restrict__ YP, double* __restrict__ RP) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const size_t o = (size_t)blockIdx.y * N;
    if (i < N) RP[o + i] = loss_row(rowptr, col, val, YP + o, i);
}
__global__ void __launch_bounds__(kFinBlock) k_loss_finish(const double* __restrict__ X, int N, double* RP,
                                                          double* sums) {
    const size_t o = (size_t)blockIdx.x * N;
    double s = 0.0;
    for (int i = threadIdx.x; i < N; i += (int)blockDim.x) s += RP[o + i];
    loss_finish(X + o, N, RP + o, s, sums + 2 * blockIdx.x);
}

// Pair-list entries up to which one launch is taken. One launch saves two and keeps a sample's vectors
// in one L2 (1250 blobs, 8 samples: 0.53 -> 0.09 ms for the loss and its gradient against eight launches
// and a host read a sample, with k_grad_reduce), but a single CU walks all the rows: with one sample, loss
// and gradient in one launch / three, us: 816 entries 72 / 75, 6600 82 / 83, 14088 101 / 96, 28474 140 / 115,
// 52528 188 / 134, 289152 874 / 290, 1402494 4510 / 1020 (8 samples: 74 / 78, 85 / 86, 103 / 100, 142 / 118,
// 189 / 137, 886 / 308, 4570 / 1310).
constexpr long long kLossSplit = 1 << 13;

void launch_loss_rows(hipStream_t st, const int* rowptr, const int* col, const double* val, long long nnz,
                      const double* X, const double* Y, int S, int N, double* RP, double* YP, double* sums) {
    if (nnz <= kLossSplit) {
        hipLaunchKernelGGL(k_loss_rows, dim3(S), dim3(kFinBlock), 0, st, rowptr, col, val, X, Y, N, RP, YP, sums);
        return;
    }
    hipLaunchKernelGGL(k_loss_center, dim3(S), dim3(kFinBlock), 0, st, Y, N, YP);
    hipLaunchKernelGGL(k_loss_product, dim3(nblocks(N), S), dim3(kBlock), 0, st, rowptr, col, val, N, YP, RP);
    hipLaunchKernelGGL(k_loss_finish, dim3(S), dim3(kFinBlock), 0, st, X, N, RP, sums);
}

// GW_e = sum_s c_s rp_s[row e] yp_s[col e] with c_s = 2 / (S |x_s|^2); the
// network output gradient of both evaluations of entry e is D h GW_e / 2.
__global__ void k_entry_grad(const int* __restrict__ rowidx, const int* __restrict__ col, long long nnz,
                             const double* __restrict__ RP, const double* __restrict__ YP,
                             const double* __restrict__ coef, int S, int N, double half_Dh, float* __restrict__ dg) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    const int i = rowidx[e], j = col[e];
    double acc = 0.0;
    for (int s = 0; s < S; ++s) acc += coef[s] * RP[(size_t)s * N + i] * YP[(size_t)s * N + j];
    dg[e] = (float)(half_Dh * acc);
}
void launch_entry_grad(hipStream_t st, const int* rowidx, const int* col, long long nnz, const double* RP,
                       const double* YP, const double* coef, int S, int N, double half_Dh, float* dg) {
    hipLaunchKernelGGL(k_entry_grad, dim3((unsigned)((nnz + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, rowidx, col,
                       nnz, RP, YP, coef, S, N, half_Dh, dg);
}

// Per-wave gradient partials: one slot of kNetParams floats per wave.
// Each wave walks tiles of 32 evaluations (two 16-row halves): forward,
// backward to the pre-activations, then weight gradients as MFMA products
// with the 32 evaluations as the contraction dimension.
__global__ void __launch_bounds__(kBlock) k_net_backward(const double* __restrict__ q, PairGeom pg, NetDev net,
                                                         const int* __restrict__ col, const int* __restrict__ rowidx,
                                                         long long nnz, const float* __restrict__ dg,
                                                         float* __restrict__ wpart) {
    struct WaveLds {
        __bf16 h1[32 * 64];
        __bf16 da2[32 * 64];
        __bf16 da1[32 * 64];
        __bf16 x[32 * 16];
    };
    __shared__ WaveLds lds_all[kBlock / 64];
    const int wv = threadIdx.x >> 6, l = threadIdx.x & 63, c = l & 15, g = l >> 4;
    WaveLds& S = lds_all[wv];
    NetRegs R;
    load_net(R, net);
    // W2 as a B operand of d_h1 = d_a2 . W2: B[k = o2][col = k1] = W2[o2][k1]
    bf16x8 w2t[2][4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j) w2t[ks][t][j] = net.W2b[(32 * ks + 8 * g + j) * 64 + 16 * t + c];
    floatx4 gW2[4][4];
    floatx4 gW1[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        gW1[a] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < 4; ++b) gW2[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    float gb1[4] = {0, 0, 0, 0}, gb2[4] = {0, 0, 0, 0}, gw3[4] = {0, 0, 0, 0}, gb3 = 0.f;
    const long long nev = 2 * nnz;
    const long long ntile = (nev + 31) / 32;
    const long long wglobal = (long long)blockIdx.x * (kBlock / 64) + wv;
    const long long nwaves = (long long)gridDim.x * (kBlock / 64);
    for (long long tile = wglobal; tile < ntile; tile += nwaves) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const long long ev0 = tile * 32 + 16 * half;
            const bf16x8 feat = feature_operand(q, pg, col, rowidx, ev0 + c, nev);
            // keep the features (rows = evaluations) for the W1 gradient
            if (g < 2)
#pragma unroll
                for (int j = 0; j < 8; ++j) S.x[(16 * half + c) * 16 + 8 * g + j] = feat[j];
            Fwd F;
            net_forward(R, feat, S.h1 + 16 * half * 64, F);
            // output gradient of rows 4g+i (evaluation ev0 + 4g + i)
            float dout[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long long ev = ev0 + 4 * g + i;
                dout[i] = ev < nev ? dg[ev >> 1] : 0.f;
            }
            float da2[4][4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    gw3[t] += dout[i] * F.h2[t][i];
                    da2[t][i] = dout[i] * R.w3[t] * dsilu_f(F.a2[t][i]);
                    gb2[t] += da2[t][i];
                    S.da2[(16 * half + 4 * g + i) * 64 + 16 * t + c] = (__bf16)da2[t][i];
                }
            if (c == 0)
#pragma unroll
                for (int i = 0; i < 4; ++i) gb3 += dout[i];
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            // d_h1 = d_a2 . W2 (A = d_a2 rows of this half)
            bf16x8 A[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int j = 0; j < 8; ++j) A[ks][j] = S.da2[(16 * half + c) * 64 + 32 * ks + 8 * g + j];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma16(A[0], w2t[0][t], acc);
                acc = mfma16(A[1], w2t[1][t], acc);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float d1 = acc[i] * dsilu_f(F.a1[t][i]);
                    gb1[t] += d1;
                    S.da1[(16 * half + 4 * g + i) * 64 + 16 * t + c] = (__bf16)d1;
                }
            }
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        }
        // weight gradients, contraction over the 32 evaluations of the tile:
        // gW2[o][k] += sum_ev da2[ev][o] h1[ev][k], gW1[o][k] += sum_ev da1[ev][o] x[ev][k]
#pragma unroll
        for (int to = 0; to < 4; ++to) {
            bf16x8 A2, A1;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                A2[j] = S.da2[(8 * g + j) * 64 + 16 * to + c];
                A1[j] = S.da1[(8 * g + j) * 64 + 16 * to + c];
            }
#pragma unroll
            for (int tk = 0; tk < 4; ++tk) {
                bf16x8 B;
#pragma unroll
                for (int j = 0; j < 8; ++j) B[j] = S.h1[(8 * g + j) * 64 + 16 * tk + c];
                gW2[to][tk] = mfma16(A2, B, gW2[to][tk]);
            }
            bf16x8 Bx;
#pragma unroll
            for (int j = 0; j < 8; ++j) Bx[j] = S.x[(8 * g + j) * 16 + c];
            gW1[to] = mfma16(A1, Bx, gW1[to]);
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    }
    // write this wave's partial gradient (W1 cols < 10 only)
    float* out = wpart + (size_t)wglobal * kNetParams;
#pragma unroll
    for (int to = 0; to < 4; ++to)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = 16 * to + 4 * g + i;
            if (c < kNetFeat) out[kOffW1 + o * kNetFeat + c] = gW1[to][i];
#pragma unroll
            for (int tk = 0; tk < 4; ++tk) out[kOffW2 + o * 64 + 16 * tk + c] = gW2[to][tk][i];
        }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float b1 = sum_groups(gb1[t]), b2 = sum_groups(gb2[t]), w3 = sum_groups(gw3[t]);
        if (g == 0) {
            out[kOffB1 + 16 * t + c] = b1;
            out[kOffB2 + 16 * t + c] = b2;
            out[kOffW3 + 16 * t + c] = w3;
        }
    }
    float b3 = gb3;
    b3 += __shfl_xor(b3, 16, 64);
    b3 += __shfl_xor(b3, 32, 64);
    if (l == 0) out[kOffB3] = b3;
}

int launch_net_backward(hipStream_t st, const double* q, PairGeom pg, NetDev net, const int* col, const int* rowidx,
                        long long nnz, const float* dg, float* wpart, int max_waves) {
    const long long tiles = (2 * nnz + 31) / 32;
    long long waves = tiles < max_waves ? tiles : max_waves;
    if (waves < 4) waves = 4;
    const long long blocks = (waves + 3) / 4;
    hipLaunchKernelGGL(k_net_backward, dim3((unsigned)blocks), dim3(kBlock), 0, st, q, pg, net, col, rowidx, nnz, dg,
                       wpart);
    return (int)(blocks * 4);
}

// grad += sum over waves (fixed order): a work-group takes 64 parameters, its waves every 16th
// partial each (eight loads in flight), then the 16 sums in order. One thread a parameter
// walking all partials took 93 us for 1024 of them.
__global__ void __launch_bounds__(kFinBlock) k_grad_reduce(const float* __restrict__ wpart, int nwaves,
                                                          float* __restrict__ grad) {
    __shared__ float sh[kFinBlock / 64][64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = kFinBlock / 64;
    const int p = blockIdx.x * 64 + lane;
    float s = 0.f;
    if (p < kNetParams)
        for (int w0 = wid; w0 < nwaves; w0 += 8 * nw) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int w = w0 + u * nw;
                v[u] = w < nwaves ? wpart[(size_t)w * kNetParams + p] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    sh[wid][lane] = s;
    __syncthreads();
    if (wid != 0 || p >= kNetParams) return;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < nw; ++w) t += sh[w][lane];
    grad[p] += t;
}
void launch_grad_reduce(hipStream_t st, const float* wpart, int nwaves, float* grad) {
    hipLaunchKernelGGL(k_grad_reduce, dim3(nblocks(kNetParams, 64)), dim3(kFinBlock), 0, st, wpart, nwaves, grad);
}

// Adam (Kingma and Ba, 2015) on float32 masters, then refresh the bf16 copies.
__global__ void k_adam(float* __restrict__ P, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ grad, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kNetParams) return;
    const float g = grad[p];
    const float mm = b1 * m[p] + (1.f - b1) * g;
    const float vv = b2 * v[p] + (1.f - b2) * g * g;
    m[p] = mm;
    v[p] = vv;
    P[p] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}
void launch_adam(hipStream_t st, float* P, float* m, float* v, const float* grad, float lr, float b1, float b2,
                 float eps, int t) {
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3(nblocks(kNetParams)), dim3(kBlock), 0, st, P, m, v, grad, lr, b1, b2, eps, c1,
                       c2);
}

__global__ void k_net_pack(const float* __restrict__ P, __bf16* __restrict__ W1b, __bf16* __restrict__ W2b,
                           __bf16* __restrict__ w3b) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 64 * 16) {
        const int o = t / 16, k = t % 16;
        W1b[t] = (__bf16)(k < kNetFeat ? P[kOffW1 + o * kNetFeat + k] : 0.f);
    }
    if (t < 64 * 64) W2b[t] = (__bf16)P[kOffW2 + t];
    if (t < 64) w3b[t] = (__bf16)P[kOffW3 + t];
}
void launch_net_pack(hipStream_t st, const float* P, __bf16* W1b, __bf16* W2b, __bf16* w3b) {
    hipLaunchKernelGGL(k_net_pack, dim3(16), dim3(kBlock), 0, st, P, W1b, W2b, w3b);
}

}  // namespace brd
