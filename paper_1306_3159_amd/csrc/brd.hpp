// Internal declarations of the blob_rd HIP library (gfx950).
//
// Data layout in device memory:
//  * FP64 grid vectors (Krylov iterates, residuals, right-hand sides) are in
//    natural order [z][y][x], x fastest, as the public ABI exposes them.
//  * Multigrid levels are stored red/black split: level l with dims
//    (nx, ny, nz), nx even, keeps two arrays per field, one per colour
//    (colour = (x + y + z) mod 2, red = 0), each [z][y][nx/2]. Cell (x, y, z)
//    of colour c sits at index x/2 of row (y, z) of array c. A Gauss-Seidel
//    half-sweep then reads the other colour's array and writes its own with
//    unit stride. The coarsest level (<= 512 cells, possibly odd) is natural.
//  * Blob data are structure-of-arrays in original blob order plus a
//    permutation that sorts blobs by the grid tile of their base cell.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "cg_scalars.hpp"

namespace brd {

constexpr int kBlock = 256;
constexpr int kMaxTuneBlock = 512;  // largest work-group the autotuner may pick
constexpr int kFinBlock = 1024;
constexpr int kMaxLevels = 16;
constexpr int kMaxCoarse = 512;
constexpr int kTailPad = 8;          // values between the planes of the tail's split levels in LDS
constexpr int kTailDense = 64;       // coarsest cells up to which its inverse is applied as a dense matrix
constexpr int kMaxCoarseCols = 256;  // columns of the Schur preconditioner's Fourier coarse level
constexpr int kCoarseChunk = 2048;   // rows per work-group in the coarse level's dot products
constexpr int kStageBlobs = 128;   // candidate blobs staged in LDS per pass of the spread planner

// A reduction of CG that a vector pass finishes itself (np = 0: done before it): np partials a
// set at `in`; alpha's: the blob term's vectors Jp (na) and mu (nb) of length n.
struct CgFold {
    const double* in;
    unsigned np;
    const double *na, *nb;
    int n;
    double inv_h3;
};

// Device-resident scalars of the Schur GMRES (single work-group kernels).
struct GmresScalars {
    double beta;      // initial residual norm of the current cycle
    double res;       // current residual estimate |g_{k+1}|
    double hk1;       // last subdiagonal entry
    int32_t k;        // columns in the current cycle
    int32_t status;
};

// Longest restart of the flexible GMRES on the block saddle system.
constexpr int kFgMaxRestart = 1024;

// Levels handled by the single-work-group coarse tail (index 0 = first tail
// level, last = coarsest). LDS byte offsets: each level's work arrays, its result in
// natural order (levels 1 ..), the coarsest solve's FP64 vectors and its spectral tables (nspec
// doubles, followed in device memory by the dense inverse where there is one).
struct TailDesc {
    int nlev;
    int nspec;
    int nx[kMaxLevels], ny[kMaxLevels], nz[kMaxLevels];
    double s[kMaxLevels], diag[kMaxLevels];
    double inv_diag[kMaxLevels][4];  // box: by the faces a cell touches, rounded as 1 / (diag + f s) in T
    unsigned off_u[kMaxLevels], off_nat[kMaxLevels];
    unsigned off_ab, off_spec;
    unsigned lds_bytes;
};

// Learned preconditioner network: flat float32 parameter vector
// [W1 (64 x 12, row = output) | b1 | W2 (64 x 64) | b2 | w3 | b3].
constexpr int kNetFeat = 12;
constexpr int kOffW1 = 0, kOffB1 = 768, kOffW2 = 832, kOffB2 = 4928, kOffW3 = 4992, kOffB3 = 5056;
constexpr int kNetParams = 5057;
constexpr float kNuScale = 0.25f;  // neighbour counts enter the network as nu / 4

struct NetDev {
    const float* P;     // float32 masters
    const __bf16* W1b;  // [64][16] bfloat16, columns >= 10 zero
    const __bf16* W2b;  // [64][64] bfloat16
    const __bf16* w3b;  // [64] bfloat16
};

struct PairGeom {
    double box[3];  // box edge per axis (x, y, z)
    double h;
    double rc;      // pair cutoff
    int ncx, ncy, ncz;  // pair-search cells per axis
    const float* nu;    // per blob: other blobs within rc / 2 (network input; null while the list is built)
};

struct BlobGeom {
    int nx, ny, nz;
    int tx, ty, tz;      // tile edge per axis (divides the grid edge)
    int ntx, nty, ntz;   // tiles per axis
    double h;
    int w;
};

// Contribution lists of the spread: n touched cells, cell[k] its grid index,
// entries ptr[k] .. ptr[k+1] of (blob[e], weight w[e]).
struct SpreadLists {
    int n;
    const int* cell;
    const int* ptr;
    const int* blob;
    const double* w;
};
// Multipliers a spread takes: lam[b] + c2 lam2[b] + shift (lam, lam2 may be null).
struct SpreadMult {
    const double* lam;
    const double* lam2;
    double c2;
    double shift;
};

// A box held at a fixed face value (Dirichlet): the homogeneous operator takes the
// ghost beyond a face as minus the boundary cell, so a cell touching f faces has
// the diagonal alpha + s (6 + f) and no neighbour term across them. v[f] holds
// the per-cell coefficient (diagonal or its inverse) for f = 0..3.
struct BoxCoef {
    double v[4];
};

// Logical block of a launch: partial-sum slot b of nb. Solo kernels pass
// (blockIdx.x, gridDim.x); batched kernels pass an instance's local slot, so
// every instance's partition of work and of partial sums is the solo one.
struct Blk {
    unsigned b, nb;
};

// One instance's slice of a batched launch: global blocks [block0, block0 + nb)
// (block0 a multiple of 8, so a slot keeps the XCD of its solo launch).
struct BatchEntry {
    unsigned block0, nb;
    int inst;
    int pad;
};

// Everything a batched CG iteration reads about one instance (device memory).
struct InstDev {
    Scalars* sc;
    double* part;
    double *x, *r, *q, *p[2];             // CG vectors of the current solve (direction of iteration k in p[k & 1])
    double alpha;                         // operator alpha I - D L (+ S kappa J)
    int nx, ny, nz, nlev, t;              // level 0 dims, levels, first tail level
    int np_apply, np_update, np_dots;     // partial slots of the three reductions
    void* lv[kMaxLevels][5];              // split level arrays u0, u1, f0, f1, r0
    int lnx[kMaxLevels], lny[kMaxLevels], lnz[kMaxLevels];
    double ls[kMaxLevels], ldiag[kMaxLevels];  // D / h_l^2 and alpha + 6 s_l
    int blobs, N;                         // blob term in the operator (reactive)
    BlobGeom geom;
    const int* base;
    const double* wts;
    const int* offsets;
    const int* perm;
    const double* kappa;
    double* jx;
    double* mu;
    double inv_h3;
    int ntouched;                         // spread contribution lists (touched cells, entries)
    const int* tcell;
    const int* tptr;
    const int* tblob;
    const double* tw;
    const double* spec;                   // coarsest solve's spectral tables for alpha
    TailDesc tail;
};

struct LevelDims {
    int nx, ny, nz;   // cells
    int hx;           // nx / 2 (split levels)
    double h;         // spacing at this level
};

// ---- helpers -------------------------------------------------------------
__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// The smoother's update, the red residual and one row of the restriction, with their
// roundings fixed (no contraction beyond the explicit FMAs), so that every form of a level
// (per step, two launches a level, LDS tail) gives the same bits.
template <typename T>
__device__ __forceinline__ T relax(T f, T s, T nb, T inv_diag) {
#pragma clang fp contract(off)
    return fma(s, nb, f) * inv_diag;
}
template <typename T>
__device__ __forceinline__ T relax_zero(T f, T inv_diag) {  // from a zero guess
#pragma clang fp contract(off)
    return f * inv_diag;
}
template <typename T>
__device__ __forceinline__ T red_resid(T f, T diag, T u, T s, T nb) {
#pragma clang fp contract(off)
    return f - fma(diag, u, -(s * nb));
}
// p = 1: (a, b) = r0[X-1], r0[X]; p = 0: (b, c) = r0[X], r0[X+1]
template <typename T>
__device__ __forceinline__ T restrict_row(T w0, T w1, int p, T a, T b, T c) {
#pragma clang fp contract(off)
    return fma(w1, b, w0 * (p ? a : c));
}

// Tile of a two-launch level: lanes vectors of vw cells to a row, ty rows and tz planes to a
// work-group, nty x ntz tiles, and the multipliers that divide by lanes and by the windows'
// rows a plane. lanes = 0: not applicable.
struct LevelTile {
    int lanes, vw, ty, tz, nty, ntz;
    unsigned mlanes, mdown, mup;
};

// Coefficients of a level in its precision: s = D / h^2 and, by the box faces a cell touches
// (all alike in the periodic cell), the diagonals, their inverses and the next level's.
template <typename T>
struct LevelCoef {
    T s, diag[4], inv[4], invc[4];
};

// u plus the trilinear correction of one fine cell from its four coarse rows (J0, K0),
// (J1, K0), (J0, K1), (J1, K1): m is a row's value at the cell's own coarse x, n the one at
// the neighbour on the cell's side. Evaluated as written, with no contraction beyond the
// explicit FMAs, so that every form of the correction (per level, blocked, LDS tail) rounds
// alike.
template <typename T>
__device__ __forceinline__ T tri_add(T u, T m00, T n00, T m10, T n10, T m01, T n01, T m11, T n11) {
#pragma clang fp contract(off)
    const T a00 = fma((T)0.75, m00, (T)0.25 * n00);
    const T a10 = fma((T)0.75, m10, (T)0.25 * n10);
    const T a01 = fma((T)0.75, m01, (T)0.25 * n01);
    const T a11 = fma((T)0.75, m11, (T)0.25 * n11);
    const T b0 = fma((T)0.75, a00, (T)0.25 * a10);
    const T b1 = fma((T)0.75, a01, (T)0.25 * a11);
    return u + fma((T)0.75, b0, (T)0.25 * b1);
}

// number of box faces cell (x, y, z) touches (at most one per axis for edges >= 2)
__device__ __forceinline__ int box_faces(int x, int y, int z, int nx, int ny, int nz) {
    return (x == 0) + (x == nx - 1) + (y == 0) + (y == ny - 1) + (z == 0) + (z == nz - 1);
}

// Value of cell (X, Y, Z) of a red/black split level (colour (X + Y + Z) mod 2,
// index X/2 of row (Y, Z) of its colour array, hx = nx/2) as a double.
template <typename T>
__device__ __forceinline__ double split_at(const T* __restrict__ z0, const T* __restrict__ z1, int X, int Y, int Z,
                                           int hx, int ny) {
    const size_t j = ((size_t)Z * ny + Y) * hx + (X >> 1);
    return ((X + Y + Z) & 1) ? (double)z1[j] : (double)z0[j];
}

// g - (alpha c - D L c) at natural cell (X, Y, Z) of the periodic level 0 (nx even, s = D / h^2)
// with c in the split layout, in FP64 on c's values: the stencil association of the natural
// two-cell form (x pair, y pair, z pair, then the centre).
template <typename T>
__device__ __forceinline__ double split_resid(const double* __restrict__ g, const T* __restrict__ c0,
                                              const T* __restrict__ c1, int X, int Y, int Z, int nx, int ny, int nz,
                                              double alpha, double s) {
    const int hx = nx >> 1;
    const double c = split_at(c0, c1, X, Y, Z, hx, ny);
    const double xl = split_at(c0, c1, wrapi(X - 1, nx), Y, Z, hx, ny);
    const double xr = split_at(c0, c1, wrapi(X + 1, nx), Y, Z, hx, ny);
    const double ym = split_at(c0, c1, X, wrapi(Y - 1, ny), Z, hx, ny);
    const double yp = split_at(c0, c1, X, wrapi(Y + 1, ny), Z, hx, ny);
    const double zm = split_at(c0, c1, X, Y, wrapi(Z - 1, nz), hx, ny);
    const double zp = split_at(c0, c1, X, Y, wrapi(Z + 1, nz), hx, ny);
    const double a = alpha * c - s * ((xl + xr) + (ym + yp) + (zm + zp) - 6.0 * c);
    return g[((size_t)Z * ny + Y) * nx + X] - a;
}

// Blocks are dispatched to the 8 XCDs round-robin; this remaps the hardware
// block id so each XCD works on one contiguous eighth of the index space,
// keeping neighbouring rows and planes in the same XCD's L2.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned nb) {
    unsigned full = nb >> 3, rem = nb & 7u, xcd = b & 7u, local = b >> 3;
    return xcd * full + (xcd < rem ? xcd : rem) + local;
}

// Work-group barrier that orders LDS accesses only: unlike __syncthreads() it does not wait
// for global loads and stores in flight. For kernels whose threads exchange data in LDS alone.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The value of lane c of every quad of lanes (DPP quad_perm).
template <int C>
__device__ __forceinline__ float quad_value(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x55 * C, 0xf, 0xf, false));
}
template <int C>
__device__ __forceinline__ double quad_value(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x55 * C, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x55 * C, 0xf, 0xf, false));
}

// v plus the value DPP moves to this lane (zero where it moves none): register moves between
// lanes, without the LDS round trip of a shuffle.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return v + __hiloint2double(hi, lo);
}
// Lane 15 of each row of 16 lanes gets the row's sum (row_shr 1, 2, 4, 8).
__device__ __forceinline__ double row_sum(double v) {
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    return dpp_add<0x118, 0xf>(v);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum over a whole wave (all 64 lanes active), the same value in every lane.
__device__ __forceinline__ double wave_sum(double v) {
    v = row_sum(v);
    v = dpp_add<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3
    return lane_value(v, 63);
}

// Sums of K values over one work-group: wave sums, then the waves' sums by a row of lanes.
// Every thread gets the totals. A single work-group that reduces is a chain of latencies: with
// shuffles and a loop over the waves' sums a kernel of three such sums took 4.8 us, as here
// 2.9 us (k_fin at 32^3; 5.6 -> 4.2 us at 128^3, k_gmres_arnoldi 10.5 -> 7.0 us at 156 blobs,
// k_nvec_project 3.1 -> 2.2 us).
template <int K>
__device__ __forceinline__ void wg_sums(double (&v)[K]) {
    __shared__ double sh[K][kFinBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
    lds_barrier();  // readers of an earlier call are done
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) sh[k][wid] = v[k];
    lds_barrier();
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = lane_value(row_sum(lane < nw ? sh[k][lane & 15] : 0.0), 15);
}
__device__ __forceinline__ double wg_sum(double s) {
    double v[1] = {s};
    wg_sums<1>(v);
    return v[0];
}

// Inclusive scan of one value a lane over the wave (T a 32- or 64-bit integer).
template <typename T>
__device__ __forceinline__ T wave_scan(T v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}
// Exclusive scan of one value a thread over the work-group (blockDim a multiple of 64), *total
// its sum.
template <typename T>
__device__ __forceinline__ T wg_scan(T v, T* total) {
    __shared__ T sh[kFinBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
    const T inc = wave_scan(v);
    lds_barrier();  // readers of an earlier call are done
    if (lane == 63) sh[wid] = inc;
    lds_barrier();
    const T w = wave_scan(lane < nw ? sh[lane & 15] : (T)0);
    *total = __shfl(w, nw - 1, 64);
    const T before = __shfl(w, wid > 0 ? wid - 1 : 0, 64);
    return (wid > 0 ? before : (T)0) + inc - v;
}

// Deterministic block reduction of K values; the first wave writes block partial k to
// part[k * nparts + slot].
template <int K>
__device__ __forceinline__ void block_partials(double (&v)[K], double* part, unsigned nparts, unsigned slot) {
    __shared__ double sh[K][16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) sh[k][wid] = v[k];
    lds_barrier();
    if (wid == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double t = row_sum(lane < nw ? sh[k][lane & 15] : 0.0);
            if (lane == 15) part[(size_t)k * nparts + slot] = t;
        }
}

inline unsigned nblocks(size_t n, int bs = kBlock) { return (unsigned)((n + bs - 1) / bs); }

// Reductions over grid vectors use at most kRedBlocks blocks, each owning one
// contiguous chunk of the index space, so the finalize reads few partials.
constexpr unsigned kRedBlocks = 4096;
inline unsigned red_blocks(size_t n) {
    const unsigned nb = nblocks(n);
    return nb < kRedBlocks ? nb : kRedBlocks;
}
// Blocks of CG's vector passes over n cell pairs: a pair per thread up to 2^19 pairs (10^6 cells);
// beyond, two blocks to a CU, whose longer contiguous runs use HBM better on large grids (256^3:
// direction 149 us, update 75; 256 blocks 148, 113; 768: 157, 74; 4096: 165, 87) and whose partials
// are few enough for the next pass to sum by itself. Without that folding a set-up at 128^3 (2^20
// pairs) was 1 % slower in 512 blocks; with it, whole reactive solves (FP32, us, a pair per thread /
// 512 blocks): 80 x 112 x 96 1201 / 1203, 96^3 1080 / 1095, 96 x 96 x 112 1397 / 1380 (just below
// the line), 112 x 112 x 96 1295 / 1259, 112^3 1506 / 1488, 128^3 1535 / 1495, 128 x 160 x 128
// 1765 / 1708, 160^3 2289 / 2275, 192^3 3257 / 3294.
inline unsigned cg_blocks(size_t n) { return n > ((size_t)1 << 19) ? 512 : nblocks(n); }
// Entry of a batched launch that owns global block g (entries sorted by block0).
__device__ __forceinline__ int batch_entry(const BatchEntry* e, int n, unsigned g) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (e[mid].block0 <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// A batched launch's work list, rebuilt for the instances taking part in each
// round: `total` virtual blocks over `n` entries (the BatchEntry array follows
// the header). Launches have a fixed grid that strides over the virtual blocks.
struct BatchTab {
    unsigned total;
    int n;
    int pad0, pad1;
};
__device__ __forceinline__ const BatchEntry* tab_entries(const BatchTab* t) {
    return reinterpret_cast<const BatchEntry*>(t + 1);
}

// The instance and local block of virtual block g, or null when g is padding,
// the instance is not gated in, or its solve is done (uniform per block, so
// callers may skip barriers together).
__device__ __forceinline__ const InstDev* batch_slot(const InstDev* inst, const int* gate, const BatchEntry* ent,
                                                     int nent, unsigned g, Blk& blk) {
    const BatchEntry e = ent[batch_entry(ent, nent, g)];
    const unsigned b = g - e.block0;
    if (b >= e.nb || !gate[e.inst]) return nullptr;
    const InstDev* I = inst + e.inst;
    if (I->sc->done) return nullptr;
    blk.b = b;
    blk.nb = e.nb;
    return I;
}

// chunk [lo, hi) of logical block b of nb over n items (chunks are multiples of blockDim)
__device__ __forceinline__ void chunk_of(unsigned b, unsigned nb, unsigned n, unsigned* lo, unsigned* hi) {
    const unsigned per = ((n + nb - 1) / nb + blockDim.x - 1) / blockDim.x * blockDim.x;
    const unsigned l = b * per;
    *lo = l < n ? l : n;
    *hi = l + per < n ? l + per : n;
}

}  // namespace brd
