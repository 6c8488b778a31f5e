// A large level of the V-cycle in tiles cut on all three axes: pre-smoothing, red residual and
// restriction in two launches (k_slab_open, k_slab_restrict), three post-smoothing half-sweeps
// in one (k_slab_post), for alpha I - D L on the periodic cell and in a box with homogeneous
// faces (arXiv:1306.3159 Sec. III.E, eq. Helmholtz; the box of Sec. IV.C). The cells'
// arithmetic is that of the per-step kernels, so in the periodic cell the results are bitwise
// theirs.
//
// On levels above some 10^6 cells the per-step launches are bound by the bytes that each
// half-sweep moves (its colour's f and u, the other colour's u: 16 us at 256^3 in FP32, 6 TB/s).
// Several steps in one launch move f once and leave out values that only the next step reads. A
// work-group owns 8 x 8 rows of 8 vectors and works outwards-in: the opening colour on the cells
// at most 3 from the tile (|dx| + |dy| + |dz|, the cells a result depends on), then 2, 1, 0.
// Each thread owns at most one vector of every distance (512 own vectors, then 384, 352 and
// 392), so that no step leaves waves idle, holds values and right-hand sides in registers and
// takes its neighbours from LDS. What bounds it then is the load of a window and the four steps
// behind it, so it needs work-groups that overlap: three to a CU by LDS (53 KB each) and
// registers; with two, the launches of 31 and 29 us below took 43 and 34.
// Measured (kernel trace, FP32): 256^3 down 23.6 + 31.0 us (per-step launches 88), correction
// and post-smoothing without the closing red sweep 16.6 + 28.6 (65); box 22.0 + 36.6 (87) and
// 22.3 + 35.5 (72); 128^3 5.2 + 7.0 and 5.1 + 6.1 (two launches of kernels_level.hip: 15.1 and
// 15.5). Residual and restriction alone in one launch, behind three half-sweeps: 31.8 + 36.8.
#include "level.hpp"

namespace brd {

namespace {

constexpr int kSlab = 8;                                 // rows and planes of a tile, vectors of its rows
constexpr int kSlabThreads = kSlab * kSlab * kSlab;
constexpr int kSlabRow = kSlab + 2;                      // vectors of a window row: one more on each side

// A vector of the window: rows relative to the tile, vector relative to the segment.
struct SlabPos {
    int y, z, v;
    bool on;
};

// Thread t's vector at distance d >= 1 from the tile: rows at that distance over each face of
// the tile (256 threads), rows over its edges (32 (d - 1)), and the vectors beside rows at
// distance d - 1 (their cells next to the segment are at distance d and more).
__device__ __forceinline__ SlabPos slab_ring(int t, int d) {
    SlabPos p{0, 0, 0, true};
    const int edge = 32 * (d - 1);
    if (t < 256 + edge) {
        p.v = t & 7;
        if (t < 256) {
            const int side = t >> 6, a = (t >> 3) & 7, out = (side & 1) ? kSlab - 1 + d : -d;
            p.y = side < 2 ? out : a;
            p.z = side < 2 ? a : out;
        } else {
            const int c = (t - 256) >> 3, ey = 1 + (c >> 2), ez = d - ey;
            p.y = (c & 1) ? kSlab - 1 + ey : -ey;
            p.z = (c & 2) ? kSlab - 1 + ez : -ez;
        }
        return p;
    }
    const int e = t - 256 - edge, r = e >> 1;
    p.v = (e & 1) ? kSlab : -1;
    if (d == 1) {
        p.y = r & 7;
        p.z = r >> 3;
        p.on = r < 64;
    } else if (r < 32) {
        const int side = r >> 3, a = r & 7, out = (side & 1) ? kSlab - 2 + d : 1 - d;
        p.y = side < 2 ? out : a;
        p.z = side < 2 ? a : out;
    } else {
        const int c = r - 32;
        p.y = (c & 1) ? kSlab : -1;
        p.z = (c & 2) ? kSlab : -1;
        p.on = d == 3 && c < 4;
    }
    return p;
}

// Where a vector of the window lies in the grid: offset in a colour's array, x parity of its
// red cells, faces of a box and whether it is inside it (always in the periodic cell, whose
// window wraps), first / last vector of the row.
struct SlabItem {
    unsigned goff;
    int par, faces;
    bool in, first, last;
};

template <int VW, bool BOX>
__device__ __forceinline__ SlabItem slab_item(const SlabPos& p, int v0, int y0, int z0, int hv, int ny, int nz) {
    SlabItem it;
    const int vu = v0 + p.v, yu = y0 + p.y, zu = z0 + p.z;
    const int v = wrapi(vu, hv), y = wrapi(yu, ny), z = wrapi(zu, nz);
    it.goff = (((unsigned)z * ny + y) * hv + v) * VW;
    it.par = (y + z) & 1;
    it.in = !BOX || (vu >= 0 && vu < hv && yu >= 0 && yu < ny && zu >= 0 && zu < nz);
    it.faces = BOX ? (y == 0) + (y + 1 == ny) + (z == 0) + (z + 1 == nz) : 0;
    it.first = v == 0;
    it.last = v + 1 == hv;
    return it;
}

// tab by the faces a cell touches, for a vector's cells of x parity so
template <typename T, int VW, bool BOX>
__device__ __forceinline__ typename RowVec<T, VW>::type slab_diag(const T* tab, const SlabItem& it, int so) {
    typedef typename RowVec<T, VW>::type V;
    if (!BOX) return (V)(tab[0]);
    const T t0 = tab[0], t1 = tab[1], t2 = tab[2], t3 = tab[3];
    const int f = it.faces;
    const T base = f == 0 ? t0 : (f == 1 ? t1 : t2), edge = f == 0 ? t1 : (f == 1 ? t2 : t3);
    V d = (V)(base);
    if (so == 0 && it.first) d[0] = edge;
    if (so == 1 && it.last) d[VW - 1] = edge;
    return d;
}

// Neighbour sums of a vector whose cells have x parity so: o the other colour's vector at the
// same place, e its neighbour value in the row, and the four rows around.
template <typename T, int VW>
__device__ __forceinline__ typename RowVec<T, VW>::type slab_nb(typename RowVec<T, VW>::type o, T e, int so,
                                                                typename RowVec<T, VW>::type ym,
                                                                typename RowVec<T, VW>::type yp,
                                                                typename RowVec<T, VW>::type zm,
                                                                typename RowVec<T, VW>::type zp) {
    typename RowVec<T, VW>::type nb;
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        const T x = so ? (k + 1 < VW ? o[k + 1] : e) : (k ? o[k - 1] : e);
        nb[k] = ((o[k] + x) + (ym[k] + yp[k])) + (zm[k] + zp[k]);
    }
    return nb;
}

// The same from a colour's window in LDS (q: the vector's place; rows of a plane).
template <typename T, int VW, int ROWS>
__device__ __forceinline__ typename RowVec<T, VW>::type slab_sum(const T* q, typename RowVec<T, VW>::type o, int so) {
    typedef typename RowVec<T, VW>::type V;
    constexpr int Y = kSlabRow * VW, Z = ROWS * Y;
    return slab_nb<T, VW>(o, q[so ? VW : -1], so, *reinterpret_cast<const V*>(q - Y),
                          *reinterpret_cast<const V*>(q + Y), *reinterpret_cast<const V*>(q - Z),
                          *reinterpret_cast<const V*>(q + Z));
}

// Tile t: segments of a row first, then up to four planes of tiles, then rows. The tiles that an
// XCD works on at a time then share their window's rows in y and z through its L2; in the order
// rows before planes the six planes around a tile were read again (the post-smoothing: 33.8 us
// against 31.7 then).
struct SlabTile {
    int v0, y0, z0;
    __device__ __forceinline__ SlabTile(unsigned t, int hv, int ny, int nz) {
        const unsigned ns = (hv + kSlab - 1) / kSlab, nty = (ny + kSlab - 1) / kSlab, ntz = (nz + kSlab - 1) / kSlab;
        const unsigned group = t / (4 * ns * nty), r = t - group * 4 * ns * nty;
        const unsigned gz = min(4u, ntz - 4 * group), row = r / ns, y = row / gz;
        v0 = (int)(r - row * ns) * kSlab;
        y0 = (int)y * kSlab;
        z0 = (int)(4 * group + row - y * gz) * kSlab;
    }
};

}  // namespace

// A colour's window in LDS: HALO rows and planes around the tile. The first CUT rows of the
// first plane and the last CUT of the last, at its edges, are not needed and not allocated:
// three work-groups of the two large windows then fit a CU (LDS is given out in 1280 bytes).
template <int HALO, int CUT>
struct SlabWin {
    static constexpr int rows = kSlab + 2 * HALO, size = (rows * rows - 2 * CUT) * kSlabRow;
    static __device__ __forceinline__ int place(const SlabPos& p) {
        return ((p.z + HALO) * rows + p.y + HALO - CUT) * kSlabRow + p.v + 1;
    }
};
constexpr int kSlabWaves = 6;  // waves per SIMD: three work-groups
__device__ __forceinline__ SlabPos slab_own(int t) { return SlabPos{(t >> 3) & 7, t >> 6, t & 7, true}; }

// One half-sweep of a vector (x parity so) from the other colour's window: q the vector's place
// in it, o its value there. Cells outside a box stay zero.
template <typename T, int VW, int ROWS, bool BOX>
__device__ __forceinline__ typename RowVec<T, VW>::type slab_relax(const typename RowVec<T, VW>::type* q,
                                                                   typename RowVec<T, VW>::type o,
                                                                   typename RowVec<T, VW>::type f, const SlabItem& it,
                                                                   int so, const LevelCoef<T>& c) {
    typedef typename RowVec<T, VW>::type V;
    const V nb = slab_sum<T, VW, ROWS>(reinterpret_cast<const T*>(q), o, so);
    const V d = slab_diag<T, VW, BOX>(c.inv, it, so);
    V u;
#pragma unroll
    for (int k = 0; k < VW; ++k) u[k] = BOX && !it.in ? (T)0 : relax(f[k], c.s, nb[k], d[k]);
    return u;
}

// Red (f0 / diag, from a zero guess), black and red half-sweeps; red is written (the black
// values are those of the next black half-sweep, which the residual's launch takes first).
template <typename T, int VW, bool BOX>
__global__ void __launch_bounds__(kSlabThreads) k_slab_open(T* __restrict__ u0g, const T* __restrict__ f0g,
                                                            const T* __restrict__ f1g, int hv, int ny, int nz,
                                                            LevelCoef<T> c, const Scalars* sc) {
    typedef typename RowVec<T, VW>::type V;
    if (sc && sc->done) return;
    typedef SlabWin<2, 2> Red;
    typedef SlabWin<1, 1> Black;
    __shared__ V red[Red::size], black[Black::size];
    const SlabTile tile(xcd_block(blockIdx.x, gridDim.x), hv, ny, nz);
    const int t = threadIdx.x;
    SlabItem it[3];
    int ro[3], bo[2];
    bool on[3];
    V F0[3], F1[2], u0[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const SlabPos p = j == 0 ? slab_own(t) : slab_ring(t, j);
        on[j] = p.on;
        it[j] = slab_item<VW, BOX>(p, tile.v0, tile.y0, tile.z0, hv, ny, nz);
        ro[j] = Red::place(p);
        F0[j] = (V)(T)0;
        if (p.on && it[j].in) F0[j] = *reinterpret_cast<const V*>(f0g + it[j].goff);
        if (j < 2) {
            bo[j] = Black::place(p);
            F1[j] = (V)(T)0;
            if (p.on && it[j].in) F1[j] = *reinterpret_cast<const V*>(f1g + it[j].goff);
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j)
        if (on[j]) {
            const V d = slab_diag<T, VW, BOX>(c.inv, it[j], it[j].par);
#pragma unroll
            for (int k = 0; k < VW; ++k) u0[j][k] = relax_zero(F0[j][k], d[k]);
            red[ro[j]] = u0[j];
        }
    lds_barrier();
    V u1 = (V)(T)0;
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (on[j]) {
            const V u = slab_relax<T, VW, Red::rows, BOX>(red + ro[j], u0[j], F1[j], it[j], it[j].par ^ 1, c);
            black[bo[j]] = u;
            if (j == 0) u1 = u;
        }
    lds_barrier();
    if (tile.v0 + (t & 7) < hv && tile.y0 + ((t >> 3) & 7) < ny && tile.z0 + (t >> 6) < nz)
        *reinterpret_cast<V*>(u0g + it[0].goff) =
            slab_relax<T, VW, Black::rows, BOX>(black + bo[0], u1, F0[0], it[0], it[0].par, c);
}

// Thread t's vector of set j of the window of k_slab_restrict, whose tile takes one row, plane
// and vector more on each side (the residual there enters the restriction): the own vectors,
// the 488 around them, then the rows next to those (400) and the rows next to these (440).
__device__ __forceinline__ SlabPos slab_wide(int t, int j) {
    if (j == 0) return slab_own(t);
    if (j == 1) {
        if (t < 256) return slab_ring(t, 1);
        const int q = (t - 256) >> 3, e = t - 288, r = e >> 1;
        if (t < 288) return SlabPos{(q & 1) ? kSlab : -1, (q & 2) ? kSlab : -1, t & 7, true};
        return SlabPos{r % kSlabRow - 1, r / kSlabRow - 1, (e & 1) ? kSlab : -1, r < kSlabRow * kSlabRow};
    }
    const int row = t / kSlabRow, v = t - row * kSlabRow - 1;
    if (row < 4 * kSlabRow) {
        const int side = row / kSlabRow, a = row - side * kSlabRow - 1, out = (side & 1) ? kSlab - 1 + j : -j;
        return SlabPos{side < 2 ? out : a, side < 2 ? a : out, v, true};
    }
    const int q = row - 4 * kSlabRow;
    return SlabPos{(q & 1) ? kSlab + 1 : -2, (q & 2) ? kSlab + 1 : -2, v, j == 3 && q < 4};
}

// Black half-sweep, red residual and its restriction to the tile's coarse cells (the four fine
// planes of a coarse vector by the lanes of a quad). No fine value is written: the black ones
// are not read again (post-smoothing starts with black).
template <typename T, int VW, bool BOX>
__global__ void __launch_bounds__(kSlabThreads, kSlabWaves) k_slab_restrict(const T* __restrict__ u0g, const T* __restrict__ f0g,
                                                                const T* __restrict__ f1g, int hv, int ny, int nz,
                                                                LevelCoef<T> c, T* __restrict__ cf0,
                                                                T* __restrict__ cf1, T* __restrict__ cu0,
                                                                const Scalars* sc) {
    typedef typename RowVec<T, VW>::type V;
    if (sc && sc->done) return;
    typedef SlabWin<3, 2> Red;
    typedef SlabWin<2, 1> Black;
    __shared__ V red[Red::size], black[Black::size];
    const SlabTile tile(xcd_block(blockIdx.x, gridDim.x), hv, ny, nz);
    const int t = threadIdx.x;
    SlabItem it[4];
    int ro[4], bo[3];
    bool on[4];
    V F0[2], F1[3], u0[4], u1[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const SlabPos p = slab_wide(t, j);
        on[j] = p.on;
        it[j] = slab_item<VW, BOX>(p, tile.v0, tile.y0, tile.z0, hv, ny, nz);
        ro[j] = Red::place(p);
        const bool ld = p.on && it[j].in;
        u0[j] = (V)(T)0;
        if (ld) u0[j] = *reinterpret_cast<const V*>(u0g + it[j].goff);
        if (j < 2) {
            F0[j] = (V)(T)0;
            if (ld) F0[j] = *reinterpret_cast<const V*>(f0g + it[j].goff);
        }
        if (j < 3) {
            bo[j] = Black::place(p);
            F1[j] = (V)(T)0;
            if (ld) F1[j] = *reinterpret_cast<const V*>(f1g + it[j].goff);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (on[j]) red[ro[j]] = u0[j];
    lds_barrier();
#pragma unroll
    for (int j = 0; j < 3; ++j)
        if (on[j]) {
            const V u = slab_relax<T, VW, Red::rows, BOX>(red + ro[j], u0[j], F1[j], it[j], it[j].par ^ 1, c);
            black[bo[j]] = u;
            if (j < 2) u1[j] = u;
        }
    lds_barrier();
    // residuals over the red values (their owners keep them)
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (on[j]) {
            const V nb = slab_sum<T, VW, Black::rows>(reinterpret_cast<const T*>(black + bo[j]), u1[j], it[j].par);
            const V d = slab_diag<T, VW, BOX>(c.diag, it[j], it[j].par);
            V r;
#pragma unroll
            for (int k = 0; k < VW; ++k)
                r[k] = BOX && !it[j].in ? (T)0 : red_resid(F0[j][k], d[k], u0[j][k], c.s, nb[k]);
            red[ro[j]] = r;
        }
    lds_barrier();
    // coarse vector q of the tile, plane a of its four
    const int a = t & 3, q = t >> 2, v = q & 7, qy = (q >> 3) & 3, qz = q >> 5;
    const int gv = tile.v0 + v, Y = (tile.y0 >> 1) + qy, Z = (tile.z0 >> 1) + qz;
    T acc[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) acc[k] = (T)0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const V* r = red + Red::place(SlabPos{2 * qy - 1 + b, 2 * qz - 1 + a, v, true});
        const int pr = (a + b) & 1;  // red cells of the row (y, z): x = 2i + pr (y0 and z0 are even)
        const T x = reinterpret_cast<const T*>(r)[pr ? -1 : VW];
        const T wgt = BOX ? level_rweight<T>(b, Y, ny) : ((b == 0 || b == 3) ? (T)0.125 : (T)0.375);
        level_restrict_row<T, VW, BOX>(acc, *r, x, pr, wgt, gv == 0, gv + 1 == hv);
    }
    T sum[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        const T p[4] = {quad_value<0>(acc[k]), quad_value<1>(acc[k]), quad_value<2>(acc[k]), quad_value<3>(acc[k])};
        sum[k] = (T)0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const T wgt = BOX ? level_rweight<T>(b, Z, nz) : ((b == 0 || b == 3) ? (T)0.125 : (T)0.375);
            sum[k] = fma(wgt, p[b], sum[k]);
        }
    }
    if (a == 0 && gv < hv && 2 * Y < ny && 2 * Z < nz)
        level_coarse_store<T, VW, BOX>(sum, gv * VW, Y, Z, hv * VW, ny >> 1, nz >> 1, c, cf0, cf1, cu0);
}

// Black, red and black half-sweeps of the corrected values; black is written (the closing red
// half-sweep reads black and f0 only).
template <typename T, int VW, bool BOX>
__global__ void __launch_bounds__(kSlabThreads, kSlabWaves) k_slab_post(const T* __restrict__ u0g, T* __restrict__ u1g,
                                                            const T* __restrict__ f0g, const T* __restrict__ f1g,
                                                            int hv, int ny, int nz, LevelCoef<T> c,
                                                            const Scalars* sc) {
    typedef typename RowVec<T, VW>::type V;
    if (sc && sc->done) return;
    typedef SlabWin<3, 3> Red;
    typedef SlabWin<2, 2> Black;
    __shared__ V red[Red::size], black[Black::size];
    const SlabTile tile(xcd_block(blockIdx.x, gridDim.x), hv, ny, nz);
    const int t = threadIdx.x;
    SlabItem it[4];
    int ro[4], bo[3];
    bool on[4];
    V F0[2], F1[3], u0[4], u1[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const SlabPos p = j == 0 ? slab_own(t) : slab_ring(t, j);
        on[j] = p.on;
        it[j] = slab_item<VW, BOX>(p, tile.v0, tile.y0, tile.z0, hv, ny, nz);
        ro[j] = Red::place(p);
        const bool ld = p.on && it[j].in;
        u0[j] = (V)(T)0;
        if (ld) u0[j] = *reinterpret_cast<const V*>(u0g + it[j].goff);
        if (j < 2) {
            F0[j] = (V)(T)0;
            if (ld) F0[j] = *reinterpret_cast<const V*>(f0g + it[j].goff);
        }
        if (j < 3) {
            bo[j] = Black::place(p);
            F1[j] = (V)(T)0;
            if (ld) F1[j] = *reinterpret_cast<const V*>(f1g + it[j].goff);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (on[j]) red[ro[j]] = u0[j];
    lds_barrier();
#pragma unroll
    for (int j = 0; j < 3; ++j)
        if (on[j]) {
            const V u = slab_relax<T, VW, Red::rows, BOX>(red + ro[j], u0[j], F1[j], it[j], it[j].par ^ 1, c);
            black[bo[j]] = u;
            if (j < 2) u1[j] = u;
        }
    lds_barrier();
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (on[j]) {
            u0[j] = slab_relax<T, VW, Black::rows, BOX>(black + bo[j], u1[j], F0[j], it[j], it[j].par, c);
            red[ro[j]] = u0[j];
        }
    lds_barrier();
    if (tile.v0 + (t & 7) < hv && tile.y0 + ((t >> 3) & 7) < ny && tile.z0 + (t >> 6) < nz)
        *reinterpret_cast<V*>(u1g + it[0].goff) =
            slab_relax<T, VW, Red::rows, BOX>(red + ro[0], u0[0], F1[0], it[0], it[0].par ^ 1, c);
}

// Work-groups of a level.
unsigned slab_tiles(int nx, int ny, int nz, size_t esz) {
    const int hv = nx / 2 / (int)(16 / esz);
    return (unsigned)((hv + kSlab - 1) / kSlab) * ((ny + kSlab - 1) / kSlab) * ((nz + kSlab - 1) / kSlab);
}

// Levels that these kernels take: rows of whole 16-byte vectors, axes that a window, at most 3
// below and 10 above a tile's first row, wraps at most once.
bool slab_fits(int nx, int ny, int nz, size_t esz) {
    const int vw = (int)(16 / esz);
    return nx % (2 * vw) == 0 && nx / 2 / vw >= kSlab + 1 && ny >= 2 * kSlab && nz >= 2 * kSlab;
}

template <typename T>
void launch_slab_down(hipStream_t st, bool box, T* u0, const T* f0, const T* f1, int nx, int ny, int nz,
                      const LevelCoef<T>& c, T* cf0, T* cf1, T* cu0, const Scalars* sc) {
    constexpr int VW = 16 / (int)sizeof(T);
    const int hv = nx / 2 / VW;
    const dim3 g(slab_tiles(nx, ny, nz, sizeof(T))), b(kSlabThreads);
    if (box) {
        hipLaunchKernelGGL((k_slab_open<T, VW, true>), g, b, 0, st, u0, f0, f1, hv, ny, nz, c, sc);
        hipLaunchKernelGGL((k_slab_restrict<T, VW, true>), g, b, 0, st, u0, f0, f1, hv, ny, nz, c, cf0, cf1, cu0, sc);
    } else {
        hipLaunchKernelGGL((k_slab_open<T, VW, false>), g, b, 0, st, u0, f0, f1, hv, ny, nz, c, sc);
        hipLaunchKernelGGL((k_slab_restrict<T, VW, false>), g, b, 0, st, u0, f0, f1, hv, ny, nz, c, cf0, cf1, cu0, sc);
    }
}

template <typename T>
void launch_slab_post(hipStream_t st, bool box, const T* u0, T* u1, const T* f0, const T* f1, int nx, int ny, int nz,
                      const LevelCoef<T>& c, const Scalars* sc) {
    constexpr int VW = 16 / (int)sizeof(T);
    const int hv = nx / 2 / VW;
    const dim3 g(slab_tiles(nx, ny, nz, sizeof(T))), b(kSlabThreads);
    if (box) hipLaunchKernelGGL((k_slab_post<T, VW, true>), g, b, 0, st, u0, u1, f0, f1, hv, ny, nz, c, sc);
    else hipLaunchKernelGGL((k_slab_post<T, VW, false>), g, b, 0, st, u0, u1, f0, f1, hv, ny, nz, c, sc);
}

#define BRD_SLAB_INST(T)                                                                                             \
    template void launch_slab_down<T>(hipStream_t, bool, T*, const T*, const T*, int, int, int, const LevelCoef<T>&, \
                                      T*, T*, T*, const Scalars*);                                                   \
    template void launch_slab_post<T>(hipStream_t, bool, const T*, T*, const T*, const T*, int, int, int,            \
                                      const LevelCoef<T>&, const Scalars*);
BRD_SLAB_INST(float)
BRD_SLAB_INST(double)
#undef BRD_SLAB_INST

}  // namespace brd
