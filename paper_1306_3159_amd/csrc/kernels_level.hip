// One level of the V-cycle in two launches: pre-smoothing, red residual and restriction
// (k_level_down), red correction and post-smoothing (k_level_up), for alpha I - D L on the
// periodic cell and in a box with homogeneous faces (arXiv:1306.3159 Sec. III.E, eq.
// Helmholtz; the box of Sec. IV.C). The cells' arithmetic is that of the per-step kernels
// (relax, red_resid, restrict_row, the trilinear FMAs), so in the periodic cell the results
// are bitwise theirs.
//
// On levels of up to about 10^6 cells a launch costs more than its bytes, and a V-cycle has
// ten of them a level. Here a work-group owns ty x tz rows (whole in x, so x needs no halo)
// and holds the window of rows that the steps of one launch depend on: every step is done by
// all threads on a region that shrinks towards the tile, neighbouring tiles recompute the
// halo they share. A thread owns K vectors of VW cells of a window row in both colours, with
// their values and right-hand sides in registers; the neighbours' values come from LDS, which
// holds the window's two colours. A row enters a step only if the result depends on it there
// (a distance to the tile, in rows, that the remaining steps can bridge). What bounds it is
// the chain of steps, about 0.5 us each, behind one load of the window.
// Measured (kernel trace, FP32, down / up): 64^3 7.4 / 8.7 us where ten per-step launches took
// about 45; 32^3 5.0 / 5.3 us (an earlier form with an 18^3 window per 8^3 cells and one cell
// per thread and step: 8.7 / 7.8); 128^3 15.3 / 15.6 us.
#include "level.hpp"

namespace brd {

namespace {

constexpr int kDownHalo = 5;  // rows around a tile that the pre-smoothing starts from
constexpr int kUpHalo = 4;    // the same for the post-smoothing
constexpr int kLevelThreads = kFinBlock;

// A vector of a window row: LDS offset, offset in a grid array, and packed: the distance to
// the rows the launch writes (bits 0-7), x parity of its red cells (8), first / last vector
// of the row (9, 10), own row of the tile (11), row in the grid (12; a box's window has rows
// beyond its faces), box: y and z faces (13-15).
struct Item {
    int row;
    unsigned goff;
    int m;
    __device__ __forceinline__ int dist() const { return m & 255; }
    __device__ __forceinline__ int par() const { return (m >> 8) & 1; }
    __device__ __forceinline__ bool first() const { return m & 512; }
    __device__ __forceinline__ bool last() const { return m & 1024; }
    __device__ __forceinline__ bool own() const { return m & 2048; }
    __device__ __forceinline__ bool inside() const { return m & 4096; }
    __device__ __forceinline__ int faces() const { return (m >> 13) & 7; }
};

// The tile a work-group owns: rows y0 .. y0 + tyv - 1 of planes z0 .. z0 + tzv - 1.
struct TileBox {
    int y0, z0, tyv, tzv;
    __device__ __forceinline__ TileBox(const LevelTile& g, unsigned tile, int ny, int nz) {
        y0 = (int)(tile % g.nty) * g.ty;
        z0 = (int)(tile / g.nty) * g.tz;
        tyv = min(g.ty, ny - y0);
        tzv = min(g.tz, nz - z0);
    }
};

// Item `id` of a window with `halo` rows around the tile. core: rows next to the tile that
// count as the tile (1 where the restriction reads the residual's 3 x 3 rows around).
template <int VW, bool BOX>
__device__ __forceinline__ Item level_item(const LevelTile& g, const TileBox& b, int id, int halo, int core, int hx,
                                           int ny, int nz) {
    const int r = (int)__umulhi((unsigned)id, g.mlanes), lane = id - r * g.lanes;
    const int wy_n = g.ty + 2 * halo;
    const int wz = (int)__umulhi((unsigned)r, halo == kDownHalo ? g.mdown : g.mup), wy = r - wz * wy_n;
    const int ry = wy - halo, rz = wz - halo;  // relative to the tile
    const int dy = max(max(-ry, ry - (b.tyv - 1)), core) - core, dz = max(max(-rz, rz - (b.tzv - 1)), core) - core;
    const int yu = b.y0 + ry, zu = b.z0 + rz;
    const int y = modi(yu, ny), z = modi(zu, nz);
    const bool in = !BOX || (yu >= 0 && yu < ny && zu >= 0 && zu < nz);
    const bool own = ry >= 0 && ry < b.tyv && rz >= 0 && rz < b.tzv;
    const int faces = BOX ? (y == 0) + (y + 1 == ny) + (z == 0) + (z + 1 == nz) : 0;
    const int i0 = lane * VW;
    Item it;
    it.row = r * hx + i0;
    it.goff = ((unsigned)z * ny + y) * hx + i0;
    it.m = min(dy + dz, 255) | (((y + z) & 1) << 8) | (lane == 0 ? 512 : 0) | (lane + 1 == g.lanes ? 1024 : 0) |
           (own ? 2048 : 0) | (in ? 4096 : 0) | (faces << 13);
    return it;
}

// Diagonals (or inverse diagonals) of a vector's cells with x parity so; a row outside a box
// gives zeros, which keeps its values zero.
template <typename T, int VW, bool BOX>
__device__ __forceinline__ typename RowVec<T, VW>::type level_diag(const T* tab, const Item& it, int so) {
    typedef typename RowVec<T, VW>::type V;
    if (!BOX) return (V)(tab[0]);
    const T t0 = tab[0], t1 = tab[1], t2 = tab[2], t3 = tab[3];
    const int f = it.faces();
    const T base = it.inside() ? (f == 0 ? t0 : (f == 1 ? t1 : t2)) : (T)0;
    const T edge = it.inside() ? (f == 0 ? t1 : (f == 1 ? t2 : t3)) : (T)0;
    V d = (V)(base);
    if (so == 0 && it.first()) d[0] = edge;
    if (so == 1 && it.last()) d[VW - 1] = edge;
    return d;
}

// Neighbour sums of a vector of cells with x parity so: o the other colour's vector at the
// same place, P that colour in LDS (zstr: offset between window planes).
template <typename T, int VW, bool BOX>
__device__ __forceinline__ typename RowVec<T, VW>::type level_sum(const Item& it, const T* P,
                                                                  typename RowVec<T, VW>::type o, int so, int hx,
                                                                  int zstr) {
    typedef typename RowVec<T, VW>::type V;
    const T* q = P + it.row;
    const V ym = *reinterpret_cast<const V*>(q - hx);
    const V yp = *reinterpret_cast<const V*>(q + hx);
    const V zm = *reinterpret_cast<const V*>(q - zstr);
    const V zp = *reinterpret_cast<const V*>(q + zstr);
    T e = so ? q[it.last() ? VW - hx : VW] : q[it.first() ? hx - 1 : -1];
    if (BOX && (so ? it.last() : it.first())) e = (T)0;
    V nb;
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        const T x = so ? (k + 1 < VW ? o[k + 1] : e) : (k ? o[k - 1] : e);
        nb[k] = ((o[k] + x) + (ym[k] + yp[k])) + (zm[k] + zp[k]);
    }
    return nb;
}

template <typename T, int VW>
__device__ __forceinline__ typename RowVec<T, VW>::type level_relax(typename RowVec<T, VW>::type f, T s,
                                                                    typename RowVec<T, VW>::type nb,
                                                                    typename RowVec<T, VW>::type inv) {
    typename RowVec<T, VW>::type u;
#pragma unroll
    for (int k = 0; k < VW; ++k) u[k] = relax(f[k], s, nb[k], inv[k]);
    return u;
}

// ---------------------------------------------------------------------------
template <typename T, int VW, int K, bool BOX>
__device__ __forceinline__ void level_down(const T* __restrict__ f0, const T* __restrict__ f1, T* __restrict__ ured,
                                           int nx, int ny, int nz, const LevelCoef<T>& c, T* __restrict__ cf0,
                                           T* __restrict__ cf1, T* __restrict__ cu0, const LevelTile& g, unsigned tile,
                                           T* lds) {
    typedef typename RowVec<T, VW>::type V;
    constexpr int H = kDownHalo;
    const int hx = nx >> 1, wy = g.ty + 2 * H, rows = wy * (g.tz + 2 * H), zstr = wy * hx, items = rows * g.lanes;
    const TileBox b(g, tile, ny, nz);
    T* const U0 = lds;
    T* const U1 = lds + rows * hx;
    Item it[K];
    V F0[K], F1[K], u0[K], u1[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int id = (int)threadIdx.x + k * (int)blockDim.x;
        it[k] = level_item<VW, BOX>(g, b, min(id, items - 1), H, 1, hx, ny, nz);
        if (id >= items) it[k].m = 255;
        F0[k] = F1[k] = u0[k] = u1[k] = (V)(T)0;
        if (it[k].dist() <= 4 && it[k].inside()) F0[k] = *reinterpret_cast<const V*>(f0 + it[k].goff);
        if (it[k].dist() <= 3 && it[k].inside()) F1[k] = *reinterpret_cast<const V*>(f1 + it[k].goff);
    }
    // first red sweep from zero
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (it[k].dist() <= 4) {
            const V d = level_diag<T, VW, BOX>(c.inv, it[k], it[k].par());
#pragma unroll
            for (int j = 0; j < VW; ++j) u0[k][j] = relax_zero(F0[k][j], d[j]);
            *reinterpret_cast<V*>(U0 + it[k].row) = u0[k];
        }
    lds_barrier();
    auto black = [&](int dist) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (it[k].dist() <= dist) {
                const int so = it[k].par() ^ 1;
                const V nb = level_sum<T, VW, BOX>(it[k], U0, u0[k], so, hx, zstr);
                u1[k] = level_relax<T, VW>(F1[k], c.s, nb, level_diag<T, VW, BOX>(c.inv, it[k], so));
                *reinterpret_cast<V*>(U1 + it[k].row) = u1[k];
            }
        lds_barrier();
    };
    black(3);
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (it[k].dist() <= 2) {
            const int so = it[k].par();
            const V nb = level_sum<T, VW, BOX>(it[k], U1, u1[k], so, hx, zstr);
            u0[k] = level_relax<T, VW>(F0[k], c.s, nb, level_diag<T, VW, BOX>(c.inv, it[k], so));
            *reinterpret_cast<V*>(U0 + it[k].row) = u0[k];
            if (it[k].own()) *reinterpret_cast<V*>(ured + it[k].goff) = u0[k];
        }
    lds_barrier();
    black(1);
    // red residual, over the red values (their owners keep them)
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (it[k].dist() == 0) {
            const int so = it[k].par();
            const V nb = level_sum<T, VW, BOX>(it[k], U1, u1[k], so, hx, zstr);
            const V d = level_diag<T, VW, BOX>(c.diag, it[k], so);
            V r;
#pragma unroll
            for (int j = 0; j < VW; ++j) r[j] = red_resid(F0[k][j], d[j], u0[k][j], c.s, nb[j]);
            if (BOX && !it[k].inside()) r = (V)(T)0;
            *reinterpret_cast<V*>(U0 + it[k].row) = r;
        }
    lds_barrier();
    // restriction: the four planes of a coarse vector by four threads, then their weighted sum
    const int cty = g.ty >> 1, ctz = g.tz >> 1, nc = cty * ctz * g.lanes;
    const int cx = nx >> 1, cy = ny >> 1, cz = nz >> 1;
    T* const P = U1;
    auto coarse_of = [&](int q, int& i0, int& qy, int& qz) {
        const int r = (int)__umulhi((unsigned)q, g.mlanes);
        i0 = (q - r * g.lanes) * VW;
        qz = r / cty;
        qy = r - qz * cty;
    };
    for (int t = threadIdx.x; t < 4 * nc; t += blockDim.x) {
        const int a = t / nc, q = t - a * nc;
        int i0, qy, qz;
        coarse_of(q, i0, qy, qz);
        const int wz = 2 * qz - 1 + a + H, Y = (b.y0 >> 1) + qy;
        T accb[VW];
#pragma unroll
        for (int k = 0; k < VW; ++k) accb[k] = (T)0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const T* r = U0 + (wz * wy + 2 * qy - 1 + e + H) * hx;
            const int pr = (a + e) & 1;  // red cells of the row (y, z): x = 2i + pr (y0 and z0 are even)
            const V m = *reinterpret_cast<const V*>(r + i0);
            T x = pr ? r[i0 ? i0 - 1 : hx - 1] : r[i0 + VW == hx ? 0 : i0 + VW];
            T wgt = (e == 0 || e == 3) ? (T)0.125 : (T)0.375;
            if (BOX) {
                if (pr ? i0 == 0 : i0 + VW == hx) x = (T)0;
                wgt = level_rweight<T>(e, Y, ny);
            }
            level_restrict_row<T, VW, BOX>(accb, m, x, pr, wgt, i0 == 0, i0 + VW == hx);
        }
#pragma unroll
        for (int k = 0; k < VW; ++k) P[t * VW + k] = accb[k];
    }
    lds_barrier();
    for (int q = threadIdx.x; q < nc; q += blockDim.x) {
        int i0, qy, qz;
        coarse_of(q, i0, qy, qz);
        if (2 * qy >= b.tyv || 2 * qz >= b.tzv) continue;
        const int Y = (b.y0 >> 1) + qy, Z = (b.z0 >> 1) + qz;
        T acc[VW];
#pragma unroll
        for (int k = 0; k < VW; ++k) acc[k] = (T)0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const T wgt = BOX ? level_rweight<T>(a, Z, nz) : ((a == 0 || a == 3) ? (T)0.125 : (T)0.375);
#pragma unroll
            for (int k = 0; k < VW; ++k) acc[k] = fma(wgt, P[(a * nc + q) * VW + k], acc[k]);
        }
        level_coarse_store<T, VW, BOX>(acc, i0, Y, Z, cx, cy, cz, c, cf0, cf1, cu0);
    }
}

// ---------------------------------------------------------------------------
// The raw coarse values a thread needs of one coarse row: its run and the value at each end.
template <typename T, int VW, bool BOX>
__device__ __forceinline__ void level_coarse_row(const T* __restrict__ c0, const T* __restrict__ c1, int J, int K,
                                                 int i0, int cx, int cy, T (&m)[VW], T& l, T& r) {
    const size_t row = ((size_t)K * cy + J) * (cx >> 1);
    const int pc = (J + K) & 1;
    auto at = [&](int X) { return (((X + pc) & 1) ? c1 : c0)[row + (X >> 1)]; };
    typedef T H __attribute__((ext_vector_type(VW / 2)));
    const H a = *reinterpret_cast<const H*>(c0 + row + (i0 >> 1));
    const H b = *reinterpret_cast<const H*>(c1 + row + (i0 >> 1));
#pragma unroll
    for (int d = 0; d < VW; ++d) m[d] = ((d + pc) & 1) ? b[d >> 1] : a[d >> 1];
    if (BOX) {  // clamped: beyond a face the end cell itself (its weight is then zero)
        l = at(i0 ? i0 - 1 : 0);
        r = at(i0 + VW < cx ? i0 + VW : cx - 1);
    } else {
        l = at(i0 ? i0 - 1 : cx - 1);
        r = at(i0 + VW < cx ? i0 + VW : 0);
    }
}

// 3/4 a + 1/4 b with the rounding of tri_add
template <typename T>
__device__ __forceinline__ T level_lerp(T a, T b) {
#pragma clang fp contract(off)
    return fma((T)0.75, a, (T)0.25 * b);
}

// Red correction of a vector in grid row (y, z) added to u: its cells x = 2 (i0 + k) + s.
template <typename T, int VW, bool BOX>
__device__ __forceinline__ typename RowVec<T, VW>::type level_correct(typename RowVec<T, VW>::type u,
                                                                      const T* __restrict__ cu0,
                                                                      const T* __restrict__ cu1, int i0, int y, int z,
                                                                      int s, const Item& it, int cx, int cy, int cz) {
    typedef typename RowVec<T, VW>::type V;
    const int J0 = y >> 1, K0 = z >> 1;
    int J1 = (y & 1) ? J0 + 1 : J0 - 1, K1 = (z & 1) ? K0 + 1 : K0 - 1;
    T b0 = (T)0.75, b1 = (T)0.25, c0 = b0, c1 = b1;
    if (BOX) {
        // beyond a face the coarse ghost is -u of the parent, which then takes 1/2
        if (J1 < 0 || J1 >= cy) J1 = J0, b0 = (T)0.5, b1 = (T)0;
        if (K1 < 0 || K1 >= cz) K1 = K0, c0 = (T)0.5, c1 = (T)0;
    } else {
        J1 = wrapi(J1, cy);
        K1 = wrapi(K1, cz);
    }
    T m[4][VW], l[4], r[4];
    level_coarse_row<T, VW, BOX>(cu0, cu1, J0, K0, i0, cx, cy, m[0], l[0], r[0]);
    level_coarse_row<T, VW, BOX>(cu0, cu1, J1, K0, i0, cx, cy, m[1], l[1], r[1]);
    level_coarse_row<T, VW, BOX>(cu0, cu1, J0, K1, i0, cx, cy, m[2], l[2], r[2]);
    level_coarse_row<T, VW, BOX>(cu0, cu1, J1, K1, i0, cx, cy, m[3], l[3], r[3]);
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        T n[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) n[q] = s ? (k + 1 < VW ? m[q][k + 1] : r[q]) : (k ? m[q][k - 1] : l[q]);
        if (BOX) {
            const bool edge = s ? it.last() && k == VW - 1 : it.first() && k == 0;
            const T a0 = edge ? (T)0.5 : (T)0.75, a1 = edge ? (T)0 : (T)0.25;
            T v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = a0 * m[q][k] + a1 * n[q];
            u[k] += c0 * (b0 * v[0] + b1 * v[1]) + c1 * (b0 * v[2] + b1 * v[3]);
        } else {
            u[k] = tri_add(u[k], m[0][k], n[0], m[1][k], n[1], m[2][k], n[2], m[3][k], n[3]);
        }
    }
    return u;
}

// SWEEPS: 4, or 3 where the caller does the closing red sweep itself (then only black is written)
template <typename T, int VW, int K, bool BOX, int SWEEPS>
__device__ __forceinline__ void level_up(const T* __restrict__ cu0, const T* __restrict__ cu1,
                                         const T* __restrict__ ured, const T* __restrict__ f0,
                                         const T* __restrict__ f1, T* __restrict__ u0g, T* __restrict__ u1g, int nx,
                                         int ny, int nz, const LevelCoef<T>& c, const LevelTile& g, unsigned tile,
                                         T* lds) {
    typedef typename RowVec<T, VW>::type V;
    constexpr int H = kUpHalo, X = SWEEPS == 4 ? 0 : 1;  // one halo row fewer is needed for three sweeps
    const int hx = nx >> 1, wy = g.ty + 2 * H, rows = wy * (g.tz + 2 * H), zstr = wy * hx, items = rows * g.lanes;
    const TileBox b(g, tile, ny, nz);
    T* const U0 = lds;
    T* const U1 = lds + rows * hx;
    Item it[K];
    V F0[K], F1[K], u0[K], u1[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int id = (int)threadIdx.x + k * (int)blockDim.x;
        it[k] = level_item<VW, BOX>(g, b, min(id, items - 1), H, 0, hx, ny, nz);
        if (id >= items) it[k].m = 255;
        F0[k] = F1[k] = u0[k] = u1[k] = (V)(T)0;
        if (it[k].dist() <= 4 - X && it[k].inside()) u0[k] = *reinterpret_cast<const V*>(ured + it[k].goff);
        if (it[k].dist() <= 3 - X && it[k].inside()) F1[k] = *reinterpret_cast<const V*>(f1 + it[k].goff);
        if (it[k].dist() <= 2 - X && it[k].inside()) F0[k] = *reinterpret_cast<const V*>(f0 + it[k].goff);
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (it[k].dist() <= 4 - X) {
            const int row = (int)(it[k].goff / (unsigned)hx), i0 = (int)it[k].goff - row * hx, z = row / ny;
            if (it[k].inside())
                u0[k] = level_correct<T, VW, BOX>(u0[k], cu0, cu1, i0, row - z * ny, z, it[k].par(), it[k], nx >> 1,
                                                  ny >> 1, nz >> 1);
            *reinterpret_cast<V*>(U0 + it[k].row) = u0[k];
        }
    lds_barrier();
    auto black = [&](int dist, bool out) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (it[k].dist() <= dist) {
                const int so = it[k].par() ^ 1;
                const V nb = level_sum<T, VW, BOX>(it[k], U0, u0[k], so, hx, zstr);
                u1[k] = level_relax<T, VW>(F1[k], c.s, nb, level_diag<T, VW, BOX>(c.inv, it[k], so));
                if (!out || SWEEPS == 4) *reinterpret_cast<V*>(U1 + it[k].row) = u1[k];
                if (out && it[k].own()) *reinterpret_cast<V*>(u1g + it[k].goff) = u1[k];
            }
        if (!out || SWEEPS == 4) lds_barrier();
    };
    auto red = [&](int k) {
        const int so = it[k].par();
        const V nb = level_sum<T, VW, BOX>(it[k], U1, u1[k], so, hx, zstr);
        return level_relax<T, VW>(F0[k], c.s, nb, level_diag<T, VW, BOX>(c.inv, it[k], so));
    };
    black(3 - X, false);
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (it[k].dist() <= 2 - X) {
            u0[k] = red(k);
            *reinterpret_cast<V*>(U0 + it[k].row) = u0[k];
        }
    lds_barrier();
    black(1 - X, true);
    if (SWEEPS == 4) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (it[k].own()) *reinterpret_cast<V*>(u0g + it[k].goff) = red(k);
    }
}

constexpr int kLevelK = 4;  // most vectors per thread

}  // namespace

template <typename T, int VW, int K, bool BOX>
__global__ void __launch_bounds__(kLevelThreads) k_level_down(const T* __restrict__ f0, const T* __restrict__ f1,
                                                              T* __restrict__ ured, int nx, int ny, int nz,
                                                              LevelCoef<T> c, T* __restrict__ cf0, T* __restrict__ cf1,
                                                              T* __restrict__ cu0, LevelTile g, const Scalars* sc) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (sc && sc->done) return;
    level_down<T, VW, K, BOX>(f0, f1, ured, nx, ny, nz, c, cf0, cf1, cu0, g, xcd_block(blockIdx.x, gridDim.x),
                              reinterpret_cast<T*>(smem));
}

template <typename T, int VW, int K, bool BOX, int SWEEPS>
__global__ void __launch_bounds__(kLevelThreads) k_level_up(const T* __restrict__ cu0, const T* __restrict__ cu1,
                                                            const T* __restrict__ ured, const T* __restrict__ f0,
                                                            const T* __restrict__ f1, T* __restrict__ u0,
                                                            T* __restrict__ u1, int nx, int ny, int nz, LevelCoef<T> c,
                                                            LevelTile g, const Scalars* sc) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (sc && sc->done) return;
    level_up<T, VW, K, BOX, SWEEPS>(cu0, cu1, ured, f0, f1, u0, u1, nx, ny, nz, c, g,
                                    xcd_block(blockIdx.x, gridDim.x), reinterpret_cast<T*>(smem));
}

namespace {

constexpr size_t kLevelLds = 160 * 1024;

int level_items(const LevelTile& g, int halo) { return (g.ty + 2 * halo) * (g.tz + 2 * halo) * g.lanes; }
size_t level_lds(const LevelTile& g, int hx, size_t esz, int halo) {
    return 2 * (size_t)(g.ty + 2 * halo) * (g.tz + 2 * halo) * hx * esz;
}
unsigned magic(int d) { return (unsigned)(((1ull << 32) + d - 1) / d); }  // umulhi(n, magic(d)) = n / d, n d < 2^32

}  // namespace

// Tile of a level. A window has to fit the threads (kLevelK vectors each) and LDS; a tile of
// 4 x 4 rows recomputes the most halo (12 window rows a tile row against 5 for 8 x 8) but
// gives the most work-groups, so it is taken while they are few enough to run at once and
// larger tiles beyond. With more than 512 work-groups the recomputed halo costs more than the
// launches it saves. One V-cycle in FP32 (us; per-step, 4 x 4, 8 x 4, 8 x 8 on every level):
// 32^3 46, 25, 26, 28; 64^3 84, 40, 42, 47; 72 x 56 x 40 81, 40, 44, 50; 96 x 112 x 80 119,
// 77, 73, 64; 128^3 (8 x 8 does not fit its first level) 122, 107, 86, 91. FP64: 64^3 82, 50,
// 55, 63. Box, FP32: 64^3 86, 50, 52, 58. From 512 tiles of kernels_slab.hip on (two to a CU; 8 MB
// a level) its four launches are faster: 128^3 in FP32 down and up 12.2 + 11.2 us against
// 15.1 + 15.5 here. Around that line (V-cycle in us, two launches on the finest level / tiles), FP32:
// 80 x 112 x 96 59 / 59, 96^3 59 / 60, 112 x 112 x 96 61 / 63 (392 tiles), 128^3 82 / 69; but rows of
// 112 and 128 cells below it, which only the 8 x 4 tile takes: 96 x 96 x 112 77 / 63 (288 tiles),
// 112^3 80 / 67, 112 x 128 x 128 81 / 69. FP64, 8 x 8 and 8 x 4: 80^3 64 / 69, 96^3 74 / 76, 112^3 86 / 88,
// 112 x 128 x 128 91 / 92.
LevelTile level_tile(int nx, int ny, int nz, size_t esz) {
    LevelTile g{};
    const int hx = nx / 2;
    if (hx % 2 || hx < 4) return g;  // a level above another split one has even half-rows
    if (slab_fits(nx, ny, nz, esz) && slab_tiles(nx, ny, nz, esz) >= 512) return g;
    g.vw = esz == 4 && hx % 4 == 0 && hx > 4 ? 4 : 2;
    g.lanes = hx / g.vw;
    const int shapes[3][2] = {{4, 4}, {8, 8}, {8, 4}};
    for (int k = 0; k < 3; ++k) {
        g.ty = shapes[k][0];
        g.tz = shapes[k][1];
        g.nty = (ny + g.ty - 1) / g.ty;
        g.ntz = (nz + g.tz - 1) / g.tz;
        if (g.nty * g.ntz > (k == 0 ? 320 : 512) || level_items(g, kDownHalo) > kLevelK * kLevelThreads ||
            level_lds(g, hx, esz, kDownHalo) > kLevelLds)
            continue;
        g.mlanes = magic(g.lanes);
        g.mdown = magic(g.ty + 2 * kDownHalo);
        g.mup = magic(g.ty + 2 * kUpHalo);
        return g;
    }
    return LevelTile{};
}

template <typename T>
LevelCoef<T> level_coef(double s, double alpha, double s_c, bool box) {
    LevelCoef<T> c;
    c.s = (T)s;
    for (int f = 0; f < 4; ++f) {
        const double d = alpha + s * (6.0 + (box ? f : 0)), dc = alpha + s_c * (6.0 + (box ? f : 0));
        c.diag[f] = (T)d;
        c.inv[f] = (T)(1.0 / d);
        c.invc[f] = (T)(1.0 / dc);
    }
    return c;
}

namespace {

// block size and vectors per thread for a window of `items` vectors
void level_shape(int items, int* threads, int* k) {
    const int t = (items + 63) / 64 * 64;
    *k = 1;
    while (*k * kLevelThreads < t) ++*k;
    *threads = ((items + *k - 1) / *k + 63) / 64 * 64;
}

template <typename F>
hipError_t level_attr(F* fn) {
    return hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLevelLds);
}

template <typename T, int VW, int K>
hipError_t level_attrs() {
    const hipError_t e[] = {level_attr(k_level_down<T, VW, K, false>), level_attr(k_level_down<T, VW, K, true>),
                            level_attr(k_level_up<T, VW, K, false, 4>), level_attr(k_level_up<T, VW, K, true, 4>),
                            level_attr(k_level_up<T, VW, K, false, 3>)};
    for (hipError_t x : e)
        if (x != hipSuccess) return x;
    if constexpr (K < kLevelK) return level_attrs<T, VW, K + 1>();
    return hipSuccess;
}

template <typename T, int VW, int K = 1>
void down_go(hipStream_t st, const LevelTile& g, bool box, int threads, int k, const T* f0, const T* f1, T* ured,
             int nx, int ny, int nz, const LevelCoef<T>& c, T* cf0, T* cf1, T* cu0, const Scalars* sc) {
    if constexpr (K < kLevelK) {
        if (k > K) return down_go<T, VW, K + 1>(st, g, box, threads, k, f0, f1, ured, nx, ny, nz, c, cf0, cf1, cu0, sc);
    }
    const dim3 grid(g.nty * g.ntz), block(threads);
    const size_t lds = level_lds(g, nx / 2, sizeof(T), kDownHalo);
    if (box)
        hipLaunchKernelGGL((k_level_down<T, VW, K, true>), grid, block, lds, st, f0, f1, ured, nx, ny, nz, c, cf0,
                           cf1, cu0, g, sc);
    else
        hipLaunchKernelGGL((k_level_down<T, VW, K, false>), grid, block, lds, st, f0, f1, ured, nx, ny, nz, c, cf0,
                           cf1, cu0, g, sc);
}

template <typename T, int VW, int K = 1>
void up_go(hipStream_t st, const LevelTile& g, bool box, int sweeps, int threads, int k, const T* cu0, const T* cu1,
           const T* ured, const T* f0, const T* f1, T* u0, T* u1, int nx, int ny, int nz, const LevelCoef<T>& c,
           const Scalars* sc) {
    if constexpr (K < kLevelK) {
        if (k > K)
            return up_go<T, VW, K + 1>(st, g, box, sweeps, threads, k, cu0, cu1, ured, f0, f1, u0, u1, nx, ny, nz, c,
                                       sc);
    }
    const dim3 grid(g.nty * g.ntz), block(threads);
    const size_t lds = level_lds(g, nx / 2, sizeof(T), kUpHalo);
    if (box)
        hipLaunchKernelGGL((k_level_up<T, VW, K, true, 4>), grid, block, lds, st, cu0, cu1, ured, f0, f1, u0, u1, nx,
                           ny, nz, c, g, sc);
    else if (sweeps == 3)
        hipLaunchKernelGGL((k_level_up<T, VW, K, false, 3>), grid, block, lds, st, cu0, cu1, ured, f0, f1, u0, u1, nx,
                           ny, nz, c, g, sc);
    else
        hipLaunchKernelGGL((k_level_up<T, VW, K, false, 4>), grid, block, lds, st, cu0, cu1, ured, f0, f1, u0, u1, nx,
                           ny, nz, c, g, sc);
}

}  // namespace

template <typename T>
void launch_level_down(hipStream_t st, const LevelTile& g, bool box, const T* f0, const T* f1, T* ured, int nx, int ny,
                       int nz, const LevelCoef<T>& c, T* cf0, T* cf1, T* cu0, const Scalars* sc) {
    int t, k;
    level_shape(level_items(g, kDownHalo), &t, &k);
    if (g.vw == 2) down_go<T, 2>(st, g, box, t, k, f0, f1, ured, nx, ny, nz, c, cf0, cf1, cu0, sc);
    else if constexpr (sizeof(T) == 4) down_go<T, 4>(st, g, box, t, k, f0, f1, ured, nx, ny, nz, c, cf0, cf1, cu0, sc);
}

template <typename T>
void launch_level_up(hipStream_t st, const LevelTile& g, bool box, int sweeps, const T* cu0, const T* cu1,
                     const T* ured, const T* f0, const T* f1, T* u0, T* u1, int nx, int ny, int nz,
                     const LevelCoef<T>& c, const Scalars* sc) {
    int t, k;
    level_shape(level_items(g, kUpHalo), &t, &k);
    if (g.vw == 2) up_go<T, 2>(st, g, box, sweeps, t, k, cu0, cu1, ured, f0, f1, u0, u1, nx, ny, nz, c, sc);
    else if constexpr (sizeof(T) == 4)
        up_go<T, 4>(st, g, box, sweeps, t, k, cu0, cu1, ured, f0, f1, u0, u1, nx, ny, nz, c, sc);
}

template <typename T>
hipError_t level_set_lds() {
    hipError_t e = level_attrs<T, 2, 1>();
    if constexpr (sizeof(T) == 4)
        if (e == hipSuccess) e = level_attrs<T, 4, 1>();
    return e;
}

#define BRD_LEVEL_INST(T)                                                                                            \
    template LevelCoef<T> level_coef<T>(double, double, double, bool);                                               \
    template void launch_level_down<T>(hipStream_t, const LevelTile&, bool, const T*, const T*, T*, int, int, int,   \
                                       const LevelCoef<T>&, T*, T*, T*, const Scalars*);                             \
    template void launch_level_up<T>(hipStream_t, const LevelTile&, bool, int, const T*, const T*, const T*,         \
                                     const T*, const T*, T*, T*, int, int, int, const LevelCoef<T>&, const Scalars*); \
    template hipError_t level_set_lds<T>();
BRD_LEVEL_INST(float)
BRD_LEVEL_INST(double)
#undef BRD_LEVEL_INST

}  // namespace brd
