// Lattice path of the Uzawa multigrid (gfx950): meshes of Kuhn macros tile
// their bounding box, so every level is one structured grid of lattice
// vertices.  The solver's cycles run on vectors over that grid instead of the
// per-macro layout of the ABI; hhg_solve, hhg_vcycle and hhg_fmg convert at
// their ends.  There are no copies of interface vertices, no mirror and no
// index tables on the volume path: every tap's address follows from the
// vertex's by adding one of three per-lane offsets and two uniform strides.
//
// Layout of a field: rows (y, z) of RS values, each split by x mod 4 into four
// sub-rows of Qp entries in the order 0, 2, 1, 3, so that the vertices of one
// parity (and of one colour) of a row are contiguous:
//   vertex (x, y, z) at (z ny + y) RS + slot(x & 3) Qp + (x >> 2).
//
// Work.  Vertices inside the box ("interior": 1 <= x <= nx - 2 and so on) are
// taken by row lanes, vertices on its surface by boundary lanes, which come
// first in every launch.  Interior rows of B and B^T do not depend on the
// viscosity, and with one viscosity for all macros (KIND 0) those of A and C
// are constants too; otherwise (KIND 1) a vertex's axis coefficients of A and
// C come from a record that its cell and the order of its fractional
// coordinates name.  Surface vertices read whole records.
//
// Measured against the per-macro kernels on 17 M vertices, FP64, red-black: an
// Uzawa step took 527 (f - B^T p with the red update) + 2 x 240 + 433 + 86 us and
// takes 3 x 176 + 265 + 61 us; the residual 679 and 655 us, restriction 258 and
// 170, prolongation 431 and 248.  A solve pays the conversions at its ends, 0.71 ms
// each.  Below 2 M vertices a launch takes 3 to 10 us whatever it computes: there
// the gain is in launches (no f - B^T p pass, the visits) and in shorter chains of
// dependent loads (no tile, neighbour and copy tables).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hhg_internal.hpp"

namespace hhg {

// surface records (global tap order) and axis records
constexpr int LR_A = 0, LR_C = 15, LR_B = 30, LR_BT = 75, LR_INVA = 120, LR_INVC = 121, LR_MASS = 122,
              LR_SIZE = 124;
constexpr int LX_A = 0, LX_INVA = 6, LX_C = 8, LX_C0 = 14, LX_INVC = 15, LX_A0 = 7, LX_SIZE = 16;
constexpr int LPAT = 216;   // record patterns per cell
// B and B^T rows by surface class (which faces of the box hold the vertex):
// they do not depend on the viscosity
constexpr int LC_B = 0, LC_BT = 45, LC_SIZE = 90;

template <typename T>
struct Lat {
    int nx, ny, nz, n, sh;      // vertices per axis, 2^R, R
    int Qi;                     // interior quads per row: (nx - 1) / 4
    int Qp, RS, ZS;             // sub-row, row and plane strides
    int cx, cy;                 // cells of the box per x and y
    int order;                  // workgroup order (opts.block_order)
    size_t len;                 // values per field
    const int* rid;             // [(cx+1)(cy+1)(cz+1) LPAT] record of a vertex
    const T* rec;               // [nrec][LR_SIZE]
    const T* axr;               // [nrec][LX_SIZE]
    const unsigned char* rdir;  // [nrec] 1: velocity Dirichlet
    const T* cls;               // [27][LC_SIZE]
    // interior constants: axis pairs of A and C (KIND 0), B^T_k over the seven
    // opposite pairs (+d minus -d; B_k is its negative), lumped mass
    T a[3], inva, a0, c[3], invc, c0, bt[3][7], mass;
};

// Surface lanes of a launch: faces z0, z1, y0, y1, x0, x1 in that order, each
// vertex on the first face that holds it; beg[f] the first lane of face f
// (empty when the launch leaves the face out).
struct LatSurf {
    int beg[7];
};

// the global directions +d of the seven pairs
__host__ __device__ __forceinline__ void lat_pair(int q, int* dx, int* dy, int* dz) {
    // x, y, z, xy, yz, xz, xyz
    const int m[7] = {1, 2, 4, 3, 6, 5, 7};
    *dx = m[q] & 1;
    *dy = m[q] >> 1 & 1;
    *dz = m[q] >> 2;
}

__host__ __device__ __forceinline__ int lat_slot(int s) { return ((s & 1) << 1) | (s >> 1); }

template <typename T>
__host__ __device__ __forceinline__ int lat_at(const Lat<T>& L, int x, int y, int z) {
    return (z * L.ny + y) * L.RS + lat_slot(x & 3) * L.Qp + (x >> 2);
}

// Record index of vertex (x, y, z): its cell (floor), which fractional
// coordinates vanish, and how the fractional coordinates compare.
template <typename T>
__host__ __device__ __forceinline__ int lat_rid_index(const Lat<T>& L, int x, int y, int z) {
    const int m = L.n - 1, fx = x & m, fy = y & m, fz = z & m;
    const int cell = ((z >> L.sh) * (L.cy + 1) + (y >> L.sh)) * (L.cx + 1) + (x >> L.sh);
    const int a = (fx > fy) - (fx < fy) + 1, b = (fy > fz) - (fy < fz) + 1, c = (fx > fz) - (fx < fz) + 1;
    return cell * LPAT + ((a * 3 + b) * 3 + c) * 8 + (fx == 0 ? 1 : 0) + (fy == 0 ? 2 : 0) +
           (fz == 0 ? 4 : 0);
}

template <typename T>
__host__ __device__ __forceinline__ int lat_class(const Lat<T>& L, int x, int y, int z) {
    return (x == 0 ? 0 : x == L.nx - 1 ? 2 : 1) + 3 * (y == 0 ? 0 : y == L.ny - 1 ? 2 : 1) +
           9 * (z == 0 ? 0 : z == L.nz - 1 ? 2 : 1);
}

// item / d for items below 2^21 (host-checked), inv = 1 / d
__host__ __device__ __forceinline__ int lat_div(int item, float inv) {
    return (int)(((float)item + 0.5f) * inv);
}

// smallest r with r d >= item
__host__ __device__ __forceinline__ int lat_div_up(int item, float inv) {
    return item <= 0 ? 0 : lat_div(item - 1, inv) + 1;
}

// Tiles of a volume launch: `per` blocks of bs lanes cover the interior rows of
// a plane.  The planes are cut into eight slabs of ZB, one per XCD (workgroup b
// runs on XCD b mod 8); inside a slab, G blocks of a plane (about 2048 lanes)
// are followed by the same rows of the next plane, so that the rows y +- 1 and
// z +- 1 of a tile are still in its XCD's L2.  Measured at 8 refinements (17 M
// vertices, FP64): plane by plane the velocity sweep fetched twice its bytes.
struct LatGrid {
    int per, G, NG, ZB, total, bs;
    int side, SB;                   // lanes per row on the x faces, their blocks in a group
    float inv_zg, inv_g, inv_row;   // 1 / (ZB (G + SB)), 1 / (G + SB), 1 / (lanes of a row)
};
// lanes: row lanes of a plane; side: lanes per row that also take the row's two
// ends on the faces x = 0 and x = nx - 1 (0: a launch without them).  These read
// the lines of the volume rows (a vertex needs one or two entries of each), so
// they go ahead of the rows of their group, in blocks of their own, and share
// the lines in L2: as part of the surface lanes the two faces fetched them again.
__host__ __device__ __forceinline__ LatGrid lat_grid(int lanes, int rows, int planes, int bs, int side = 0) {
    LatGrid g;
    const int per = (lanes + bs - 1) / bs;
    g.inv_row = (float)rows / (float)lanes;
    g.bs = bs;
    g.per = per;
    g.NG = (per + 7) / 8;
    g.G = (per + g.NG - 1) / g.NG;
    g.ZB = (planes + 7) / 8;
    const int row = lanes / rows, gl = g.G * bs;
    const int most = gl % row == 0 ? gl / row : gl / row + 1;   // rows that begin in a group
    g.side = side;
    g.SB = ((most < rows ? most : rows) * side + bs - 1) / bs;
    g.total = 8 * g.NG * g.ZB * (g.G + g.SB);
    g.inv_zg = 1.0f / (float)(g.ZB * (g.G + g.SB));
    g.inv_g = 1.0f / (float)(g.G + g.SB);
    return g;
}
struct LatTile {
    int t;          // natural index (partial sums)
    int z, part;    // interior plane and block of the plane
    int end;        // >= 0: block of the x faces beside group `part`
    bool ok;
};
__host__ __device__ __forceinline__ LatTile lat_tile(const LatGrid& g, int planes, int v, int order) {
    const int zg = g.ZB * (g.G + g.SB), slab = g.NG * zg;
    LatTile T;
    int zb, i;
    if (order == 1) {
        zb = v & 7;
        i = v >> 3;
        T.t = zb * slab + i;
    } else {
        T.t = order == 2 ? g.total - 1 - v : v;
        zb = T.t / slab;
        i = T.t - zb * slab;
    }
    const int gp = lat_div(i, g.inv_zg), r = i - gp * zg, zi = lat_div(r, g.inv_g);
    T.z = zb * g.ZB + zi;
    const int w = r - zi * (g.G + g.SB);
    T.end = w < g.SB ? w : -1;
    T.part = w < g.SB ? gp : gp * g.G + (w - g.SB);
    T.ok = T.z < planes && (w < g.SB || T.part < g.per);
    return T;
}
// vertex of lane idx of the x-face blocks of a group: rows that begin in it, two
// ends each (side 8: the ends of the four rows of a 2 x 2 block)
__host__ __device__ __forceinline__ bool lat_end_lane(const LatGrid& g, const LatTile& t, int rows, int nx, int ny,
                                                      int nz, int lane, int* x, int* y, int* z) {
    const int idx = t.end * g.bs + lane, lg = g.side == 8 ? 3 : 1, gl = g.G * g.bs;
    const int row0 = lat_div_up(t.part * gl, g.inv_row), row1 = lat_div_up((t.part + 1) * gl, g.inv_row);
    const int row = row0 + (idx >> lg);
    *x = idx & 1 ? nx - 1 : 0;
    if (g.side == 8) {
        *y = 2 * row + 1 + (idx >> 1 & 1);
        *z = 2 * t.z + 1 + (idx >> 2 & 1);
    } else {
        *y = row + 1;
        *z = t.z + 1;
    }
    return row < row1 && row < rows && *y <= ny - 2 && *z <= nz - 2;
}

// Interior row lanes of a colour launch: NC = 2 the parity col (0 or 1) of
// x + y + z, NC = 1 the colour col = (x + y + z) mod 4.  A lane takes the
// vertices x and x + 4 of one sub-row s, at entries q and q + 1.
struct LatPair {
    int y, z, s, q;
    bool ok;
};
template <typename T>
__host__ __device__ __forceinline__ int lat_pair_lanes(const Lat<T>& L, int NC) {
    return (L.ny - 2) * (NC * (L.Qi >> 1));   // per plane
}
template <int NC, typename T>
__host__ __device__ __forceinline__ LatPair lat_pair_lane(const Lat<T>& L, int col, const LatGrid& tg,
                                                          const LatTile& tile, int lane) {
    LatPair P;
    const int half = L.Qi >> 1, lpr = NC * half;
    const int item = tile.part * tg.bs + lane;
    const int row = lat_div(item, tg.inv_row), li = item - row * lpr;
    P.z = tile.z + 1;
    P.y = row + 1;
    P.ok = row < L.ny - 2;
    const int s0 = (col + 8 * (L.ny + L.nz) - P.y - P.z) & (NC == 2 ? 1 : 3);
    const int e = NC == 2 && li >= half ? 1 : 0;
    P.s = s0 + 2 * e;
    P.q = 2 * (li - e * half);
    return P;
}

// Interior row lanes of a full pass: a lane takes the quad x = 4 q .. 4 q + 3.
template <typename T>
__host__ __device__ __forceinline__ int lat_quad_lanes(const Lat<T>& L) {
    return (L.ny - 2) * L.Qi;   // per plane
}
template <typename T>
__host__ __device__ __forceinline__ LatPair lat_quad_lane(const Lat<T>& L, const LatGrid& tg,
                                                          const LatTile& tile, int lane) {
    LatPair P;
    const int item = tile.part * tg.bs + lane;
    const int row = lat_div(item, tg.inv_row);
    P.z = tile.z + 1;
    P.y = row + 1;
    P.s = 0;
    P.q = item - row * L.Qi;
    P.ok = row < L.ny - 2;
    return P;
}

// Surface lane -> vertex.  S = 1: every vertex; S = 2: parity col; S = 4:
// colour col.
template <typename T>
__host__ __device__ __forceinline__ int lat_face_lanes(const Lat<T>& L, int f, int S) {
    const int xs = (L.nx + S - 1) / S, ys = (L.ny + S - 1) / S;
    return f < 2 ? xs * L.ny : f < 4 ? xs * (L.nz - 2) : ys * (L.nz - 2);
}
template <typename T>
__host__ __device__ __forceinline__ bool lat_surf_lane(const Lat<T>& L, const LatSurf& B, int S, int col,
                                                       int idx, int* x, int* y, int* z) {
    if (idx >= B.beg[6]) return false;
    int f = 0;
    while (idx >= B.beg[f + 1]) ++f;
    const int i = idx - B.beg[f], big = 8 * (L.nx + L.ny + L.nz), m = S - 1;
    if (f < 4) {
        const int xs = (L.nx + S - 1) / S, r = i / xs;
        *y = f < 2 ? r : f == 2 ? 0 : L.ny - 1;
        *z = f >= 2 ? r + 1 : f == 0 ? 0 : L.nz - 1;
        *x = S * (i - r * xs) + ((col + big - *y - *z) & m);
        return *x < L.nx;
    }
    const int ys = (L.ny + S - 1) / S, r = i / ys;
    *x = f == 4 ? 0 : L.nx - 1;
    *z = r + 1;
    *y = S * (i - r * ys) + ((col + big - *x - *z) & m);
    return *y >= 1 && *y <= L.ny - 2;
}

// Whether the lane has a vertex of the box's surface: the blocks before the tiles
// (*tile is left alone) or a tile's x faces; *ok: it has one.  Uniform per block.
template <typename T>
__device__ __forceinline__ bool lat_surf_work(const Lat<T>& L, const LatSurf& B, int sb, const LatGrid& tg, int rows,
                                              int planes, LatTile* tile, bool* ok, int* x, int* y, int* z) {
    if ((int)blockIdx.x < sb) {
        *ok = lat_surf_lane(L, B, 1, 0, (int)blockIdx.x * tg.bs + (int)threadIdx.x, x, y, z);
        return true;
    }
    *tile = lat_tile(tg, planes, (int)blockIdx.x - sb, L.order);
    if (tile->end < 0) return false;
    *ok = tile->ok && lat_end_lane(tg, *tile, rows, L.nx, L.ny, L.nz, threadIdx.x, x, y, z);
    return true;
}

// The 14 neighbour addresses of a surface vertex in the global tap order; a
// direction that leaves the box gets the vertex itself (its coefficients are 0).
template <typename T>
__host__ __device__ __forceinline__ void lat_taps(const Lat<T>& L, int x, int y, int z, int nb[15]) {
    const int self = lat_at(L, x, y, z);
    nb[0] = self;
    for (int q = 0; q < 7; ++q) {
        int dx, dy, dz;
        lat_pair(q, &dx, &dy, &dz);
        const bool up = x + dx < L.nx && y + dy < L.ny && z + dz < L.nz;
        const bool dn = x - dx >= 0 && y - dy >= 0 && z - dz >= 0;
        nb[2 * q + 1] = up ? lat_at(L, x + dx, y + dy, z + dz) : self;
        nb[2 * q + 2] = dn ? lat_at(L, x - dx, y - dy, z - dz) : self;
    }
}

// Pairs of consecutive entries; loads need only the element's alignment.
template <typename T>
struct V2 {
    typedef T type __attribute__((ext_vector_type(2)));
    typedef T load __attribute__((ext_vector_type(2), aligned(sizeof(T))));
};
// uniform field base + 32-bit element offset (below 2^29, host-checked)
template <typename T>
__device__ __forceinline__ typename V2<T>::type ld2(const T* __restrict__ base, int at) {
    return *reinterpret_cast<const typename V2<T>::load*>(reinterpret_cast<const char*>(base) +
                                                           (uint32_t)at * (uint32_t)sizeof(T));
}
template <typename T>
__device__ __forceinline__ T ld1(const T* __restrict__ base, int at) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) +
                                       (uint32_t)at * (uint32_t)sizeof(T));
}
template <typename T>
__device__ __forceinline__ void st1(T* __restrict__ base, int at, T v) {
    *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + (uint32_t)at * (uint32_t)sizeof(T)) = v;
}

// Offsets from entry q of sub-row s to the entries of x + 1 and x - 1.
__host__ __device__ __forceinline__ void lat_x_offsets(int s, int Qp, int* P, int* M) {
    const int here = lat_slot(s);
    *P = (lat_slot((s + 1) & 3) - here) * Qp + (s == 3 ? 1 : 0);
    *M = (lat_slot((s + 3) & 3) - here) * Qp - (s == 0 ? 1 : 0);
}

// Surface lanes of the velocity launches: lane 3 i + k takes component k of vertex
// i (its neighbour lanes read the same pressure taps).  Bound by latency, that of the
// record index and then the record: the rows of B^T come from the vertex's class
// instead, beside it, and every load is issued before the first use.  With a lane
// per vertex that took the components one after another (its stores kept the next
// one's loads back) a launch waited on these lanes: four cycles on 65 x 257 x 65
// vertices with outflow through a side of 257 x 65, colour order, FP64, 11.0 -> 7.9
// ms; 129^3 vertices, outflow, 12.5 -> 9.8 ms.
template <typename T, bool PZ>
__device__ __forceinline__ void lat_vel_surface(const Lat<T>& L, const LatSurf& B, int S, int col, int idx,
                                                const T* __restrict__ b, T* __restrict__ x) {
    const size_t len = L.len;
    const int i = idx / 3, k = idx - 3 * i;
    int X, Y, Z;
    if (!lat_surf_lane(L, B, S, col, i, &X, &Y, &Z)) return;
    const int id = L.rid[lat_rid_index(L, X, Y, Z)];
    int nb[15];
    lat_taps(L, X, Y, Z, nb);
    T* __restrict__ u = x + k * len;
    T acc = b[k * len + nb[0]], v[15], w[15], n[7], a[7];
    if (!PZ) {
        const T* __restrict__ p = x + 3 * len;
        const T* __restrict__ cr = L.cls + (size_t)lat_class(L, X, Y, Z) * LC_SIZE + LC_BT + 15 * k;
#pragma unroll
        for (int g = 0; g < 15; ++g) v[g] = p[nb[g]];
#pragma unroll
        for (int g = 0; g < 15; ++g) w[g] = cr[g];
    }
#pragma unroll
    for (int g = 1; g < 7; ++g) n[g] = u[nb[g]];
    const bool dir = L.rdir[id] != 0;
    const T* __restrict__ r = L.axr + (size_t)id * LX_SIZE;
#pragma unroll
    for (int g = 0; g < 7; ++g) a[g] = r[LX_A + g];   // the six taps, 1 / centre
    __builtin_amdgcn_sched_barrier(0);
    if (dir) return;
    if (!PZ)
#pragma unroll
        for (int g = 0; g < 15; ++g) acc -= w[g] * v[g];
#pragma unroll
    for (int g = 1; g < 7; ++g) acc -= a[g - 1] * n[g];
    u[nb[0]] = acc * a[LX_INVA];
}
// The surface lanes of the other passes: whole records, taps by address.
template <typename T>
__device__ __forceinline__ void lat_bp_surface(const Lat<T>& L, int X, int Y, int Z, int cm, int col,
                                               const T* __restrict__ g, T* __restrict__ x,
                                               T* __restrict__ sx, T omega, int all) {
    const size_t len = L.len;
    T* __restrict__ p = x + 3 * len;
    const T* __restrict__ r = L.rec + (size_t)L.rid[lat_rid_index(L, X, Y, Z)] * LR_SIZE;
    int nb[15];
    lat_taps(L, X, Y, Z, nb);
    T s = -g[nb[0]];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int t = 0; t < 15; ++t) s += r[LR_B + 15 * k + t] * x[k * len + nb[t]];
    if (((X + Y + Z) & cm) == col) {
        T cp = T(0);
#pragma unroll
        for (int t = 0; t < 7; ++t) cp += r[LR_C + t] * p[nb[t]];
        p[nb[0]] += omega * (s - cp) * r[LR_INVC];
        if (!all) return;
    }
    sx[nb[0]] = s;
}
// returns the lane's sum of r^2
template <typename T, bool WR, bool NRM, bool AP>
__device__ __forceinline__ double lat_res_surface(const Lat<T>& L, int X, int Y, int Z,
                                                  const T* __restrict__ b, const T* __restrict__ x,
                                                  T* __restrict__ r) {
    const size_t len = L.len;
    const T* __restrict__ p = x + 3 * len;
    double acc = 0.0;
    const int id = L.rid[lat_rid_index(L, X, Y, Z)];
    const T* __restrict__ rc = L.rec + (size_t)id * LR_SIZE;
    int nb[15];
    lat_taps(L, X, Y, Z, nb);
    T v = AP ? T(0) : b[3 * len + nb[0]];
#pragma unroll
    for (int t = 0; t < 7; ++t) v += rc[LR_C + t] * p[nb[t]];
#pragma unroll 1
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int t = 0; t < 15; ++t) v -= rc[LR_B + 15 * k + t] * x[k * len + nb[t]];
    if (WR) r[3 * len + nb[0]] = AP ? -v : v;
    if (NRM) acc += (double)v * (double)v;
    const bool dir = L.rdir[id] != 0;
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        T w = T(0);
        if (!dir) {
            w = AP ? T(0) : b[k * len + nb[0]];
#pragma unroll
            for (int t = 0; t < 15; ++t) w -= rc[LR_BT + 15 * k + t] * p[nb[t]];
            for (int t = 0; t < 7; ++t) w -= rc[LR_A + t] * x[k * len + nb[t]];
        }
        if (WR) r[k * len + nb[0]] = AP ? -w : w;
        if (NRM) acc += (double)w * (double)w;
    }
    return acc;
}

// ---------------------------------------------------------------------------
// Velocity sweep of one parity or colour (Section 3.5): u_k <- (f_k - (B^T p)_k
// - sum A u_k) / A_xx.  The B^T p rows are formed on the fly from p instead of
// being stored by a pass of their own: a parity launch then moves 5.5 values
// per vertex (p, half of u read, of f read, of u written) instead of 4.5, and
// the 10 values of that pass are gone.  PZ: p = 0 (the iterate starts at 0).
// A lane takes two vertices of a row that are four apart: their taps are pairs of
// consecutive entries.  Bound by L2 requests: 17 M vertices, FP64 209 us (3.6 TB/s
// of its 5.5 values), 2.1 M vertices 19.2 us, a level of up to 36 thousand 3.4 us
// (launch and two dependent loads).
// ---------------------------------------------------------------------------
template <typename T, int KIND, int NC, bool PZ>
__global__ void __launch_bounds__(256) k_lat_vel(Lat<T> L, LatSurf B, int col, int sb, LatGrid tg,
                                                 const T* __restrict__ b, T* __restrict__ x) {
    const size_t len = L.len;
    const T* __restrict__ p = x + 3 * len;
    if ((int)blockIdx.x < sb) {
        lat_vel_surface<T, PZ>(L, B, 4 / NC, col, (int)blockIdx.x * tg.bs + (int)threadIdx.x, b, x);
        return;
    }
    const LatTile tile = lat_tile(tg, L.nz - 2, (int)blockIdx.x - sb, L.order);
    if (!tile.ok) return;
    const LatPair P = lat_pair_lane<NC>(L, col, tg, tile, threadIdx.x);
    if (!P.ok) return;
    typedef typename V2<T>::type v2;
    const int at = (P.z * L.ny + P.y) * L.RS + lat_slot(P.s) * L.Qp + P.q;
    int xp, xm;
    lat_x_offsets(P.s, L.Qp, &xp, &xm);
    xp += at;
    xm += at;
    const int RS = L.RS, ZS = L.ZS;
    v2 t[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) t[k] = ld2(b + k * len, at);
    if (!PZ) {
        v2 d[7];
        d[0] = ld2(p, xp) - ld2(p, xm);
        d[1] = ld2(p, at + RS) - ld2(p, at - RS);
        d[2] = ld2(p, at + ZS) - ld2(p, at - ZS);
        d[3] = ld2(p, xp + RS) - ld2(p, xm - RS);
        d[4] = ld2(p, at + RS + ZS) - ld2(p, at - RS - ZS);
        d[5] = ld2(p, xp + ZS) - ld2(p, xm - ZS);
        d[6] = ld2(p, xp + RS + ZS) - ld2(p, xm - RS - ZS);
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int q = 0; q < 7; ++q) t[k] -= L.bt[k][q] * d[q];
    }
    const bool first = P.s != 0 || P.q != 0;   // x = 0 is a surface vertex
    v2 w[6], inv;
    if (KIND == 0) {
        inv = v2{L.inva, L.inva};
    } else {
        const int X = 4 * P.q + P.s;
        const T* ra = L.axr + (size_t)L.rid[lat_rid_index(L, X, P.y, P.z)] * LX_SIZE + LX_A;
        const T* rb = L.axr + (size_t)L.rid[lat_rid_index(L, X + 4, P.y, P.z)] * LX_SIZE + LX_A;
#pragma unroll
        for (int g = 0; g < 6; ++g) w[g] = v2{ra[g], rb[g]};
        inv = v2{ra[LX_INVA], rb[LX_INVA]};
    }
    v2 res[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const T* __restrict__ u = x + k * len;
        if (KIND == 0) {
            res[k] = t[k] - L.a[0] * (ld2(u, xp) + ld2(u, xm)) - L.a[1] * (ld2(u, at + RS) + ld2(u, at - RS)) -
                     L.a[2] * (ld2(u, at + ZS) + ld2(u, at - ZS));
        } else {
            res[k] = t[k] - w[0] * ld2(u, xp) - w[1] * ld2(u, xm) - w[2] * ld2(u, at + RS) -
                     w[3] * ld2(u, at - RS) - w[4] * ld2(u, at + ZS) - w[5] * ld2(u, at - ZS);
        }
        res[k] *= inv;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        T* __restrict__ u = x + k * len + at;
        if (first)
            *reinterpret_cast<typename V2<T>::load*>(u) = res[k];
        else
            u[1] = res[k][1];
    }
}

// ---------------------------------------------------------------------------
// Windows of a full pass: the seven rows around a quad, entries x = 4q - 1 ..
// 4q + 4 at v[row][0..5] (rows ahead hold 1..5, rows behind 0..4).
// ---------------------------------------------------------------------------
template <typename T>
struct LatWin {
    T v[7][6];
};
// row 0 (0,0); 1, 2 (+-y); 3, 4 (+-z); 5, 6 +-(y+z)
template <typename T>
__device__ __forceinline__ void lat_window(const Lat<T>& L, const T* __restrict__ f, int at, LatWin<T>& W) {
    const int Qp = L.Qp;
#pragma unroll
    for (int r = 0; r < 7; ++r) {
        const int o = r == 0 ? 0 : r == 1 ? L.RS : r == 2 ? -L.RS : r == 3 ? L.ZS : r == 4 ? -L.ZS
                    : r == 5 ? L.RS + L.ZS : -L.RS - L.ZS;
        const int a = at + o;
        // sub-rows 0, 2, 1, 3 at a, a + Qp, a + 2 Qp, a + 3 Qp
        W.v[r][2] = ld1(f, a + 2 * Qp);
        W.v[r][3] = ld1(f, a + Qp);
        if (r == 0 || (r & 1)) {
            const typename V2<T>::type e = ld2(f, a);
            W.v[r][1] = e[0];
            W.v[r][5] = e[1];
        } else {
            W.v[r][1] = ld1(f, a);
        }
        if (r == 0 || !(r & 1)) {
            const typename V2<T>::type e = ld2(f, a + 3 * Qp - 1);
            W.v[r][0] = e[0];
            W.v[r][4] = e[1];
        } else {
            W.v[r][4] = ld1(f, a + 3 * Qp);
        }
    }
}
// +d minus -d over the seven pairs at vertex j of the quad
template <typename T>
__device__ __forceinline__ void lat_diffs(const LatWin<T>& W, int j, T d[7]) {
    d[0] = W.v[0][j + 2] - W.v[0][j];
    d[1] = W.v[1][j + 1] - W.v[2][j + 1];
    d[2] = W.v[3][j + 1] - W.v[4][j + 1];
    d[3] = W.v[1][j + 2] - W.v[2][j];
    d[4] = W.v[5][j + 1] - W.v[6][j + 1];
    d[5] = W.v[3][j + 2] - W.v[4][j];
    d[6] = W.v[5][j + 2] - W.v[6][j];
}
// sub-row offset of vertex j of a quad
__host__ __device__ __forceinline__ int lat_sub(int j, int Qp) { return lat_slot(j) * Qp; }

// ---------------------------------------------------------------------------
// s = B u - g on every pressure row with the pressure update of the colour set
// col: p += omega (s - C p) / C_xx on its vertices.  s is stored for the
// vertices that a later sweep relaxes (all of them with ALL).  A lane takes a quad
// of consecutive vertices, one window of 36 values per field.  Bound by L2
// requests, a quarter of them by the box's surface, whose lanes read 52 taps each
// (2.1 M vertices, FP64: 40 us, without the surface 29); 17 M vertices 340 us.
// ---------------------------------------------------------------------------
template <typename T, int KIND, int NC>
__global__ void __launch_bounds__(256) k_lat_bp(Lat<T> L, LatSurf B, int col, int sb, LatGrid tg,
                                                const T* __restrict__ b, T* __restrict__ x,
                                                T* __restrict__ sx, T omega, int all) {
    const size_t len = L.len;
    T* __restrict__ p = x + 3 * len;
    const T* __restrict__ g = b + 3 * len;
    const int cm = NC == 2 ? 1 : 3;
    LatTile tile;
    bool ok;
    int X, Y, Z;
    if (lat_surf_work(L, B, sb, tg, L.ny - 2, L.nz - 2, &tile, &ok, &X, &Y, &Z)) {
        if (ok) lat_bp_surface<T>(L, X, Y, Z, cm, col, g, x, sx, omega, all);
        return;
    }
    if (!tile.ok) return;
    const LatPair P = lat_quad_lane(L, tg, tile, threadIdx.x);
    if (!P.ok) return;
    const int at = (P.z * L.ny + P.y) * L.RS + P.q, Qp = L.Qp;
    T s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = -ld1(g, at + lat_sub(j, Qp));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        LatWin<T> W;
        lat_window(L, x + k * len, at, W);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            T d[7];
            lat_diffs(W, j, d);
#pragma unroll
            for (int q = 0; q < 7; ++q) s[j] -= L.bt[k][q] * d[q];
        }
    }
    const int s0 = (col + 8 * (L.ny + L.nz) - P.y - P.z) & cm;
#pragma unroll
    for (int e = 0; e < NC; ++e) {
        const int j = s0 + 2 * e;
        if (j == 0 && P.q == 0) continue;   // x = 0
        const int a = at + lat_sub(j, Qp);
        int xp, xm;
        lat_x_offsets(j, Qp, &xp, &xm);
        const T p0 = ld1(p, a);
        const T xa = ld1(p, a + xp), xb = ld1(p, a + xm), ya = ld1(p, a + L.RS), yb = ld1(p, a - L.RS),
                za = ld1(p, a + L.ZS), zb = ld1(p, a - L.ZS);
        T cp, inv;
        if (KIND == 0) {
            cp = L.c0 * p0 + L.c[0] * (xa + xb) + L.c[1] * (ya + yb) + L.c[2] * (za + zb);
            inv = L.invc;
        } else {
            const T* r = L.axr + (size_t)L.rid[lat_rid_index(L, 4 * P.q + j, P.y, P.z)] * LX_SIZE;
            cp = r[LX_C0] * p0 + r[LX_C] * xa + r[LX_C + 1] * xb + r[LX_C + 2] * ya + r[LX_C + 3] * yb +
                 r[LX_C + 4] * za + r[LX_C + 5] * zb;
            inv = r[LX_INVC];
        }
        const T sj = NC == 2 ? (e == 0 ? (s0 ? s[1] : s[0]) : (s0 ? s[3] : s[2]))
                             : (j == 0 ? s[0] : j == 1 ? s[1] : j == 2 ? s[2] : s[3]);
        st1(p, a, p0 + omega * (sj - cp) * inv);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if ((all || (j & cm) != s0) && (j > 0 || P.q > 0)) st1(sx, at + lat_sub(j, Qp), s[j]);
}

// pressure sweep of one parity or colour: p += omega (s - C p) / C_xx.  Bound by
// HBM: 17 M vertices, FP64 61 us, 4.5 TB/s of its 2 values per vertex.
template <typename T, int KIND, int NC>
__global__ void __launch_bounds__(256) k_lat_pres(Lat<T> L, LatSurf B, int col, int sb, LatGrid tg,
                                                  const T* __restrict__ sx, T* __restrict__ p, T omega) {
    if ((int)blockIdx.x < sb) {
        int X, Y, Z;
        if (!lat_surf_lane(L, B, 4 / NC, col, (int)blockIdx.x * tg.bs + (int)threadIdx.x, &X, &Y, &Z)) return;
        const T* __restrict__ r = L.rec + (size_t)L.rid[lat_rid_index(L, X, Y, Z)] * LR_SIZE;
        int nb[15];
        lat_taps(L, X, Y, Z, nb);
        T cp = T(0);
#pragma unroll
        for (int t = 0; t < 7; ++t) cp += r[LR_C + t] * p[nb[t]];
        p[nb[0]] += omega * (sx[nb[0]] - cp) * r[LR_INVC];
        return;
    }
    const LatTile tile = lat_tile(tg, L.nz - 2, (int)blockIdx.x - sb, L.order);
    if (!tile.ok) return;
    const LatPair P = lat_pair_lane<NC>(L, col, tg, tile, threadIdx.x);
    if (!P.ok) return;
    typedef typename V2<T>::type v2;
    const int at = (P.z * L.ny + P.y) * L.RS + lat_slot(P.s) * L.Qp + P.q;
    int xp, xm;
    lat_x_offsets(P.s, L.Qp, &xp, &xm);
    xp += at;
    xm += at;
    const int RS = L.RS, ZS = L.ZS;
    const v2 p0 = ld2(p, at), s = ld2(sx, at);
    v2 cp, inv;
    if (KIND == 0) {
        cp = L.c0 * p0 + L.c[0] * (ld2(p, xp) + ld2(p, xm)) + L.c[1] * (ld2(p, at + RS) + ld2(p, at - RS)) +
             L.c[2] * (ld2(p, at + ZS) + ld2(p, at - ZS));
        inv = v2{L.invc, L.invc};
    } else {
        const int X = 4 * P.q + P.s;
        const T* ra = L.axr + (size_t)L.rid[lat_rid_index(L, X, P.y, P.z)] * LX_SIZE;
        const T* rb = L.axr + (size_t)L.rid[lat_rid_index(L, X + 4, P.y, P.z)] * LX_SIZE;
        cp = v2{ra[LX_C0], rb[LX_C0]} * p0 + v2{ra[LX_C], rb[LX_C]} * ld2(p, xp) +
             v2{ra[LX_C + 1], rb[LX_C + 1]} * ld2(p, xm) + v2{ra[LX_C + 2], rb[LX_C + 2]} * ld2(p, at + RS) +
             v2{ra[LX_C + 3], rb[LX_C + 3]} * ld2(p, at - RS) + v2{ra[LX_C + 4], rb[LX_C + 4]} * ld2(p, at + ZS) +
             v2{ra[LX_C + 5], rb[LX_C + 5]} * ld2(p, at - ZS);
        inv = v2{ra[LX_INVC], rb[LX_INVC]};
    }
    const v2 r = p0 + omega * (s - cp) * inv;
    if (P.s != 0 || P.q != 0)
        *reinterpret_cast<typename V2<T>::load*>(p + at) = r;
    else
        p[at + 1] = r[1];
}

// ---------------------------------------------------------------------------
// r = b - K x (Dirichlet velocity rows 0); AP: r = K x instead.  WR: r is stored; NRM: per-block
// partial sums of r^2 at partials[tile] (volume) and partials[total + block]
// (surface), independent of the workgroup order.  200 VGPRs leave two waves per
// SIMD; held to three it spills and takes 746 us instead of 655 (17 M vertices,
// FP64, written: 2.5 TB/s of 12 values; norm only 440 us).
// ---------------------------------------------------------------------------
template <typename T, int KIND, bool WR, bool NRM, bool AP = false>
__global__ void __launch_bounds__(256) k_lat_res(Lat<T> L, LatSurf B, int sb, LatGrid tg,
                                                 const T* __restrict__ b, const T* __restrict__ x,
                                                 T* __restrict__ r, double* __restrict__ partials) {
    __shared__ double sh[4];
    const size_t len = L.len;
    const T* __restrict__ p = x + 3 * len;
    double acc = 0.0;
    int slot = -1;
    LatTile tile;
    bool ok;
    int X, Y, Z;
    if (lat_surf_work(L, B, sb, tg, L.ny - 2, L.nz - 2, &tile, &ok, &X, &Y, &Z)) {
        if ((int)blockIdx.x >= sb)
            slot = tile.t;
        else if ((int)blockIdx.x * tg.bs < B.beg[6])
            slot = tg.total + (int)blockIdx.x;
        if (ok) acc = lat_res_surface<T, WR, NRM, AP>(L, X, Y, Z, b, x, r);
    } else {
        slot = tile.t;
        const LatPair P = lat_quad_lane(L, tg, tile, threadIdx.x);
        if (tile.ok && P.ok) {
            const int at = (P.z * L.ny + P.y) * L.RS + P.q, Qp = L.Qp;
            const bool first = P.q > 0;   // x = 0 is a surface vertex
            const T* ra[4];
            if (KIND == 1)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    ra[j] = L.axr + (size_t)L.rid[lat_rid_index(L, 4 * P.q + j, P.y, P.z)] * LX_SIZE;
            T rp[4], t[3][4];
            {
                LatWin<T> W;
                lat_window(L, p, at, W);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    T d[7];
                    lat_diffs(W, j, d);
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        T v = T(0);
#pragma unroll
                        for (int q = 0; q < 7; ++q) v += L.bt[k][q] * d[q];
                        t[k][j] = v;
                    }
                    const T c = W.v[0][j + 1], xa = W.v[0][j + 2], xb = W.v[0][j], ya = W.v[1][j + 1],
                            yb = W.v[2][j + 1], za = W.v[3][j + 1], zb = W.v[4][j + 1];
                    rp[j] = KIND == 0 ? L.c0 * c + L.c[0] * (xa + xb) + L.c[1] * (ya + yb) + L.c[2] * (za + zb)
                                      : ra[j][LX_C0] * c + ra[j][LX_C] * xa + ra[j][LX_C + 1] * xb +
                                            ra[j][LX_C + 2] * ya + ra[j][LX_C + 3] * yb +
                                            ra[j][LX_C + 4] * za + ra[j][LX_C + 5] * zb;
                }
            }
            // rolled: one window live at a time
#pragma unroll 1
            for (int k = 0; k < 3; ++k) {
                LatWin<T> W;
                lat_window(L, x + k * len, at, W);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    T d[7];
                    lat_diffs(W, j, d);
#pragma unroll
                    for (int q = 0; q < 7; ++q) rp[j] += L.bt[k][q] * d[q];
                    const T c = W.v[0][j + 1], xa = W.v[0][j + 2], xb = W.v[0][j], ya = W.v[1][j + 1],
                            yb = W.v[2][j + 1], za = W.v[3][j + 1], zb = W.v[4][j + 1];
                    const T au = KIND == 0 ? L.a0 * c + L.a[0] * (xa + xb) + L.a[1] * (ya + yb) + L.a[2] * (za + zb)
                                           : ra[j][LX_A0] * c + ra[j][LX_A] * xa + ra[j][LX_A + 1] * xb +
                                                 ra[j][LX_A + 2] * ya + ra[j][LX_A + 3] * yb +
                                                 ra[j][LX_A + 4] * za + ra[j][LX_A + 5] * zb;
                    const int a = at + lat_sub(j, Qp);
                    const T bt = k == 0 ? t[0][j] : k == 1 ? t[1][j] : t[2][j];
                    const T v = AP ? bt + au : ld1(b + k * len, a) - bt - au;
                    if (j > 0 || first) {
                        if (WR) st1(r + k * len, a, v);
                        if (NRM) acc += (double)v * (double)v;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int a = at + lat_sub(j, Qp);
                const T v = AP ? -rp[j] : ld1(b + 3 * len, a) + rp[j];
                if (j > 0 || first) {
                    if (WR) st1(r + 3 * len, a, v);
                    if (NRM) acc += (double)v * (double)v;
                }
            }
        }
    }
    if (NRM) {
        const double tot = tg.bs == 64 ? wave_sum(acc) : block_sum256(acc, sh);
        if (threadIdx.x == 0 && slot >= 0) partials[slot] = tot;
    }
}

// ---------------------------------------------------------------------------
// Large levels in the red-black ordering with one viscosity (KIND 0): a lane takes
// the quads of a block of 2 x 2 rows (y0, y0 + 1) x (z0, z0 + 1), y0 and z0 odd.
// The one-row kernels above run at the rate of L2 requests (85 G lines/s, 11 TB/s,
// of which HBM sees half): every tap row of a wave is fetched from L2 again, since
// the L1 does not hold the rows of 16 waves.  A block of four rows reads 14 rows
// where four single rows read 28 (the seven rows of B and B^T), and 12 where they
// read 20 (the five rows of A and C).  Rows past the box (a side has an odd number
// of interior rows) are clamped into it; what they give is not stored.  Parities
// are constants: y0 + z0 is even.  17 M vertices, FP64 / FP32: the velocity sweep
// 209 -> 176 / 127 -> 91 us (4.2 / 4.1 TB/s of the bytes it cannot do without),
// B u with the red pressures 340 -> 265 / 222 -> 157 us (its neighbours' planes come
// from HBM twice: 5 TB/s of traffic); at 2.1 M vertices the 512
// workgroups leave the chip half empty (19.2 -> 21.7 and 40.3 -> 42.0 us, FP64), hence
// the rule of eight workgroups per CU.  The residual (k_lat_res) lost in this form:
// its 64 sums leave two waves per SIMD (448 -> 590 us).
// ---------------------------------------------------------------------------
template <typename T>
struct LatBlock {
    int y0, z0, q;
    unsigned v0, v2;   // byte offsets of rows y0 and y0 + 2 in a plane
    bool ok;
    // uniform base of row (dy, dz): the lane adds v0 (v2 for dy = 2)
    template <int DY, int DZ, typename F>
    __host__ __device__ __forceinline__ F* base(const Lat<T>& L, F* f, int sub) const {
        const int z = DZ == 2 ? (z0 + 2 < L.nz ? z0 + 2 : L.nz - 1) : z0 + DZ;
        return f + (ptrdiff_t)z * L.ZS + ((DY == 2 ? 0 : DY * L.RS) + sub);
    }
    template <int DY, int DZ, typename F>
    __host__ __device__ __forceinline__ F* at(const Lat<T>& L, F* f, int sub) const {
        using C = typename std::conditional<std::is_const<F>::value, const char, char>::type;
        return (F*)((C*)base<DY, DZ>(L, f, sub) + (DY == 2 ? v2 : v0));
    }
    // what follows is not moved ahead of this point
    __device__ __forceinline__ void anew() {
        asm volatile("" : "+v"(v0), "+v"(v2));
        __builtin_amdgcn_sched_barrier(0);
    }
    // row (oy, oz) of the block is an interior row
    __host__ __device__ bool in(const Lat<T>& L, int oy, int oz) const {
        return y0 + oy <= L.ny - 2 && z0 + oz <= L.nz - 2;
    }
};
template <typename T>
__host__ __device__ __forceinline__ int lat_block_lanes(const Lat<T>& L) { return L.ny / 2 * L.Qi; }   // per plane pair
template <typename T>
__host__ __device__ __forceinline__ LatBlock<T> lat_block_lane(const Lat<T>& L, const LatGrid& tg,
                                                               const LatTile& tile, int lane) {
    LatBlock<T> P;
    const int item = tile.part * tg.bs + lane, row = lat_div(item, tg.inv_row);
    P.z0 = 2 * tile.z + 1;
    P.y0 = 2 * row + 1;
    P.q = item - row * L.Qi;
    P.ok = row < L.ny / 2;
    P.v0 = (unsigned)((P.y0 * L.RS + P.q) * (int)sizeof(T));
    P.v2 = P.v0 + (unsigned)((P.y0 + 2 < L.ny ? 2 : 1) * L.RS * (int)sizeof(T));
    return P;
}
// the offset of row (dy, dz) from output row (oy, oz): 0 itself, 1, 2 +-y, 3, 4
// +-z, 5, 6 +-(y + z), -1 none
__host__ __device__ constexpr int lat_rel(int dy, int dz, int oy, int oz) {
    return dy == oy && dz == oz          ? 0
           : dy == oy + 1 && dz == oz     ? 1
           : dy == oy - 1 && dz == oz     ? 2
           : dy == oy && dz == oz + 1     ? 3
           : dy == oy && dz == oz - 1     ? 4
           : dy == oy + 1 && dz == oz + 1 ? 5
           : dy == oy - 1 && dz == oz - 1 ? 6
                                          : -1;
}
// whether any output row of the block reads row (dy, dz): among its 7 or 5 rows
__host__ __device__ constexpr bool lat_reads(int dy, int dz, int most) {
    for (int o = 0; o < 4; ++o) {
        const int r = lat_rel(dy, dz, o & 1, o >> 1);
        if (r >= 0 && r <= most) return true;
    }
    return false;
}
// entries x = 4q - 1 .. 4q + 4 of row (DY, DZ) at e[0..5]
template <int DY, int DZ, typename T>
__device__ __forceinline__ void lat_row6(const Lat<T>& L, const LatBlock<T>& P, const T* f, T e[6]) {
    const typename V2<T>::type l = ld2(P.template at<DY, DZ>(L, f, 0), 0);
    const typename V2<T>::type r = ld2(P.template at<DY, DZ>(L, f, 3 * L.Qp - 1), 0);
    e[0] = r[0];
    e[1] = l[0];
    e[2] = *P.template at<DY, DZ>(L, f, 2 * L.Qp);
    e[3] = *P.template at<DY, DZ>(L, f, L.Qp);
    e[4] = r[1];
    e[5] = l[1];
}
// what a row at relation r adds to sum_pairs w[q] (u(+d) - u(-d)) at position j
template <int R, typename T, typename W>
__device__ __forceinline__ T lat_row_diff(const W& w, const T e[6], int j) {
    if (R == 0) return w[0] * (e[j + 2] - e[j]);
    if (R == 1) return w[1] * e[j + 1] + w[3] * e[j + 2];
    if (R == 2) return -(w[1] * e[j + 1] + w[3] * e[j]);
    if (R == 3) return w[2] * e[j + 1] + w[5] * e[j + 2];
    if (R == 4) return -(w[2] * e[j + 1] + w[5] * e[j]);
    if (R == 5) return w[4] * e[j + 1] + w[6] * e[j + 2];
    return -(w[4] * e[j + 1] + w[6] * e[j]);
}
// rows of the block's neighbourhood, body(dy, dz) as constants.  Two rows are in
// flight per wave: with all of them the loads' registers leave two waves per SIMD
// (k_lat_bp_blk at 8 refinements 406 us, with two rows 287 us)
template <int MOST, typename P, typename F>
__device__ __forceinline__ void lat_rows(P& blk, F&& body) {
    auto one = [&](auto dyc, auto dzc) __attribute__((always_inline)) {
        if constexpr (lat_reads(decltype(dyc)::value, decltype(dzc)::value, MOST)) body(dyc, dzc);
    };
    using std::integral_constant;
#define LAT_ROWS(y, z) \
    one(integral_constant<int, y>{}, integral_constant<int, z>{}); \
    one(integral_constant<int, y + 1>{}, integral_constant<int, z>{}); \
    blk.anew()
    LAT_ROWS(-1, -1);
    LAT_ROWS(1, -1);
    LAT_ROWS(-1, 0);
    LAT_ROWS(1, 0);
    LAT_ROWS(-1, 1);
    LAT_ROWS(1, 1);
    LAT_ROWS(-1, 2);
    LAT_ROWS(1, 2);
#undef LAT_ROWS
}
// Values that a launch touches once, right-hand sides and results, do not take L2
// from the rows that its blocks share (nontemporal).  17 M vertices, FP64 / FP32:
// the sweep 195 -> 176 / 104 -> 91 us, B u 274 -> 265 / 178 -> 157 us.  The one-row
// kernels lose by it, at every size: the sweep 19.3 -> 26.5 us and B u 40 -> 48 us
// at 2.1 M vertices (the next launch finds its data in L2), the prolongation 249 ->
// 307 us at 17 M; the residual does not change.
template <typename T>
__device__ __forceinline__ T lat_once(const T* p) {
    return __builtin_nontemporal_load(p);
}
template <typename T>
__device__ __forceinline__ void lat_once(T* p, T v) {
    __builtin_nontemporal_store(v, p);
}
// the value is worked out here, not where it is (conditionally) stored
template <typename T>
__device__ __forceinline__ void lat_pin(T& v) {
    asm volatile("" : "+v"(v));
}
// body(o) for the four output rows, o a constant
template <typename F>
__device__ __forceinline__ void lat_four(F&& body) {
    body(std::integral_constant<int, 0>{});
    body(std::integral_constant<int, 1>{});
    body(std::integral_constant<int, 2>{});
    body(std::integral_constant<int, 3>{});
}
// body(output row o, relation) for the output rows that read row (dy, dz)
template <int MOST, int DY, int DZ, typename F>
__device__ __forceinline__ void lat_outs(F&& body) {
    using std::integral_constant;
    auto one = [&](auto oc) __attribute__((always_inline)) {
        constexpr int o = decltype(oc)::value, r = lat_rel(DY, DZ, o & 1, o >> 1);
        if constexpr (r >= 0 && r <= MOST) body(oc, integral_constant<int, r>{});
    };
    one(integral_constant<int, 0>{});
    one(integral_constant<int, 1>{});
    one(integral_constant<int, 2>{});
    one(integral_constant<int, 3>{});
}
// first position of parity col in output row o of a block (y0 + z0 even)
__host__ __device__ constexpr int lat_first(int col, int o) { return (col + (o & 1) + (o >> 1)) & 1; }

template <typename T, int COL, bool PZ>
__global__ void __launch_bounds__(256, 4) k_lat_vel_blk(Lat<T> L, LatSurf B, int sb, LatGrid tg,
                                                     const T* __restrict__ b, T* __restrict__ x) {
    const size_t len = L.len;
    const T* __restrict__ p = x + 3 * len;
    if ((int)blockIdx.x < sb) {
        lat_vel_surface<T, PZ>(L, B, 2, COL, (int)blockIdx.x * tg.bs + (int)threadIdx.x, b, x);
        return;
    }
    LatTile tile = lat_tile(tg, L.nz / 2, (int)blockIdx.x - sb, L.order);
    tile.z = __builtin_amdgcn_readfirstlane(tile.z);
    if (!tile.ok) return;
    LatBlock<T> P = lat_block_lane(L, tg, tile, threadIdx.x);
    if (!P.ok) return;
    const int Qp = L.Qp;
    T t[4][3][2];
    lat_four([&](auto oc) __attribute__((always_inline)) {
        constexpr int o = decltype(oc)::value;
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int e = 0; e < 2; ++e)
                t[o][k][e] =
                    lat_once(P.template at<(o & 1), (o >> 1)>(L, b + k * len, lat_sub(lat_first(COL, o) + 2 * e, Qp)));
    });
    if (!PZ)
        lat_rows<6>(P, [&](auto dyc, auto dzc) __attribute__((always_inline)) {
            constexpr int dy = decltype(dyc)::value, dz = decltype(dzc)::value;
            T e[6];
            lat_row6<dy, dz>(L, P, (const T*)p, e);
            lat_outs<6, dy, dz>([&](auto oc, auto rc) __attribute__((always_inline)) {
                constexpr int o = decltype(oc)::value, s0 = lat_first(COL, o);
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        t[o][k][h] -= lat_row_diff<decltype(rc)::value>(L.bt[k], e, s0 + 2 * h);
                        lat_pin(t[o][k][h]);
                    }
            });
        });
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const T* __restrict__ u = x + k * len;
        lat_rows<4>(P, [&](auto dyc, auto dzc) __attribute__((always_inline)) {
            constexpr int dy = decltype(dyc)::value, dz = decltype(dzc)::value;
            // the row's vertices of the other parity, positions b0, b0 + 2 (and
            // one more beside the quad for the row's own update)
            constexpr int b0 = (1 + COL + dy + dz + 4) & 1;
            constexpr bool own = lat_rel(dy, dz, dy, dz) == 0 && dy >= 0 && dy < 2 && dz >= 0 && dz < 2;
            T e[6];
            e[b0 + 1] = *P.template at<dy, dz>(L, u, lat_sub(b0, Qp));
            e[b0 + 3] = *P.template at<dy, dz>(L, u, lat_sub(b0 + 2, Qp));
            if (own) {
                if (b0 == 1)
                    e[0] = *P.template at<dy, dz>(L, u, 3 * Qp - 1);
                else
                    e[5] = *P.template at<dy, dz>(L, u, 1);
            }
            lat_outs<4, dy, dz>([&](auto oc, auto rc) __attribute__((always_inline)) {
                constexpr int o = decltype(oc)::value, r = decltype(rc)::value, s0 = lat_first(COL, o);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int j = s0 + 2 * h + 1;
                    t[o][k][h] -= r == 0 ? L.a[0] * (e[j + 1] + e[j - 1]) : (r <= 2 ? L.a[1] : L.a[2]) * e[j];
                }
            });
        });
        lat_four([&](auto oc) __attribute__((always_inline)) {
            constexpr int o = decltype(oc)::value;
#pragma unroll
            for (int h = 0; h < 2; ++h) lat_pin(t[o][k][h]);
            if (!P.in(L, o & 1, o >> 1)) return;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = lat_first(COL, o) + 2 * h;
                if (j == 0 && P.q == 0) continue;   // x = 0
                lat_once(P.template at<(o & 1), (o >> 1)>(L, x + k * len, lat_sub(j, Qp)), t[o][k][h] * L.inva);
            }
        });
    }
}

template <typename T>
__global__ void __launch_bounds__(256, 4) k_lat_bp_blk(Lat<T> L, LatSurf B, int sb, LatGrid tg,
                                                    const T* __restrict__ b, T* __restrict__ x,
                                                    T* __restrict__ sx, T omega, int all) {
    const size_t len = L.len;
    T* __restrict__ p = x + 3 * len;
    const T* __restrict__ g = b + 3 * len;
    LatTile tile;
    bool ok;
    int X, Y, Z;
    if (lat_surf_work(L, B, sb, tg, L.ny / 2, L.nz / 2, &tile, &ok, &X, &Y, &Z)) {
        if (ok) lat_bp_surface<T>(L, X, Y, Z, 1, 0, g, x, sx, omega, all);
        return;
    }
    tile.z = __builtin_amdgcn_readfirstlane(tile.z);
    if (!tile.ok) return;
    LatBlock<T> P = lat_block_lane(L, tg, tile, threadIdx.x);
    if (!P.ok) return;
    const int Qp = L.Qp;
    T s[4][4], cp[4][2], p0[4][2];
    lat_four([&](auto oc) __attribute__((always_inline)) {
        constexpr int o = decltype(oc)::value;
#pragma unroll
        for (int j = 0; j < 4; ++j) s[o][j] = -lat_once(P.template at<(o & 1), (o >> 1)>(L, g, lat_sub(j, Qp)));
    });
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const T* __restrict__ u = x + k * len;
        lat_rows<6>(P, [&](auto dyc, auto dzc) __attribute__((always_inline)) {
            constexpr int dy = decltype(dyc)::value, dz = decltype(dzc)::value;
            T e[6];
            lat_row6<dy, dz>(L, P, (const T*)u, e);
            lat_outs<6, dy, dz>([&](auto oc, auto rc) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    s[decltype(oc)::value][j] -= lat_row_diff<decltype(rc)::value>(L.bt[k], e, j);
            });
        });
    }
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int h = 0; h < 2; ++h) cp[o][h] = T(0);
    lat_rows<4>(P, [&](auto dyc, auto dzc) __attribute__((always_inline)) {
        constexpr int dy = decltype(dyc)::value, dz = decltype(dzc)::value;
        constexpr bool own = dy >= 0 && dy < 2 && dz >= 0 && dz < 2;
        constexpr int b0 = (1 + dy + dz + 4) & 1;   // black positions of the row
        T e[6];
        if (own) {
            lat_row6<dy, dz>(L, P, (const T*)p, e);
        } else {
            e[b0 + 1] = *P.template at<dy, dz>(L, p, lat_sub(b0, Qp));
            e[b0 + 3] = *P.template at<dy, dz>(L, p, lat_sub(b0 + 2, Qp));
        }
        lat_outs<4, dy, dz>([&](auto oc, auto rc) __attribute__((always_inline)) {
            constexpr int o = decltype(oc)::value, r = decltype(rc)::value, s0 = lat_first(0, o);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = s0 + 2 * h + 1;
                if (r == 0) {
                    p0[o][h] = e[j];
                    cp[o][h] += L.c0 * e[j] + L.c[0] * (e[j + 1] + e[j - 1]);
                } else {
                    cp[o][h] += (r <= 2 ? L.c[1] : L.c[2]) * e[j];
                }
            }
        });
    });
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int h = 0; h < 2; ++h) lat_pin(cp[o][h]);
    lat_four([&](auto oc) __attribute__((always_inline)) {
        constexpr int o = decltype(oc)::value;
        if (!P.in(L, o & 1, o >> 1)) return;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j == 0 && P.q == 0) continue;   // x = 0
            const bool red = ((j + lat_first(0, o)) & 1) == 0;
            if (red)
                lat_once(P.template at<(o & 1), (o >> 1)>(L, p, lat_sub(j, Qp)),
                         p0[o][j / 2] + omega * (s[o][j] - cp[o][j / 2]) * L.invc);
            if (!red || all) lat_once(P.template at<(o & 1), (o >> 1)>(L, sx, lat_sub(j, Qp)), s[o][j]);
        }
    });
}

// t_k = b_k - (A u)_k (k = 0..2; Dirichlet rows 0): the velocity residual of the
// velocity multigrid.
template <typename T, int KIND>
__global__ void __launch_bounds__(256) k_lat_ares(Lat<T> L, LatSurf B, int sb, LatGrid tg,
                                                  const T* __restrict__ b, const T* __restrict__ x,
                                                  T* __restrict__ r) {
    const size_t len = L.len;
    LatTile tile;
    bool ok;
    int X, Y, Z;
    if (lat_surf_work(L, B, sb, tg, L.ny - 2, L.nz - 2, &tile, &ok, &X, &Y, &Z)) {
        if (!ok) return;
        const int id = L.rid[lat_rid_index(L, X, Y, Z)];
        const T* __restrict__ rc = L.rec + (size_t)id * LR_SIZE;
        const bool dir = L.rdir[id] != 0;
        int nb[15];
        lat_taps(L, X, Y, Z, nb);
        for (int k = 0; k < 3; ++k) {
            T w = T(0);
            if (!dir) {
                w = b[k * len + nb[0]];
#pragma unroll
                for (int t = 0; t < 7; ++t) w -= rc[LR_A + t] * x[k * len + nb[t]];
            }
            r[k * len + nb[0]] = w;
        }
        return;
    }
    if (!tile.ok) return;
    const LatPair P = lat_quad_lane(L, tg, tile, threadIdx.x);
    if (!P.ok) return;
    const int at = (P.z * L.ny + P.y) * L.RS + P.q, Qp = L.Qp;
    const T* ra[4];
    if (KIND == 1)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            ra[j] = L.axr + (size_t)L.rid[lat_rid_index(L, 4 * P.q + j, P.y, P.z)] * LX_SIZE;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const T* __restrict__ u = x + k * len;
        T c[6];   // x = 4q - 1 .. 4q + 4
        c[1] = ld1(u, at);
        c[2] = ld1(u, at + 2 * Qp);
        c[3] = ld1(u, at + Qp);
        c[4] = ld1(u, at + 3 * Qp);
        c[5] = ld1(u, at + 1);
        c[0] = ld1(u, at + 3 * Qp - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int a = at + lat_sub(j, Qp);
            const T ya = ld1(u, a + L.RS), yb = ld1(u, a - L.RS), za = ld1(u, a + L.ZS), zb = ld1(u, a - L.ZS);
            const T au = KIND == 0 ? L.a0 * c[j + 1] + L.a[0] * (c[j + 2] + c[j]) + L.a[1] * (ya + yb) + L.a[2] * (za + zb)
                                   : ra[j][LX_A0] * c[j + 1] + ra[j][LX_A] * c[j + 2] + ra[j][LX_A + 1] * c[j] +
                                         ra[j][LX_A + 2] * ya + ra[j][LX_A + 3] * yb + ra[j][LX_A + 4] * za +
                                         ra[j][LX_A + 5] * zb;
            const T v = ld1(b + k * len, a) - au;
            if (j > 0 || P.q > 0) st1(r + k * len, a, v);
        }
    }
}

// ---------------------------------------------------------------------------
// Restriction bc = P^T rf (weights 1 and 1/2, Dirichlet velocity rows 0), with
// the coarse iterate xc set to 0 in the same pass.  Interior lanes: the coarse
// quad q reads the fine row segments 8 q - 1 .. 8 q + 7 as pairs.  17 M fine
// vertices, FP64: 170 us, 4.0 TB/s of the four fine values it reads and the eight
// coarse ones it writes (5.4 TB/s of its traffic, 0.92 GB).
// ---------------------------------------------------------------------------
template <typename T, int NF = 4>
__global__ void __launch_bounds__(256) k_lat_restrict(Lat<T> C, Lat<T> F, LatSurf B, int sb, LatGrid tg,
                                                      const T* __restrict__ rf, T* __restrict__ bc,
                                                      T* __restrict__ xc) {
    const size_t lc = C.len, lf = F.len;
    LatTile tile;
    bool ok;
    int X, Y, Z;
    if (lat_surf_work(C, B, sb, tg, C.ny - 2, C.nz - 2, &tile, &ok, &X, &Y, &Z)) {
        if (!ok) return;
        const bool dir = C.rdir[C.rid[lat_rid_index(C, X, Y, Z)]] != 0;
        const int a = lat_at(C, X, Y, Z);
        int nb[15];
        lat_taps(F, 2 * X, 2 * Y, 2 * Z, nb);
        for (int f = 0; f < NF; ++f) {
            T acc = T(0);
            if (f == 3 || !dir) {
#pragma unroll
                for (int g = 1; g < 15; ++g) acc += nb[g] != nb[0] ? rf[f * lf + nb[g]] : T(0);
                acc = rf[f * lf + nb[0]] + T(0.5) * acc;
            }
            bc[f * lc + a] = acc;
            xc[f * lc + a] = T(0);
        }
        return;
    }
    if (!tile.ok) return;
    const LatPair P = lat_quad_lane(C, tg, tile, threadIdx.x);
    if (!P.ok) return;
    typedef typename V2<T>::type v2;
    const int at = (P.z * C.ny + P.y) * C.RS + P.q;
    const int fa = (2 * P.z * F.ny + 2 * P.y) * F.RS + 2 * P.q;
#pragma unroll 1
    for (int f = 0; f < NF; ++f) {
        const T* __restrict__ v = rf + f * lf;
        T acc[4], ctr[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = T(0);
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            const int o = r == 0 ? 0 : r == 1 ? F.RS : r == 2 ? -F.RS : r == 3 ? F.ZS : r == 4 ? -F.ZS
                        : r == 5 ? F.RS + F.ZS : -F.RS - F.ZS;
            const int a = fa + o;
            const v2 e0 = ld2(v, a), e2 = ld2(v, a + F.Qp), o1 = ld2(v, a + 2 * F.Qp),
                     o3 = ld2(v, a + 3 * F.Qp);
            const T e[4] = {e0[0], e2[0], e0[1], e2[1]}, od[4] = {o1[0], o3[0], o1[1], o3[1]};
            const bool back = r == 0 || !(r & 1), ahead = r == 0 || (r & 1);
            const T left = back ? ld1(v, a + 3 * F.Qp - 1) : T(0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (r == 0)
                    ctr[j] = e[j];
                else
                    acc[j] += e[j];
                if (ahead) acc[j] += od[j];
                if (back) acc[j] += j > 0 ? od[j - 1] : left;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j == 0 && P.q == 0) continue;
            const int a = at + lat_sub(j, C.Qp);
            st1(bc + f * lc, a, ctr[j] + T(0.5) * acc[j]);
            st1(xc + f * lc, a, T(0));
        }
    }
}

// Prolongation over every fine vertex: x_f += P e_c (SET: x_f = P e_c except on
// Dirichlet velocity).  A fine vertex with odd bits d is the midpoint of the
// coarse vertices (X - d) / 2 and (X + d) / 2.  17 M fine vertices, FP64: 248 us,
// 4.7 TB/s of its bytes.
template <typename T, bool SET, int NF = 4>
__global__ void __launch_bounds__(256) k_lat_prolong(Lat<T> F, Lat<T> C, const T* __restrict__ ec,
                                                     T* __restrict__ xf) {
    const size_t lc = C.len, lf = F.len;
    const int Q = F.Qi + 1;
    const int item = (int)blockIdx.x * 256 + (int)threadIdx.x, z = (int)blockIdx.y;
    const int y = lat_div(item, 1.0f / (float)Q), q = item - y * Q;
    if (y >= F.ny) return;
    const int by = y & 1, bz = z & 1;
    const int lo = (((z - bz) >> 1) * C.ny + ((y - by) >> 1)) * C.RS,
              hi = (((z + bz) >> 1) * C.ny + ((y + by) >> 1)) * C.RS;
    // coarse x = 2 q, 2 q + 1, 2 q + 2
    const int X = 2 * q;
    const int i0 = lat_slot(X & 3) * C.Qp + (X >> 2), i1 = lat_slot((X + 1) & 3) * C.Qp + ((X + 1) >> 2),
              i2 = lat_slot((X + 2) & 3) * C.Qp + ((X + 2) >> 2);
    const int at = (z * F.ny + y) * F.RS + q;
    const bool last = q == F.Qi;   // only x = nx - 1
    bool keep[4] = {false, false, false, false};
    if (SET)
        for (int j = 0; j < 4; ++j) {
            const int x = 4 * q + j;
            if (x < F.nx && (x == 0 || x == F.nx - 1 || y == 0 || y == F.ny - 1 || z == 0 || z == F.nz - 1))
                keep[j] = F.rdir[F.rid[lat_rid_index(F, x, y, z)]] != 0;
        }
    T e[NF][4], xv[NF][4];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const T* __restrict__ c = ec + f * lc;
        const T l0 = ld1(c, lo + i0), l1 = ld1(c, lo + i1), h0 = ld1(c, hi + i0), h1 = ld1(c, hi + i1),
                h2 = ld1(c, hi + i2);
        e[f][0] = T(0.5) * (l0 + h0);
        e[f][1] = T(0.5) * (l0 + h1);
        e[f][2] = T(0.5) * (l1 + h1);
        e[f][3] = T(0.5) * (l1 + h2);
#pragma unroll
        for (int j = 0; j < 4; ++j) xv[f][j] = ld1(xf + f * lf, at + lat_sub(j, F.Qp));
    }
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j > 0 && last) continue;
            if (SET && f < 3 && keep[j]) continue;
            st1(xf + f * lf, at + lat_sub(j, F.Qp), SET ? e[f][j] : xv[f][j] + e[f][j]);
        }
}

// sum_i m_i p_i over every vertex, per-block partials at the natural index
template <typename T>
__global__ void __launch_bounds__(256) k_lat_mass(Lat<T> L, const T* __restrict__ p,
                                                  double* __restrict__ partials) {
    __shared__ double sh[4];
    const int Q = L.Qi + 1;
    const int item = (int)blockIdx.x * 256 + (int)threadIdx.x, z = (int)blockIdx.y;
    const int y = lat_div(item, 1.0f / (float)Q), q = item - y * Q;
    double acc = 0.0;
    if (y < L.ny) {
        const bool edge = y == 0 || y == L.ny - 1 || z == 0 || z == L.nz - 1;
        const int at = (z * L.ny + y) * L.RS + q;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int x = 4 * q + j;
            if (x >= L.nx) continue;
            const T w = edge || x == 0 || x == L.nx - 1
                            ? L.rec[(size_t)L.rid[lat_rid_index(L, x, y, z)] * LR_SIZE + LR_MASS]
                            : L.mass;
            acc += (double)w * (double)ld1(p, at + lat_sub(j, L.Qp));
        }
    }
    const double tot = block_sum256(acc, sh);
    if (threadIdx.x == 0) partials[(size_t)z * gridDim.x + blockIdx.x] = tot;
}

// Conversions between the ABI's per-macro layout (4 fields of stride plen) and
// the lattice layout.  In: one lane per lattice vertex, from its primary slot.
// Out: one lane per slot (every copy is written; padding untouched).  17 M vertices,
// FP64: 0.71 ms each, bound by the scattered side (64 lines per wave and field).
template <typename T, int NF = 4>
__global__ void __launch_bounds__(256) k_lat_in(Lat<T> L, const int* __restrict__ node_slot,
                                                const double* __restrict__ v, size_t plen,
                                                T* __restrict__ x) {
    const int item = (int)blockIdx.x * 256 + (int)threadIdx.x, z = (int)blockIdx.y;
    const int y = lat_div(item, 1.0f / (float)L.nx), X = item - y * L.nx;
    if (y >= L.ny) return;
    const int s = node_slot[(size_t)(z * L.ny + y) * L.nx + X], a = lat_at(L, X, y, z);
#pragma unroll
    for (int f = 0; f < NF; ++f) x[f * L.len + a] = (T)v[f * plen + s];
}
template <typename T>
__global__ void __launch_bounds__(256) k_lat_out(Lat<T> L, const int* __restrict__ slot_node, size_t plen,
                                                 const T* __restrict__ x, double* __restrict__ v) {
    const size_t s = blockIdx.x * (size_t)256 + threadIdx.x;
    if (s >= plen) return;
    const int node = slot_node[s];
    if (node < 0) return;
    const int row = node / L.nx, X = node - row * L.nx, z = row / L.ny, y = row - z * L.ny;
    const int a = lat_at(L, X, y, z);
#pragma unroll
    for (int f = 0; f < 4; ++f) v[f * plen + s] = (double)x[f * L.len + a];
}

// ---------------------------------------------------------------------------
// Levels whose iterate fits the LDS of one CU: all smoothing steps of a visit
// in one workgroup of 16 waves, with barriers instead of launches, and the
// residual after the last step.  On such a level a launch is all latency (3 to
// 5 us for a few thousand vertices; five launches per Uzawa step in the
// red-black order, eleven in the colour order).  A lane owns one interior quad
// (x = 4 q .. 4 q + 3) and keeps its rows f - B^T p and B u - g in registers,
// ordered by colour; surface vertices are dealt out face by face, so that a
// wave's records are the same and come from scalar loads.
// Measured, FP64, an Uzawa step: 9^3 vertices 7 us red-black, 13 us colours
// (launches: 19 and 42), bound by latency; 17^3 vertices 21 and 30 us (19.5 and
// 42), bound by one CU's LDS (two thirds of the cycles, half of them bank
// conflicts) and FP64 rate.
// ---------------------------------------------------------------------------
// LDS layout of a visit: rows of SX values (sub-row 0 first with one entry more
// than the others), planes of SX SY.  The strides are constants, so that a tap is
// an immediate offset of its vertex; smaller boxes leave entries unused.  A pad
// in front and behind keeps the taps of surface vertices that leave the box in
// range: their coefficients are 0 and every value there is finite.
template <int SX_, int SY_>
struct LdsGeom {
    static constexpr int SX = SX_, PS = SX_ * SY_, Q = (SX_ - 1) / 4, PAD = PS + SX_ + 1;
    int nx, ny, nz;
    __host__ __device__ static constexpr int off(int s) { return s * Q + (s > 0 ? 1 : 0); }
    __host__ __device__ int at(int x, int y, int z) const { return z * PS + y * SX + off(x & 3) + (x >> 2); }
    __host__ __device__ int field() const { return PS * nz; }
    __host__ __device__ int values() const { return 4 * field() + 2 * PAD; }
    __host__ __device__ bool holds() const { return nx <= SX_ && ny <= SY_; }
};

// i / d for small i and d
__host__ __device__ __forceinline__ int lat_idiv(int i, int d) { return (int)(((float)i + 0.5f) / (float)d); }

// Surface lane i of a visit: faces z0, z1, y0, y1, x0, x1 without their edges,
// each padded to whole waves, then edges and corners.
template <typename G>
__host__ __device__ __forceinline__ int lat_rim_waves(const G& g, int f) {
    const int a = f < 4 ? g.nx - 2 : g.ny - 2, b = f < 2 ? g.ny - 2 : g.nz - 2;
    if (f < 6) return (a * b + 63) / 64;
    return (4 * (g.nx + g.ny + g.nz - 6) + 8 + 63) / 64;
}
template <typename G>
__host__ __device__ __forceinline__ bool lat_rim_lane(const G& g, int i, int* x, int* y, int* z) {
    int w = i >> 6, f = 0;
    for (; f < 7; ++f) {
        const int c = lat_rim_waves(g, f);
        if (w < c) break;
        w -= c;
    }
    if (f == 7) return false;
    int k = (w << 6) + (i & 63);
    if (f < 6) {
        const int a = f < 4 ? g.nx - 2 : g.ny - 2, b = f < 2 ? g.ny - 2 : g.nz - 2;
        if (k >= a * b) return false;
        const int r = lat_idiv(k, a), s = k - r * a;
        *x = f < 4 ? s + 1 : f == 4 ? 0 : g.nx - 1;
        *y = f < 2 ? r + 1 : f == 2 ? 0 : f == 3 ? g.ny - 1 : s + 1;
        *z = f == 0 ? 0 : f == 1 ? g.nz - 1 : r + 1;
        return true;
    }
    if (k < 8) {
        *x = k & 1 ? g.nx - 1 : 0;
        *y = k & 2 ? g.ny - 1 : 0;
        *z = k & 4 ? g.nz - 1 : 0;
        return true;
    }
    k -= 8;
    const int n0 = 4 * (g.nx - 2), n1 = 4 * (g.ny - 2), n2 = 4 * (g.nz - 2);
    const int c = k & 3, m = k >> 2;
    if (k < n0) {
        *x = m + 1;
        *y = c & 1 ? g.ny - 1 : 0;
        *z = c & 2 ? g.nz - 1 : 0;
        return true;
    }
    if (k < n0 + n1) {
        *y = m - (g.nx - 2) + 1;
        *x = c & 1 ? g.nx - 1 : 0;
        *z = c & 2 ? g.nz - 1 : 0;
        return true;
    }
    if (k < n0 + n1 + n2) {
        *z = m - (g.nx - 2) - (g.ny - 2) + 1;
        *x = c & 1 ? g.nx - 1 : 0;
        *y = c & 2 ? g.ny - 1 : 0;
        return true;
    }
    return false;
}

// surface wave w of a visit lies in a face (its lanes share their class)
template <typename G>
__host__ __device__ __forceinline__ bool lat_rim_is_face(const G& g, int w) {
    int c = 0;
    for (int f = 0; f < 6; ++f) c += lat_rim_waves(g, f);
    return w < c;
}
// Interior item i: V = 4 the quad that starts at (*x, *y, *z), V = 1 a vertex.
// Rows four apart come first: with 17 values to an LDS row, eight of them then
// fall into distinct banks.
template <int V, typename G>
__host__ __device__ __forceinline__ bool lat_visit_item(const G& g, int i, int* x, int* y, int* z) {
    const int w = V == 4 ? (g.nx - 1) / 4 : g.nx - 2, row = lat_idiv(i, w), h = g.ny - 2;
    const int zz = lat_idiv(row, h), yy = row - zz * h;
    const bool ok = zz < g.nz - 2;
    // yy counts 0, 4, 8, .., 1, 5, 9, ..
    int r = yy, c = 0;
    for (; c < 3; ++c) {
        const int m = (h + 3 - c) >> 2;
        if (r < m) break;
        r -= m;
    }
    *x = ok ? (V == 4 ? 4 * (i - row * w) : i - row * w + 1) : 0;
    *y = ok ? 4 * r + c + 1 : 1;
    *z = ok ? zz + 1 : 1;
    return ok;
}

// rows of a group around a quad: a[e + 1] of the row ahead (the quad's own row
// in group 0), b[e + 1] of the row behind, e = -1 .. 4
template <typename T>
struct LdsRows {
    T a[6], b[6];
};
template <typename GEO, int G, typename T>
__device__ __forceinline__ void lds_rows(const T* f, LdsRows<T>& R) {
    constexpr int o = G == 0 ? 0 : G == 1 ? GEO::SX : G == 2 ? GEO::PS : GEO::SX + GEO::PS;
    constexpr int o1 = GEO::off(1), o2 = GEO::off(2), o3 = GEO::off(3);
    const T* p = f + o;
    R.a[1] = p[0];
    R.a[2] = p[o1];
    R.a[3] = p[o2];
    R.a[4] = p[o3];
    R.a[5] = p[1];
    if (G == 0) {
        R.a[0] = p[o3 - 1];
    } else {
        const T* m = f - o;
        R.b[0] = m[o3 - 1];
        R.b[1] = m[0];
        R.b[2] = m[o1];
        R.b[3] = m[o2];
        R.b[4] = m[o3];
    }
}
// acc[j] += w0 (first pair of the group) + w1 (second pair)
template <int G, typename T>
__device__ __forceinline__ void lds_diff(const LdsRows<T>& R, T w0, T w1, T acc[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (G == 0)
            acc[j] += w0 * (R.a[j + 2] - R.a[j]);
        else
            acc[j] += w0 * (R.a[j + 1] - R.b[j + 1]) + w1 * (R.a[j + 2] - R.b[j]);
    }
}
// pairs of group G
__host__ __device__ constexpr int lat_gp0(int G) { return G == 0 ? 0 : G == 1 ? 1 : G == 2 ? 2 : 4; }
__host__ __device__ constexpr int lat_gp1(int G) { return G == 0 ? 0 : G == 1 ? 3 : G == 2 ? 5 : 6; }

// v[e] <- v[(e + r) & 3]: rows by position in the quad -> rows by colour
template <typename T>
__device__ __forceinline__ void lat_rotate(T v[4], int r) {
    const T a0 = r & 1 ? v[1] : v[0], a1 = r & 1 ? v[2] : v[1], a2 = r & 1 ? v[3] : v[2],
            a3 = r & 1 ? v[0] : v[3];
    v[0] = r & 2 ? a2 : a0;
    v[1] = r & 2 ? a3 : a1;
    v[2] = r & 2 ? a0 : a2;
    v[3] = r & 2 ? a1 : a3;
}

// LDS offsets of x + 1 and x - 1 from a vertex of sub-row s
template <typename GEO>
__host__ __device__ __forceinline__ void lds_x_offsets(int s, int* P, int* M) {
    constexpr int q = GEO::Q;
    *P = s == 3 ? -3 * q : s == 0 ? q + 1 : q;
    *M = s == 0 ? 3 * q : s == 1 ? -q - 1 : -q;
}

template <typename T>
using LatConst = const __attribute__((address_space(4))) T*;

// passes of a visit: the rows f - B^T p, the rows B u - g, the velocity sweep of
// colour (parity) op - LOP_V, the pressure sweep of colour op - LOP_P
enum { LOP_T = 0, LOP_S = 1, LOP_V = 4, LOP_P = 8 };
struct LatProg {
    int n;
    unsigned char op[24];
};

constexpr int LDS_WAVES = 16, LDS_TPB = 64 * LDS_WAVES;

// V: vertices of an interior item, 4 (quads) or 1 (levels with at most 1024
// interior vertices: more waves share the latency); QR, SR: interior items and
// surface vertices per lane (at most).  S = 2: red-black, 4: colours.  zero: x =
// 0 on entry; rim: some surface vertex has a free velocity; res: r = b - K x
// after the last step.  prog: the passes of a step.  vo: the
// velocity block alone (A u = b, fields 0..2; field 3 is left alone).
template <typename T, int KIND, int S, typename GEO, int V, int QR, int SR>
__global__ void __launch_bounds__(LDS_TPB) k_lat_visit(Lat<T> L, const T* __restrict__ b,
                                                       T* __restrict__ x, T* __restrict__ r, int steps,
                                                       int zero, int rim, int res, int vo, LatProg prog, T omega) {
    extern __shared__ char lds_raw[];
    const size_t len = L.len;
    const GEO g{L.nx, L.ny, L.nz};
    constexpr int SX = GEO::SX, PS = GEO::PS;
    const int N = g.field(), tid = (int)threadIdx.x;
    T* f0 = reinterpret_cast<T*>(lds_raw) + GEO::PAD;
    T* pr = f0 + 3 * N;
    for (int i = tid; i < g.values(); i += LDS_TPB) f0[i - GEO::PAD] = T(0);
    __syncthreads();
    // whole rows in and out
    auto copy = [&](auto body) __attribute__((always_inline)) {
        for (int i = tid; i < g.nx * g.ny * g.nz; i += LDS_TPB) {
            const int row = lat_idiv(i, g.nx), e = i - row * g.nx, z = lat_idiv(row, g.ny), y = row - z * g.ny;
            const int s = e <= L.Qi ? 0 : e <= 2 * L.Qi ? 1 : e <= 3 * L.Qi ? 2 : 3, q = e - s * L.Qi - (s > 0 ? 1 : 0);
            body(z * PS + y * SX + GEO::off(s) + q, row * L.RS + lat_slot(s) * L.Qp + q);
        }
    };
    if (!zero)
        copy([&](int i, int a) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < 3 || !vo) f0[k * N + i] = x[k * len + a];
        });
    // this lane's interior items: LDS and global address of x = 4 q (V = 4) or of
    // the vertex, position of colour 0 (V = 4) or the vertex's colour (V = 1)
    int qat[QR], gat[QR], rot[QR], qpm[QR];
    bool qok0[QR];
    int rid[QR][V];
#pragma unroll
    for (int c = 0; c < QR; ++c) {
        int X, Y, Z;
        const bool ok = lat_visit_item<V>(g, tid + c * LDS_TPB, &X, &Y, &Z);
        qat[c] = g.at(X, Y, Z);
        gat[c] = lat_at(L, X, Y, Z);
        int P, M;
        lds_x_offsets<GEO>(X & 3, &P, &M);
        qpm[c] = P * 65536 + (M & 65535);
        qok0[c] = X > 0;
        rot[c] = V == 4 ? (4 * (g.ny + g.nz) - Y - Z) & (S - 1) : (X + Y + Z) & (S - 1);
        if (!ok) rot[c] |= 64;
        if (KIND == 1)
#pragma unroll
            for (int e = 0; e < V; ++e)
                rid[c][e] = ok ? L.rid[lat_rid_index(L, V == 4 ? X + ((e + rot[c]) & 3) : X, Y, Z)] : 0;
    }
    // this lane's surface vertices, dealt from the last wave down; a face's
    // waves share their class, edges and corners do not (scls < 0)
    int sat[SR], sga[SR], sPM[SR], sok[SR], srid[SR];
    int sface[SR], scls[SR];
#pragma unroll
    for (int c = 0; c < SR; ++c) {
        const int wave = c * LDS_WAVES + (LDS_WAVES - 1 - (tid >> 6));
        int X = 0, Y = 0, Z = 0;
        const bool ok = lat_rim_lane(g, wave * 64 + (tid & 63), &X, &Y, &Z);
        sat[c] = g.at(X, Y, Z);
        sga[c] = lat_at(L, X, Y, Z);
        srid[c] = L.rid[lat_rid_index(L, X, Y, Z)];
        int P, M;
        lds_x_offsets<GEO>(X & 3, &P, &M);
        sPM[c] = P * 65536 + (M & 65535);
        scls[c] = lat_class(L, X, Y, Z);
        // lane 0 of a face's wave is a vertex of the face
        const bool face = lat_rim_is_face(g, __builtin_amdgcn_readfirstlane(wave));
        sface[c] = face ? __builtin_amdgcn_readfirstlane(scls[c]) : -1;
        sok[c] = ok ? 64 | (L.rdir[srid[c]] ? 0 : 128) | ((X + Y + Z) & (S - 1)) << 8 : 0;
    }
    __syncthreads();
    // LDS offset of tap t (global order) from its vertex, whose x +- 1 lie at P, M
    auto tap = [](int t, int P, int M) __attribute__((always_inline)) -> int {
        if (t == 0) return 0;
        const int q = (t - 1) >> 1, m = q == 0 ? 1 : q == 1 ? 2 : q == 2 ? 4 : q == 3 ? 3 : q == 4 ? 6 : q == 5 ? 5 : 7;
        const bool plus = (t & 1) != 0;
        return (m & 1 ? (plus ? P : M) : 0) + (plus ? 1 : -1) * ((m & 2 ? SX : 0) + (m & 4 ? PS : 0));
    };
#define RIM_PM(c) const int P = sPM[c] >> 16, M = (int)(short)sPM[c]
    T t3[QR][3][V], s4[QR][V], st[SR][3], ss[SR];
    // addresses derived from these are formed anew in every pass: hoisted out
    // of the step loop they would not fit the registers
    // The constants come from the kernel's arguments again in every pass (more
    // than the scalar registers hold).
    const __attribute__((address_space(4))) Lat<T>* C =
        (const __attribute__((address_space(4))) Lat<T>*)__builtin_amdgcn_kernarg_segment_ptr();
    auto anew = [&]() __attribute__((always_inline)) {
        asm volatile("" : "+s"(C));
#pragma unroll
        for (int c = 0; c < QR; ++c) asm volatile("" : "+v"(qat[c]), "+v"(rot[c]), "+v"(gat[c]), "+v"(qpm[c]));
#pragma unroll
        for (int c = 0; c < SR; ++c) asm volatile("" : "+v"(sat[c]), "+v"(sok[c]), "+v"(sPM[c]), "+v"(scls[c]));
    };
    // differences over the opposite pairs at an interior vertex; every load
    // before the first use (the compiler would wait for each in turn)
    auto diffs1 = [&](const T* u, int P, int M, T d[7]) __attribute__((always_inline)) {
        const T v[14] = {u[P],         u[M],          u[SX],         u[-SX],         u[PS],
                         u[-PS],     u[P + SX],   u[M - SX],     u[SX + PS],   u[-SX - PS],
                         u[P + PS],  u[M - PS],   u[P + SX + PS], u[M - SX - PS]};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 7; ++q) d[q] = v[2 * q] - v[2 * q + 1];
    };
    // rows f - B^T p, by colour; with zero pressure just f
    auto form_t = [&](bool pz) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < QR; ++c) {
            if (rot[c] & 64) continue;
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int j = 0; j < V; ++j) t3[c][k][j] = b[k * len + gat[c] + lat_sub(j, L.Qp)];
            if (V == 1) {
                if (!pz) {
                    const int P = qpm[c] >> 16, M = (int)(short)qpm[c];
                    T d[7];
                    diffs1(pr + qat[c], P, M, d);
#pragma unroll
                    for (int k = 0; k < 3; ++k)
#pragma unroll
                        for (int q = 0; q < 7; ++q) t3[c][k][0] -= C->bt[k][q] * d[q];
                }
            } else {
                if (!pz) {
                    LdsRows<T> R;
                    lds_rows<GEO, 0>(pr + qat[c], R);
#pragma unroll
                    for (int k = 0; k < 3; ++k) lds_diff<0>(R, -C->bt[k][0], T(0), t3[c][k]);
                    lds_rows<GEO, 1>(pr + qat[c], R);
#pragma unroll
                    for (int k = 0; k < 3; ++k) lds_diff<1>(R, -C->bt[k][1], -C->bt[k][3], t3[c][k]);
                    lds_rows<GEO, 2>(pr + qat[c], R);
#pragma unroll
                    for (int k = 0; k < 3; ++k) lds_diff<2>(R, -C->bt[k][2], -C->bt[k][5], t3[c][k]);
                    lds_rows<GEO, 3>(pr + qat[c], R);
#pragma unroll
                    for (int k = 0; k < 3; ++k) lds_diff<3>(R, -C->bt[k][4], -C->bt[k][6], t3[c][k]);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) lat_rotate(t3[c][k], rot[c]);
            }
        }
        if (rim) {
#pragma unroll
            for (int c = 0; c < SR; ++c) {
                if (!(sok[c] & 128)) continue;
                RIM_PM(c);
                const T* cr = L.cls + (size_t)scls[c] * LC_SIZE + LC_BT;
#pragma unroll
                for (int k = 0; k < 3; ++k) st[c][k] = b[k * len + sga[c]];
                if (!pz)
#pragma unroll 3
                    for (int t = 0; t < 15; ++t) {
                        const T v = pr[sat[c] + tap(t, P, M)];
#pragma unroll
                        for (int k = 0; k < 3; ++k) st[c][k] -= cr[15 * k + t] * v;
                    }
            }
        }
    };
    // the vertices of colour col of interior item c: body(e, LDS offset, offsets of x +- 1)
    auto of_colour = [&](int c, int col, auto body) __attribute__((always_inline)) {
        if (V == 1) {
            if (rot[c] == col) body(0, qat[c], qpm[c] >> 16, (int)(short)qpm[c]);
            return;
        }
        if (rot[c] & 64) return;
#pragma unroll
        for (int e = col; e < V; e += S) {
            const int j = (e + rot[c]) & 3;
            if (j == 0 && !qok0[c]) continue;
            int P, M;
            lds_x_offsets<GEO>(j, &P, &M);
            body(e, qat[c] + GEO::off(j), P, M);
        }
    };
    auto vel = [&](auto colc) __attribute__((always_inline)) {
        constexpr int col = decltype(colc)::value;
#pragma unroll
        for (int c = 0; c < QR; ++c)
            of_colour(c, col, [&](int e, int at, int P, int M) __attribute__((always_inline)) {
                T w[6], inv;
                if (KIND == 0) {
                    inv = C->inva;
                } else {
                    const T* ra = L.axr + (size_t)rid[c][e] * LX_SIZE;
#pragma unroll
                    for (int q = 0; q < 6; ++q) w[q] = ra[LX_A + q];
                    inv = ra[LX_INVA];
                }
                T v[3], n[3][6];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const T* u = f0 + k * N + at;
                    n[k][0] = u[P];
                    n[k][1] = u[M];
                    n[k][2] = u[SX];
                    n[k][3] = u[-SX];
                    n[k][4] = u[PS];
                    n[k][5] = u[-PS];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (KIND == 0)
                        v[k] = t3[c][k][e] - C->a[0] * (n[k][0] + n[k][1]) - C->a[1] * (n[k][2] + n[k][3]) -
                               C->a[2] * (n[k][4] + n[k][5]);
                    else
                        v[k] = t3[c][k][e] - w[0] * n[k][0] - w[1] * n[k][1] - w[2] * n[k][2] - w[3] * n[k][3] -
                               w[4] * n[k][4] - w[5] * n[k][5];
#pragma unroll
                for (int k = 0; k < 3; ++k) f0[k * N + at] = v[k] * inv;
            });
        if (rim) {
#pragma unroll
            for (int c = 0; c < SR; ++c) {
                if (!(sok[c] & 128) || (sok[c] >> 8) != col) continue;
                RIM_PM(c);
                const T* ra = L.axr + (size_t)srid[c] * LX_SIZE;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    T v = st[c][k], n[6];
#pragma unroll
                    for (int t = 0; t < 6; ++t) n[t] = f0[k * N + sat[c] + tap(t + 1, P, M)];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int t = 0; t < 6; ++t) v -= ra[LX_A + t] * n[t];
                    f0[k * N + sat[c]] = v * ra[LX_INVA];
                }
            }
        }
        __syncthreads();
    };
    // (C p) at a vertex of an interior item
    auto cp_item = [&](int c, int e, int at, int P, int M, T* inv) __attribute__((always_inline)) -> T {
        const T* p = pr + at;
        const T n[7] = {p[0], p[P], p[M], p[SX], p[-SX], p[PS], p[-PS]};
        if (KIND == 0) {
            __builtin_amdgcn_sched_barrier(0);
            *inv = C->invc;
            return C->c0 * n[0] + C->c[0] * (n[1] + n[2]) + C->c[1] * (n[3] + n[4]) + C->c[2] * (n[5] + n[6]);
        }
        const T* ra = L.axr + (size_t)rid[c][e] * LX_SIZE;
        const T w[8] = {ra[LX_C0], ra[LX_C], ra[LX_C + 1], ra[LX_C + 2], ra[LX_C + 3], ra[LX_C + 4], ra[LX_C + 5],
                        ra[LX_INVC]};
        __builtin_amdgcn_sched_barrier(0);
        *inv = w[7];
        return w[0] * n[0] + w[1] * n[1] + w[2] * n[2] + w[3] * n[3] + w[4] * n[4] + w[5] * n[5] + w[6] * n[6];
    };
    // (C p) at surface vertex c
    auto cp_rim = [&](int c, T* inv) __attribute__((always_inline)) -> T {
        RIM_PM(c);
        const T* ra = L.axr + (size_t)srid[c] * LX_SIZE;
        T w[8], n[7];
#pragma unroll
        for (int t = 0; t < 8; ++t) w[t] = ra[LX_C + t];   // the six taps, the centre, 1 / centre
#pragma unroll
        for (int t = 0; t < 7; ++t) n[t] = pr[sat[c] + tap(t, P, M)];
        __builtin_amdgcn_sched_barrier(0);
        *inv = w[7];
        T cp = w[6] * n[0];
#pragma unroll
        for (int t = 0; t < 6; ++t) cp += w[t] * n[t + 1];
        return cp;
    };
    auto pres = [&](auto colc) __attribute__((always_inline)) {
        constexpr int col = decltype(colc)::value;
#pragma unroll
        for (int c = 0; c < QR; ++c)
            of_colour(c, col, [&](int e, int at, int P, int M) __attribute__((always_inline)) {
                T inv;
                const T cp = cp_item(c, e, at, P, M, &inv);
                pr[at] += omega * (s4[c][e] - cp) * inv;
            });
#pragma unroll
        for (int c = 0; c < SR; ++c) {
            if (!(sok[c] & 64) || (sok[c] >> 8) != col) continue;
            T inv;
            const T cp = cp_rim(c, &inv);
            pr[sat[c]] += omega * (ss[c] - cp) * inv;
        }
        __syncthreads();
    };
    // rows B u - g
    auto form_s = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < QR; ++c) {
            if (rot[c] & 64) continue;
#pragma unroll
            for (int j = 0; j < V; ++j) s4[c][j] = -b[3 * len + gat[c] + lat_sub(j, L.Qp)];
            if (V == 1) {
                const int P = qpm[c] >> 16, M = (int)(short)qpm[c];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    T d[7], e = T(0);
                    diffs1(f0 + k * N + qat[c], P, M, d);
#pragma unroll
                    for (int q = 0; q < 7; ++q) e += C->bt[k][q] * d[q];
                    s4[c][0] -= e;
                }
                continue;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                LdsRows<T> R;
                lds_rows<GEO, 0>(f0 + k * N + qat[c], R);
                lds_diff<0>(R, -C->bt[k][0], T(0), s4[c]);
                lds_rows<GEO, 1>(f0 + k * N + qat[c], R);
                lds_diff<1>(R, -C->bt[k][1], -C->bt[k][3], s4[c]);
                lds_rows<GEO, 2>(f0 + k * N + qat[c], R);
                lds_diff<2>(R, -C->bt[k][2], -C->bt[k][5], s4[c]);
                lds_rows<GEO, 3>(f0 + k * N + qat[c], R);
                lds_diff<3>(R, -C->bt[k][4], -C->bt[k][6], s4[c]);
            }
            lat_rotate(s4[c], rot[c]);
        }
#pragma unroll
        for (int c = 0; c < SR; ++c) {
            RIM_PM(c);
            T s = T(0);
            if (sok[c] & 64) s = -b[3 * len + sga[c]];
            if (sface[c] >= 0) {
                LatConst<T> cr = (LatConst<T>)(L.cls + (size_t)sface[c] * LC_SIZE + LC_B);
#pragma unroll 1
                for (int k = 0; k < 3; ++k) {
                    T n[15];
#pragma unroll
                    for (int t = 0; t < 15; ++t) n[t] = f0[k * N + sat[c] + tap(t, P, M)];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int t = 0; t < 15; ++t) s += cr[15 * k + t] * n[t];
                }
            } else if (sok[c] & 64) {
                const T* cr = L.cls + (size_t)scls[c] * LC_SIZE + LC_B;
                // fifteen coefficients in flight
#pragma unroll 1
                for (int k = 0; k < 3; ++k) {
                    T w[15], n[15];
#pragma unroll
                    for (int t = 0; t < 15; ++t) w[t] = cr[15 * k + t];
#pragma unroll
                    for (int t = 0; t < 15; ++t) n[t] = f0[k * N + sat[c] + tap(t, P, M)];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int t = 0; t < 15; ++t) s += w[t] * n[t];
                }
            }
            ss[c] = s;
        }
    };
    using std::integral_constant;
#pragma unroll 1
    for (int it = 0; it < steps; ++it)
#pragma unroll 1
        for (int i = 0; i < prog.n; ++i) {
            anew();
            switch (prog.op[i]) {
                case LOP_T: form_t(vo || (zero && it == 0)); break;
                case LOP_S: form_s(); break;
                case LOP_V: vel(integral_constant<int, 0>{}); break;
                case LOP_V + 1: vel(integral_constant<int, 1>{}); break;
                case LOP_P: pres(integral_constant<int, 0>{}); break;
                case LOP_P + 1: pres(integral_constant<int, 1>{}); break;
                default:
                    if constexpr (S == 4) {
                        if (prog.op[i] == LOP_V + 2) vel(integral_constant<int, 2>{});
                        else if (prog.op[i] == LOP_V + 3) vel(integral_constant<int, 3>{});
                        else if (prog.op[i] == LOP_P + 2) pres(integral_constant<int, 2>{});
                        else pres(integral_constant<int, 3>{});
                    }
            }
        }
    if (res) {
        // r = b - K x: the rows of the steps' functions, by colour position
        anew();
        form_t(vo != 0);
        anew();
        if (!vo) form_s();
        anew();
#pragma unroll
        for (int c = 0; c < QR; ++c)
#pragma unroll
            for (int col = 0; col < S; ++col)
                of_colour(c, col, [&](int e, int at, int P, int M) __attribute__((always_inline)) {
                    const int j = (e + rot[c]) & 3, a = gat[c] + (V == 4 ? lat_sub(j, L.Qp) : 0);
                    const T* ra = KIND == 1 ? L.axr + (size_t)rid[c][e] * LX_SIZE : nullptr;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const T* u = f0 + k * N + at;
                        T v = t3[c][k][e];
                        if (KIND == 0)
                            v -= C->a0 * u[0] + C->a[0] * (u[P] + u[M]) + C->a[1] * (u[SX] + u[-SX]) +
                                 C->a[2] * (u[PS] + u[-PS]);
                        else
                            v -= ra[LX_A0] * u[0] + ra[LX_A] * u[P] + ra[LX_A + 1] * u[M] +
                                 ra[LX_A + 2] * u[SX] + ra[LX_A + 3] * u[-SX] + ra[LX_A + 4] * u[PS] +
                                 ra[LX_A + 5] * u[-PS];
                        r[k * len + a] = v;
                    }
                    if (vo) return;
                    T inv;
                    r[3 * len + a] = cp_item(c, e, at, P, M, &inv) - s4[c][e];
                });
#pragma unroll
        for (int c = 0; c < SR; ++c) {
            if (!(sok[c] & 64)) continue;
            T inv;
            RIM_PM(c);
            if (!vo) r[3 * len + sga[c]] = cp_rim(c, &inv) - ss[c];
            const T* ra = L.axr + (size_t)srid[c] * LX_SIZE;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                T v = T(0);
                if (sok[c] & 128) {
                    v = st[c][k] - ra[LX_A0] * f0[k * N + sat[c]];
#pragma unroll
                    for (int t = 1; t < 7; ++t) v -= ra[LX_A + t - 1] * f0[k * N + sat[c] + tap(t, P, M)];
                }
                r[k * len + sga[c]] = v;
            }
        }
    }
    // steps end with a barrier
    copy([&](int i, int a) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < 3 || !vo) x[k * len + a] = f0[k * N + i];
    });
#undef RIM_PM
}

}  // namespace hhg
