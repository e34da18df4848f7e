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
#pragma once
#include <hip/hip_runtime.h>

#include "hhg_internal.hpp"

namespace hhg {

// surface records (global tap order) and axis records
constexpr int LR_A = 0, LR_C = 15, LR_B = 30, LR_BT = 75, LR_INVA = 120, LR_INVC = 121, LR_MASS = 122,
              LR_SIZE = 124;
constexpr int LX_A = 0, LX_INVA = 6, LX_C = 8, LX_C0 = 14, LX_INVC = 15, LX_A0 = 7, LX_SIZE = 16;
constexpr int LPAT = 216;   // record patterns per cell

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

// item / d for items below 2^21 (host-checked), inv = 1 / d
__host__ __device__ __forceinline__ int lat_div(int item, float inv) {
    return (int)(((float)item + 0.5f) * inv);
}

// Tiles of a volume launch: `per` blocks of bs lanes cover the interior rows of
// a plane.  The planes are cut into eight slabs of ZB, one per XCD (workgroup b
// runs on XCD b mod 8); inside a slab, G blocks of a plane (about 2048 lanes)
// are followed by the same rows of the next plane, so that the rows y +- 1 and
// z +- 1 of a tile are still in its XCD's L2.  Measured at 8 refinements (17 M
// vertices, FP64): plane by plane the velocity sweep fetched twice its bytes.
struct LatGrid {
    int per, G, NG, ZB, total, bs;
};
// lanes: row lanes of a plane
__host__ __device__ __forceinline__ LatGrid lat_grid(int lanes, int planes, int bs) {
    LatGrid g;
    const int per = (lanes + bs - 1) / bs;
    g.bs = bs;
    g.per = per;
    g.NG = (per + 7) / 8;
    g.G = (per + g.NG - 1) / g.NG;
    g.ZB = (planes + 7) / 8;
    g.total = 8 * g.NG * g.ZB * g.G;
    return g;
}
struct LatTile {
    int t;          // natural index (partial sums)
    int z, part;    // interior plane and block of the plane
    bool ok;
};
__host__ __device__ __forceinline__ LatTile lat_tile(const LatGrid& g, int planes, int v, int order) {
    const int slab = g.NG * g.ZB * g.G;
    LatTile T;
    T.t = order == 2 ? g.total - 1 - v : order == 0 ? v : (v & 7) * slab + (v >> 3);
    const int zb = T.t / slab, i = T.t - zb * slab, zg = g.ZB * g.G;
    const int gp = i / zg, r = i - gp * zg, zi = r / g.G;
    T.z = zb * g.ZB + zi;
    T.part = gp * g.G + (r - zi * g.G);
    T.ok = T.z < planes && T.part < g.per;
    return T;
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
    const int row = lat_div(item, 1.0f / (float)lpr), li = item - row * lpr;
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
    const int row = lat_div(item, 1.0f / (float)L.Qi);
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

// ---------------------------------------------------------------------------
// Velocity sweep of one parity or colour (Section 3.5): u_k <- (f_k - (B^T p)_k
// - sum A u_k) / A_xx.  The B^T p rows are formed on the fly from p instead of
// being stored by a pass of their own: a parity launch then moves 5.5 values
// per vertex (p, half of u read, of f read, of u written) instead of 4.5, and
// the 10 values of that pass are gone.  PZ: p = 0 (the iterate starts at 0).
// ---------------------------------------------------------------------------
template <typename T, int KIND, int NC, bool PZ>
__global__ void __launch_bounds__(256) k_lat_vel(Lat<T> L, LatSurf B, int col, int sb, LatGrid tg,
                                                 const T* __restrict__ b, T* __restrict__ x) {
    const size_t len = L.len;
    const T* __restrict__ p = x + 3 * len;
    if ((int)blockIdx.x < sb) {
        int X, Y, Z;
        if (!lat_surf_lane(L, B, 4 / NC, col, (int)blockIdx.x * tg.bs + (int)threadIdx.x, &X, &Y, &Z)) return;
        const int id = L.rid[lat_rid_index(L, X, Y, Z)];
        if (L.rdir[id]) return;
        const T* __restrict__ r = L.rec + (size_t)id * LR_SIZE;
        int nb[15];
        lat_taps(L, X, Y, Z, nb);
        for (int k = 0; k < 3; ++k) {
            T acc = b[k * len + nb[0]];
            if (!PZ)
                for (int g = 0; g < 15; ++g) acc -= r[LR_BT + 15 * k + g] * p[nb[g]];
            for (int g = 1; g < 7; ++g) acc -= r[LR_A + g] * x[k * len + nb[g]];
            x[k * len + nb[0]] = acc * r[LR_INVA];
        }
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
// vertices that a later sweep relaxes (all of them with ALL).
// ---------------------------------------------------------------------------
template <typename T, int KIND, int NC>
__global__ void __launch_bounds__(256) k_lat_bp(Lat<T> L, LatSurf B, int col, int sb, LatGrid tg,
                                                const T* __restrict__ b, T* __restrict__ x,
                                                T* __restrict__ sx, T omega, int all) {
    const size_t len = L.len;
    T* __restrict__ p = x + 3 * len;
    const T* __restrict__ g = b + 3 * len;
    const int cm = NC == 2 ? 1 : 3;
    if ((int)blockIdx.x < sb) {
        int X, Y, Z;
        if (!lat_surf_lane(L, B, 1, 0, (int)blockIdx.x * tg.bs + (int)threadIdx.x, &X, &Y, &Z)) return;
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
        return;
    }
    const LatTile tile = lat_tile(tg, L.nz - 2, (int)blockIdx.x - sb, L.order);
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

// pressure sweep of one parity or colour: p += omega (s - C p) / C_xx
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
// r = b - K x (Dirichlet velocity rows 0).  WR: r is stored; NRM: per-block
// partial sums of r^2 at partials[tile] (volume) and partials[total + block]
// (surface), independent of the workgroup order.
// ---------------------------------------------------------------------------
template <typename T, int KIND, bool WR, bool NRM>
__global__ void __launch_bounds__(256) k_lat_res(Lat<T> L, LatSurf B, int sb, LatGrid tg,
                                                 const T* __restrict__ b, const T* __restrict__ x,
                                                 T* __restrict__ r, double* __restrict__ partials) {
    __shared__ double sh[4];
    const size_t len = L.len;
    const T* __restrict__ p = x + 3 * len;
    double acc = 0.0;
    int slot = -1;
    if ((int)blockIdx.x < sb) {
        if ((int)blockIdx.x * tg.bs < B.beg[6]) slot = tg.total + (int)blockIdx.x;
        int X, Y, Z;
        if (lat_surf_lane(L, B, 1, 0, (int)blockIdx.x * tg.bs + (int)threadIdx.x, &X, &Y, &Z)) {
            const int id = L.rid[lat_rid_index(L, X, Y, Z)];
            const T* __restrict__ rc = L.rec + (size_t)id * LR_SIZE;
            int nb[15];
            lat_taps(L, X, Y, Z, nb);
            T v = b[3 * len + nb[0]];
#pragma unroll
            for (int t = 0; t < 7; ++t) v += rc[LR_C + t] * p[nb[t]];
#pragma unroll 1
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int t = 0; t < 15; ++t) v -= rc[LR_B + 15 * k + t] * x[k * len + nb[t]];
            if (WR) r[3 * len + nb[0]] = v;
            if (NRM) acc += (double)v * (double)v;
            const bool dir = L.rdir[id] != 0;
#pragma unroll 1
            for (int k = 0; k < 3; ++k) {
                T w = T(0);
                if (!dir) {
                    w = b[k * len + nb[0]];
#pragma unroll
                    for (int t = 0; t < 15; ++t) w -= rc[LR_BT + 15 * k + t] * p[nb[t]];
                    for (int t = 0; t < 7; ++t) w -= rc[LR_A + t] * x[k * len + nb[t]];
                }
                if (WR) r[k * len + nb[0]] = w;
                if (NRM) acc += (double)w * (double)w;
            }
        }
    } else {
        const LatTile tile = lat_tile(tg, L.nz - 2, (int)blockIdx.x - sb, L.order);
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
                    const T v = ld1(b + k * len, a) - bt - au;
                    if (j > 0 || first) {
                        if (WR) st1(r + k * len, a, v);
                        if (NRM) acc += (double)v * (double)v;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int a = at + lat_sub(j, Qp);
                const T v = ld1(b + 3 * len, a) + rp[j];
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
// Restriction bc = P^T rf (weights 1 and 1/2, Dirichlet velocity rows 0), with
// the coarse iterate xc set to 0 in the same pass.  Interior lanes: the coarse
// quad q reads the fine row segments 8 q - 1 .. 8 q + 7 as pairs.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) k_lat_restrict(Lat<T> C, Lat<T> F, LatSurf B, int sb, LatGrid tg,
                                                      const T* __restrict__ rf, T* __restrict__ bc,
                                                      T* __restrict__ xc) {
    const size_t lc = C.len, lf = F.len;
    if ((int)blockIdx.x < sb) {
        int X, Y, Z;
        if (!lat_surf_lane(C, B, 1, 0, (int)blockIdx.x * tg.bs + (int)threadIdx.x, &X, &Y, &Z)) return;
        const bool dir = C.rdir[C.rid[lat_rid_index(C, X, Y, Z)]] != 0;
        const int a = lat_at(C, X, Y, Z);
        int nb[15];
        lat_taps(F, 2 * X, 2 * Y, 2 * Z, nb);
        for (int f = 0; f < 4; ++f) {
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
    const LatTile tile = lat_tile(tg, C.nz - 2, (int)blockIdx.x - sb, C.order);
    if (!tile.ok) return;
    const LatPair P = lat_quad_lane(C, tg, tile, threadIdx.x);
    if (!P.ok) return;
    typedef typename V2<T>::type v2;
    const int at = (P.z * C.ny + P.y) * C.RS + P.q;
    const int fa = (2 * P.z * F.ny + 2 * P.y) * F.RS + 2 * P.q;
#pragma unroll 1
    for (int f = 0; f < 4; ++f) {
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
// coarse vertices (X - d) / 2 and (X + d) / 2.
template <typename T, bool SET>
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
    T e[4][4], xv[4][4];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
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
    for (int f = 0; f < 4; ++f)
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
// Out: one lane per slot (every copy is written; padding untouched).
template <typename T>
__global__ void __launch_bounds__(256) k_lat_in(Lat<T> L, const int* __restrict__ node_slot,
                                                const double* __restrict__ v, size_t plen,
                                                T* __restrict__ x) {
    const int item = (int)blockIdx.x * 256 + (int)threadIdx.x, z = (int)blockIdx.y;
    const int y = lat_div(item, 1.0f / (float)L.nx), X = item - y * L.nx;
    if (y >= L.ny) return;
    const int s = node_slot[(size_t)(z * L.ny + y) * L.nx + X], a = lat_at(L, X, y, z);
#pragma unroll
    for (int f = 0; f < 4; ++f) x[f * L.len + a] = (T)v[f * plen + s];
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

}  // namespace hhg
