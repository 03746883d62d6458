// lb_single.hpp -- the one-read step: collide-and-stream tiles that also
// produce the phase-field sums of the next step.
//
// The phase field of a site is phi = D / Rc with D = sum_i d_i and
// Rc = sum_i (w_i + t_i) over its 19 pulled (post-streaming) populations.
// The collide pass writes those populations and holds them in registers, so
// each tile also sums, for every site of its own box, the terms whose source
// lies in the same box ("own" terms): a partial (D_own, Rc_own) per site.
// The terms whose source lies in another tile ("foreign": only sites on a
// face of their box have any) are pulled from the population arrays by a
// light assembly kernel that turns the partial sums of the face sites into
// phi; the tile writes phi of every other site itself.  Each
// population is read from HBM once per step (plus the few foreign ones),
// instead of once by a phase pass and again by the collide pass.
//
// The foreign terms that enter a site through an x face of its box all come
// from the one neighbouring tile column (a source that is also outside the
// y or z range of the box belongs to that face instead), so the tile holding
// those sources sums them per destination and stores the pair in a compact
// array after the own sums; the assembly reads one pair per x-face site
// instead of ten scattered values (rows are contiguous in x, so the y and z
// faces pull whole rows and keep the direct reads).
//
// Summation order is fixed, so results are reproducible: the own terms of a
// site in four groups -- sources in plane z-1, bounce-backs from the site
// itself (ascending direction), in-plane sources, sources in plane z+1 -- the
// groups of a plane by source row (the site's own, below, above), each row's
// terms first summed over its columns (the site's own, left, right); then the
// foreign terms of the z and the y faces, each in
// ascending direction; then the x-face sums (lo face, then hi face), each
// summed from zero in the group order of the own terms.  D and Rc are summed
// term by term alike, so a pure component (d_i = +-(w_i + t_i)) gives
// phi = +-1 exactly, as in the collision.
#pragma once
#include <type_traits>

#include "lb_fused.hpp"

namespace lbm {

// Own partial sums of one site.
template <typename R>
struct Part2 {
    R dn, rc;
};

// A phase-sum buffer holds, for one state: the own sums of the sites on a
// face of their box (N pairs, indexed by site), the x-face sums of every tile
// column (2 faces x ny x nz pairs), and the phase field (N values).  The tile
// kernel writes phi itself for the sites whose every term is its own; the
// assembly completes the face sites.
template <int TX>
__host__ __device__ constexpr size_t xface_entries(int nx, int ny, int nz) {
    return (size_t)2 * ((nx + TX - 1) / TX) * ny * nz;
}
// Size of a phase-sum buffer in reals.
template <int TX>
__host__ __device__ constexpr size_t part_reals(int nx, int ny, int nz) {
    return 2 * ((size_t)nx * ny * nz + xface_entries<TX>(nx, ny, nz)) + (size_t)nx * ny * nz;
}
// The phase field of a phase-sum buffer.
template <int TX, typename R>
__host__ __device__ __forceinline__ R* phi_of(Part2<R>* part, const Geom& g) {
    return reinterpret_cast<R*>(part + (size_t)g.N + xface_entries<TX>(g.nx, g.ny, g.nz));
}

// Is the site a face site of its box (some source of its phase sums may lie
// in another box)?  x % TX, y % TY: position in the tile; za, zb: the chunk.
template <int TX, int TY>
__device__ __forceinline__ bool on_face(const Geom& g, int x, int y, int z, int za, int zb) {
    const int rx = x % TX, ry = y % TY;
    return rx == 0 || rx == TX - 1 || x == g.nx - 1 || ry == 0 || ry == TY - 1 || y == g.ny - 1 || z == za ||
           z == zb - 1;
}

// x-face sum of the site (x, y, z) on the lo (side 0, x = bx * TX) or hi
// (side 1) x face of tile column bx, in the compact array after the own sums.
__device__ __forceinline__ unsigned xface_at(const Geom& g, int bx, int side, int y, int z) {
    return (unsigned)(((bx * 2 + side) * g.nz + z) * g.ny + y);
}

// Direction with velocity (cx, cy, cz), -1 if there is none (a switch, which
// folds for constant arguments).
__host__ __device__ constexpr int dir_of(int cx, int cy, int cz) {
    switch ((cx + 1) + 3 * (cy + 1) + 9 * (cz + 1)) {
        case 13: return 0;
        case 14: return 1;
        case 12: return 2;
        case 16: return 3;
        case 10: return 4;
        case 22: return 5;
        case 4: return 6;
        case 17: return 7;
        case 9: return 8;
        case 11: return 9;
        case 15: return 10;
        case 23: return 11;
        case 3: return 12;
        case 5: return 13;
        case 21: return 14;
        case 25: return 15;
        case 1: return 16;
        case 7: return 17;
        case 19: return 18;
    }
    return -1;
}

// Rows of the one-read tile (one site per thread and plane); 12 in 16-bit
// storage only, whose records leave no LDS for 16 with a near-contact halo.
constexpr int kSingleTY = 8;
constexpr int kSingleTYSmall = 4;
constexpr int kSingleTYSplit = 12;
constexpr int kSingleTYLarge = 16;
// f(std::integral_constant<int, TY>) for a row count of the one-read tile.
template <typename F>
int with_rows(int TY, const F& f) {
    switch (TY) {
        case kSingleTYSmall: return f(std::integral_constant<int, kSingleTYSmall>());
        case kSingleTY: return f(std::integral_constant<int, kSingleTY>());
        case kSingleTYSplit: return f(std::integral_constant<int, kSingleTYSplit>());
        case kSingleTYLarge: return f(std::integral_constant<int, kSingleTYLarge>());
    }
    return -1;
}
constexpr int kTileX = 64;             // columns of a tile: one wavefront per row
constexpr size_t kLdsBytes = 163840;   // LDS of a workgroup on gfx950

// Own box of a site: its tile column [x0, x1) x [y0, y1) and z chunk [z0, z1).
struct OwnBox {
    int x0, x1, y0, y1, z0, z1;
};

template <int TX, int TY>
__device__ __forceinline__ OwnBox box_of(const Geom& g, int TZ, int x, int y, int z) {
    OwnBox b;
    b.x0 = x - x % TX;
    b.x1 = min(b.x0 + TX, g.nx);
    b.y0 = y - y % TY;
    b.y1 = min(b.y0 + TY, g.ny);
    b.z0 = z - z % TZ;
    b.z1 = min(b.z0 + TZ, g.nz);
    return b;
}

// Group of direction i at a destination, in summation order: 0 = source in
// plane z-1, 1 = reflected from the site itself, 2 = in-plane source, 3 =
// source in plane z+1.
__device__ __forceinline__ int group_of(int i, bool reflected) {
    return reflected ? 1 : (Lattice::cz[i] > 0 ? 0 : (Lattice::cz[i] == 0 ? 2 : 3));
}

// Terms entering the site (x, y, z) with c_x = SX through its x face whose
// source lies within the y and z range of the site's box b, summed from zero
// in the group order of the own terms (sources in plane z-1, in-plane
// sources, sources in plane z+1), each group in ascending direction.
template <typename R, int SX, typename Src>
__device__ __forceinline__ Part2<R> xface_sum(const Geom& g, const Src& src, const OwnBox& b, int s, int x, int y,
                                             int z) {
    using L = Lattice;
    R dn = R(0), rc = R(0);
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            if (L::cx[i] != SX || group_of(i, false) != grp) continue;
            const int ys = y - L::cy[i], zs = z - L::cz[i];
            if (ys < b.y0 || ys >= b.y1 || zs < b.z0 || zs >= b.z1) continue;
            int dir;
            const int sr = pull_source(g, i, x, y, z, s, dir);
            if (dir != i) continue;
            R t, d;
            src.template pull_one<R>(i, sr, dir, t, d);
            rc += weight<R>(i) + t;
            dn += d;
        }
    }
    return Part2<R>{dn, rc};
}

// Own partial sums (phi where they are complete) and x-face sums of the
// current state, for a state that no one-read step produced (initial,
// imported, or left by a two-pass step).
template <typename R, typename Src, int TX, int TY>
__global__ __launch_bounds__(256) void part_kernel(Geom g, Src src, int TZ, Part2<R>* __restrict__ part) {
    using L = Lattice;
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.N) return;
    int x, y, z;
    site_xyz(g, s, x, y, z);
    const OwnBox b = box_of<TX, TY>(g, TZ, x, y, z);
    R dn = R(0), rc = R(0);
    // own terms from the row (y - e, z - f), summed over its columns
    auto row_terms = [&](int e, int f) {
        if (y - e < b.y0 || y - e >= b.y1 || z - f < b.z0 || z - f >= b.z1) return;
        R rd = R(0), rr = R(0);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int cx = k == 2 ? -1 : k, i = dir_of(cx, e, f);
            if (i < 0) continue;
            if (x - cx < b.x0 || x - cx >= b.x1) continue;
            R t, d;
            src.template pull_one<R>(i, site_of(g, x - cx, y - e, z - f), i, t, d);
            rr += weight<R>(i) + t;
            rd += d;
        }
        rc += rr;
        dn += rd;
    };
    auto plane_terms = [&](int f) {
        row_terms(0, f);
        row_terms(1, f);
        row_terms(-1, f);
    };
    plane_terms(1);
    R ph = R(0);  // own post-collision phase, for the moving-wall terms
    bool have_ph = false;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        int dir;
        const int sr = pull_source(g, i, x, y, z, s, dir);
        if (dir == i) continue;
        R t, d;
        src.template pull_one<R>(i, sr, dir, t, d);
        if constexpr (Src::moving) {
            // a reflection off a moving wall, as the pull adds it
            if (g.moving) {
                if (!have_ph) {
                    ph = src.template own_phase<R>(s);
                    have_ph = true;
                }
                const R add = wall_term<R>(g, i, x, y, z);
                t += add;
                d = fma_of(add, ph, d);
            }
        }
        rc += weight<R>(i) + t;
        dn += d;
    }
    plane_terms(0);
    plane_terms(-1);
    if (on_face<TX, TY>(g, x, y, z, b.z0, b.z1)) part[s] = Part2<R>{dn, rc};
    else phi_of<TX>(part, g)[s] = dn / rc;
    // x-face sums of this site (beyond an x wall every term is a bounce-back)
    Part2<R>* xf = part + g.N;
    const bool lo = x % TX == 0 && !(g.wx && x == 0);
    const bool hi = (x % TX == TX - 1 || x == g.nx - 1) && !(g.wx && x == g.nx - 1);
    if (lo) xf[xface_at(g, x / TX, 0, y, z)] = xface_sum<R, 1>(g, src, b, s, x, y, z);
    if (hi) xf[xface_at(g, x / TX, 1, y, z)] = xface_sum<R, -1>(g, src, b, s, x, y, z);
}

// Faces of a site's own box along one axis: lo = first coordinate of its
// tile (sources at v - 1 lie outside), hi = last (sources at v + 1 outside).
struct Faces {
    bool lo, hi;
};
template <int T>
__device__ __forceinline__ Faces faces_of(int v, int n) {
    const int r = v % T;
    return Faces{r == 0, r == T - 1 || v == n - 1};
}
__device__ __forceinline__ Faces faces_z(int v, int z0, int z1) { return Faces{v == z0, v == z1 - 1}; }

// Does direction i leave the box through the faces f (c > 0 enters through
// lo, c < 0 through hi)?
__device__ __forceinline__ bool leaves(int c, const Faces& f) { return (c > 0 && f.lo) || (c < 0 && f.hi); }

// Foreign terms of site s = (x, y, z) whose source lies outside the box
// through the faces of `axis` (1 = y, 2 = z) and not through those of an
// axis summed before it (z, then y); bounce-backs are own terms.
template <typename R, typename Src, int AXIS>
__device__ __forceinline__ void foreign_terms(const Geom& g, const Src& src, int s, int x, int y, int z,
                                              const Faces& fy, const Faces& fz, R& dn, R& rc) {
    using L = Lattice;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const bool oz = leaves(L::cz[i], fz), oy = leaves(L::cy[i], fy);
        const bool mine = AXIS == 2 ? oz : (oy && !oz);
        if (!mine) continue;
        int dir;
        const int sr = pull_source(g, i, x, y, z, s, dir);
        if (dir != i) continue;
        R t, d;
        src.template pull_one<R>(i, sr, dir, t, d);
        rc += weight<R>(i) + t;
        dn += d;
    }
}

// Coordinates along an axis of extent n cut into boxes of T, ranked: the
// face coordinates (first and last of each box) and the inner ones.
struct AxisFaces {
    int n, T;
    __host__ __device__ int nface() const {
        if (T <= 2) return n;
        const int r = n % T;
        return 2 * (n / T) + (r == 0 ? 0 : (r == 1 ? 1 : 2));
    }
    __host__ __device__ int face(int k) const {
        if (T <= 2) return k;
        const int b = k >> 1, rest = n - b * T, size = rest < T ? rest : T;
        return b * T + ((k & 1) ? size - 1 : 0);
    }
    __host__ __device__ int inner(int m) const { return (m / (T - 2)) * T + m % (T - 2) + 1; }
};

// The face sites of the boxes, enumerated for the assembly: first every
// site of the face rows (the rows of a chunk's z faces, then the rows of a
// tile's y faces in the other planes), then the x-face sites of the
// remaining rows.
struct FaceSet {
    AxisFaces ax, ay, az;
    int nyf, nyi, nzf, nxf;
    int row_sites, edge_sites;
};
inline FaceSet face_set(const Geom& g, int TX, int TY, int TZ) {
    FaceSet f;
    f.ax = AxisFaces{g.nx, TX};
    f.ay = AxisFaces{g.ny, TY};
    f.az = AxisFaces{g.nz, TZ};
    f.nxf = f.ax.nface();
    f.nyf = f.ay.nface();
    f.nyi = g.ny - f.nyf;
    f.nzf = f.az.nface();
    const int nzi = g.nz - f.nzf;
    f.row_sites = (f.nzf * g.ny + nzi * f.nyf) * g.nx;
    f.edge_sites = nzi * f.nyi * f.nxf;
    return f;
}

// phi of the face sites from their own partial sums, the foreign terms of
// the z and y faces and the x-face sums.
template <typename R, typename Src, int TX, int TY>
__device__ __forceinline__ void assemble_site(const Geom& g, const Src& src, const FaceSet& fs,
                                              Part2<R>* __restrict__ part, int k) {
    int x, y, z;
    if (k < fs.row_sites) {
        const int r = k / g.nx, zrows = fs.nzf * g.ny;
        x = k - r * g.nx;
        if (r < zrows) {
            z = fs.az.face(r / g.ny);
            y = r - (r / g.ny) * g.ny;
        } else {
            const int r2 = r - zrows;
            z = fs.az.inner(r2 / fs.nyf);
            y = fs.ay.face(r2 - (r2 / fs.nyf) * fs.nyf);
        }
    } else {
        const int k2 = k - fs.row_sites;
        if (k2 >= fs.edge_sites) return;
        const int q = k2 / fs.nxf;
        x = fs.ax.face(k2 - q * fs.nxf);
        z = fs.az.inner(q / fs.nyi);
        y = fs.ay.inner(q - (q / fs.nyi) * fs.nyi);
    }
    const int s = site_of(g, x, y, z);
    const int TZ = fs.az.T, z0 = z - z % TZ;
    const Faces fx = faces_of<TX>(x, g.nx), fy = faces_of<TY>(y, g.ny), fz = faces_z(z, z0, min(z0 + TZ, g.nz));
    const Part2<R> P = part[s];
    R dn = P.dn, rc = P.rc;
    if (fz.lo || fz.hi) foreign_terms<R, Src, 2>(g, src, s, x, y, z, fy, fz, dn, rc);
    if (fy.lo || fy.hi) foreign_terms<R, Src, 1>(g, src, s, x, y, z, fy, fz, dn, rc);
    const Part2<R>* xf = part + g.N;
    if (fx.lo && !(g.wx && x == 0)) {
        const Part2<R> X = xf[xface_at(g, x / TX, 0, y, z)];
        dn += X.dn;
        rc += X.rc;
    }
    if (fx.hi && !(g.wx && x == g.nx - 1)) {
        const Part2<R> X = xf[xface_at(g, x / TX, 1, y, z)];
        dn += X.dn;
        rc += X.rc;
    }
    phi_of<TX>(part, g)[s] = dn / rc;
}

// Face site k of the enumeration above, one per thread.
template <typename R, typename Src, int TX, int TY>
__global__ __launch_bounds__(256) void assemble_kernel(Geom g, Src src, FaceSet fs, Part2<R>* __restrict__ part) {
    assemble_site<R, Src, TX, TY>(g, src, fs, part, blockIdx.x * blockDim.x + threadIdx.x);
}

// Column an edge lane's x-face sums go to: the lo edge lane (SX = -1) feeds the
// hi face of the column on its left, the hi edge lane (SX = +1) the lo face of
// the one on its right (periodic wrap; none beyond an x wall).
template <int TX>
__device__ __forceinline__ bool xface_dest(const Geom& g, int x0, int x1, int SX, int& bd) {
    if (SX < 0) {
        if (x0 > 0) {
            bd = x0 / TX - 1;
            return true;
        }
        bd = (g.nx + TX - 1) / TX - 1;
        return !g.wx;
    }
    if (x1 < g.nx) {
        bd = x0 / TX + 1;
        return true;
    }
    bd = 0;
    return !g.wx;
}

}  // namespace lbm
