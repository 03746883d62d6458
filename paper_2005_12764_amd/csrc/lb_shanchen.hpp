// lb_shanchen.hpp -- a step in the Shan-Chen interface model (Sec. 2.1,
// "Multi-component flows": the inter-component force of eq. shanchen_force with
// the exact-difference source of eq:edm), for raw (FP64/FP32) storage: one pass,
// or two.
//
// Two passes.  Density pass: the component densities (rho_r, rho_b) of every
// site of the current (post-streaming) state, as pairs.  Collide pass: 64-wide
// tiles marching a z-chunk with the density pairs of planes z-1, z, z+1 (tile
// plus one site) in an LDS ring; every site pulls its 19 populations per
// component, takes the two stencil sums sum_i w_i rho_k(x + c_i) c_i from the
// ring (mirror images beyond walls), collides (collide_sc) and stores.
//
// One pass (sc_step_kernel).  Each thread keeps the values it pulled for the
// densities of plane z + 1 until it collides that plane, so the state is read
// once and the densities never leave the LDS; the sites around the tile are
// pulled for their densities alone.
#pragma once
#include "lb_lean.hpp"

namespace lbm {

template <typename R>
struct RhoPair {
    R r, b;
};

template <typename R, typename Src>
__global__ __launch_bounds__(256) void sc_density_kernel(Geom g, Src src, RhoPair<R>* __restrict__ rho2) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.N) return;
    int x, y, z;
    site_xyz(g, s, x, y, z);
    R t[Q], d[Q];
    src.pull(g, s, x, y, z, t, d);
    R rc = R(0), dif = R(0);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        rc += weight<R>(i) + t[i];
        dif += d[i];
    }
    rho2[s] = RhoPair<R>{R(0.5) * (rc + dif), R(0.5) * (rc - dif)};
}

template <typename R>
__host__ __device__ constexpr size_t sc_ring_bytes(int TY, int TX) {
    return (size_t)3 * (TY + 2) * (TX + 2) * sizeof(RhoPair<R>);
}

template <typename R, typename Src, typename Dst, int TX>
__global__ __launch_bounds__(256) void sc_collide_kernel(Geom g, Src src, Dst dst, Coeffs<R> c, FusedShape fs,
                                                         const RhoPair<R>* __restrict__ rho2) {
    using L = Lattice;
    extern __shared__ unsigned char lds_raw[];
    RhoPair<R>* ring = reinterpret_cast<RhoPair<R>*>(lds_raw);
    constexpr int LX = TX + 2;
    const int TY = fs.TY, LY = TY + 2;
    const int tid = threadIdx.x, nt = blockDim.x;
    int x0, y0, za, zb;
    tile_of_block(fs, TX, g.nz, x0, y0, za, zb);
    for (int p = za - 1; p <= zb; ++p) {
        const int slot = (p - (za - 1)) % 3;
        {
            RhoPair<R>* dstp = ring + (size_t)slot * LY * LX;
            const int zz = halo_coord(p, g.nz, g.wz);
            for (int q = tid; q < LY * LX; q += nt) {
                const int ly = q / LX, lx = q - ly * LX;
                const int xx = halo_coord(x0 - 1 + lx, g.nx, g.wx);
                const int yy = halo_coord(y0 - 1 + ly, g.ny, g.wy);
                dstp[q] = rho2[site_of(g, xx, yy, zz)];
            }
        }
        __syncthreads();
        const int cz = p - 1;
        if (cz >= za) {
            const RhoPair<R>* pl[3] = {ring + (size_t)((cz - 1 - (za - 1)) % 3) * LY * LX,
                                       ring + (size_t)((cz - (za - 1)) % 3) * LY * LX,
                                       ring + (size_t)((cz + 1 - (za - 1)) % 3) * LY * LX};
            for (int q = tid; q < TY * TX; q += nt) {
                const int ty = q / TX, tx = q - ty * TX;
                const int x = x0 + tx, y = y0 + ty;
                if (x >= g.nx || y >= g.ny) continue;
                const int s = site_of(g, x, y, cz);
                R t[Q], d[Q];
                src.pull(g, s, x, y, cz, t, d);
                R bx = R(0), by = R(0), bz = R(0), rx = R(0), ry = R(0), rz = R(0);
#pragma unroll
                for (int i = 1; i < Q; ++i) {
                    const RhoPair<R> v = pl[1 + L::cz[i]][(ty + 1 + L::cy[i]) * LX + tx + 1 + L::cx[i]];
                    const R wb = weight<R>(i) * v.b, wr = weight<R>(i) * v.r;
                    if (L::cx[i]) { bx += L::cx[i] > 0 ? wb : -wb; rx += L::cx[i] > 0 ? wr : -wr; }
                    if (L::cy[i]) { by += L::cy[i] > 0 ? wb : -wb; ry += L::cy[i] > 0 ? wr : -wr; }
                    if (L::cz[i]) { bz += L::cz[i] > 0 ? wb : -wb; rz += L::cz[i] > 0 ? wr : -wr; }
                }
                collide_sc<R>(t, d, bx, by, bz, rx, ry, rz, c);
                dst.store(s, t, d, SiteTotals<R>{});
            }
        }
        __syncthreads();
    }
}

// One pass.  Bound by memory: 304 B per site and, for the 148 halo sites of a
// plane of 512 and the two planes more than a chunk writes, 45 % more reads, most
// of them from cache; 128^3 FP32 takes 163 us where the two passes take 214 (66 and
// 147), 256^3 1.07 ms against 1.52.  Two wavefronts per SIMD hold the values of
// planes z and z + 1 and those of z + 2 in flight (190 registers); four would
// spill (255 us).  The arithmetic is that of the two passes, value by value.
//
// Ring of the density pairs of four planes (one written while the three before
// it are read), tile plus one site.
constexpr int kScSlots = 4;
constexpr int kScRows = 8;  // one workgroup per CU, two wavefronts per SIMD (registers)
template <typename R>
constexpr size_t sc_step_bytes() {
    return (size_t)kScSlots * (kScRows + 2) * (kTileX + 2) * sizeof(RhoPair<R>);
}

template <typename R, typename Src, typename Dst, bool W>
__global__ __launch_bounds__(kTileX * kScRows, 2) void sc_step_kernel(Geom g, Src src, LeanPairs<R> rows_of, Dst dst,
                                                                Coeffs<R> c, FusedShape fs) {
    using L = Lattice;
    extern __shared__ unsigned char lds_raw[];
    RhoPair<R>* const ring = reinterpret_cast<RhoPair<R>*>(lds_raw);
    constexpr int TY = kScRows, LX = kTileX + 2, LY = TY + 2, PLANE = LY * LX;
    constexpr int HE = 2 * LX + 2 * TY;  // halo sites of a plane
    static_assert(HE <= kTileX * TY, "a tile's halo exceeds its threads");
    int x0, y0, za, zb;
    tile_of_block(fs, kTileX, g.nz, x0, y0, za, zb);
    const int lane = threadIdx.x & 63, ty = wave_uniform(threadIdx.x >> 6);
    const int x = x0 + lane, y = y0 + ty;
    const bool in = x < g.nx && y < g.ny;
    // (beyond the lattice: the site a neighbour's stencil reads there)
    const LeanLane ln = lean_lane(g, W, halo_coord(x, g.nx, g.wx), lane, ty);
    const LeanRowSet<W> rows(g, halo_coord(y, g.ny, g.wy));
    const int own = (ty + 1) * LX + lane + 1;
    // halo site of this thread
    const bool has_halo = threadIdx.x < HE;
    int hx, hy, halo;
    {
        const int e = min((int)threadIdx.x, HE - 1), e2 = e - 2 * LX;
        const int r = e2 < 0 ? (e < LX ? 0 : TY + 1) : 1 + (e2 >> 1);
        const int q = e2 < 0 ? (e < LX ? e : e - LX) : ((e2 & 1) ? kTileX + 1 : 0);
        hx = halo_coord(x0 - 1 + q, g.nx, g.wx);
        hy = halo_coord(y0 - 1 + r, g.ny, g.wy);
        halo = r * LX + q;
    }
    auto density = [](const R (&t)[Q], const R (&d)[Q]) {
        R rc = R(0), dif = R(0);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            rc += weight<R>(i) + t[i];
            dif += d[i];
        }
        return RhoPair<R>{R(0.5) * (rc + dif), R(0.5) * (rc - dif)};
    };
    auto plane = [&](int p) { return ring + ((p - za + 1) & (kScSlots - 1)) * PLANE; };
    R t[Q], d[Q], tn[Q], dn[Q];  // planes p - 1 and p
    auto pull = [&](int p) {
        rows_of.template values<W, TY>(g, rows.at(halo_plane(p, g.nz, g.wz)), ln,
                                       RecPlanes<typename LeanPairs<R>::C, 1, TY>{nullptr}, 0, 0, 0,
                                       typename LeanPairs<R>::Pre{}, [&](int i, R ti, R di) {
                                           tn[i] = ti;
                                           dn[i] = di;
                                       });
    };
    // (its slot of the ring is one the collision of plane p - 2 does not read)
    auto put_halo = [&](int p) {
        if (!has_halo) return;
        const int zz = halo_plane(p, g.nz, g.wz);
        R th[Q], dh[Q];
        src.pull(g, site_of(g, hx, hy, zz), hx, hy, zz, th, dh);
        plane(p)[halo] = density(th, dh);
    };
    pull(za - 1);
    put_halo(za - 1);
#pragma unroll 1
    for (int p = za - 1; p <= zb; ++p) {
        plane(p)[own] = density(tn, dn);
        __syncthreads();
        R tk[Q], dk[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            tk[i] = tn[i];
            dk[i] = dn[i];
        }
        pull(min(p + 1, zb));
        if (p < zb) put_halo(p + 1);
        const int cz = p - 1;
        if (cz >= za && in) {
            const RhoPair<R>* pl[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) pl[k] = plane(cz - 1 + k) + own;
            R bx = R(0), by = R(0), bz = R(0), rx = R(0), ry = R(0), rz = R(0);
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const RhoPair<R> v = pl[1 + L::cz[i]][L::cy[i] * LX + L::cx[i]];
                const R wb = weight<R>(i) * v.b, wr = weight<R>(i) * v.r;
                if (L::cx[i]) { bx += L::cx[i] > 0 ? wb : -wb; rx += L::cx[i] > 0 ? wr : -wr; }
                if (L::cy[i]) { by += L::cy[i] > 0 ? wb : -wb; ry += L::cy[i] > 0 ? wr : -wr; }
                if (L::cz[i]) { bz += L::cz[i] > 0 ? wb : -wb; rz += L::cz[i] > 0 ? wr : -wr; }
            }
            collide_sc<R>(t, d, bx, by, bz, rx, ry, rz, c);
            dst.store(site_of(g, x, y, cz), t, d, SiteTotals<R>{});
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            t[i] = tk[i];
            d[i] = dk[i];
        }
    }
}

}  // namespace lbm
