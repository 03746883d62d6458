// lb_pull.hpp -- the post-streaming populations of a packed or 16-bit state,
// handed site by site to a reader: moments, export, totals, where tiles fill their
// lanes (lb_pull.hip has the rule).
//
// A site's 19 values need the records of its 19 source sites.  Gathered per
// site they cost 16-bit states 19 record reads from L2 (256^3 fp16: 2.38 ms for the
// moments, more than two steps); here tiles march a z-chunk with the records of planes
// z - 1, z, z + 1 in an LDS ring, as the step's tiles do, so that each value is
// read once: 112 B per site and the fields written for FP32 moments.  Four ring
// slots, so that one barrier per plane is enough: a slot is written two planes
// after its last reader.
#pragma once
#include "lb_lean.hpp"

namespace lbm {

// Rows of a pulling tile: 8, or 4 where a record takes 32 bytes (two or three
// workgroups per CU then overlap their loads and stores).
template <typename S>
constexpr int pull_rows() {
    return S::NC == 1 ? 8 : 4;
}
constexpr int kPullSlots = 4;
// Planes of a chunk: 16, fewer where that leaves under two workgroups per CU (a
// chunk costs two planes of records beyond its own: 64^3 FP32 takes 38 us with
// 16 planes, 32 workgroups).
constexpr int kPullPlanes = 16, kPullBlocks = 512;
template <typename S>
constexpr size_t pull_lds() {
    return kPullSlots * RecPlanes<typename S::C, S::NC, pull_rows<S>()>::plane_bytes;
}
inline FusedShape pull_shape(const Geom& g, int rows) {
    FusedShape fs;
    fs.TY = rows;
    fs.tiles_x = (g.nx + kTileX - 1) / kTileX;
    fs.tiles_y = (g.ny + rows - 1) / rows;
    const long long planes = (long long)fs.tiles_x * fs.tiles_y * g.nz / kPullBlocks;
    fs.TZ = planes < 1 ? 1 : (int)(planes < kPullPlanes ? planes : kPullPlanes);
    fs.chunks = (g.nz + fs.TZ - 1) / fs.TZ;
    fs.nblocks = fs.tiles_x * fs.tiles_y * fs.chunks;
    return fs;
}

// Every site of one tile to read(site, t, d).  Every thread must call it.
template <typename S, bool W, bool MV, typename Read>
__device__ __forceinline__ void pull_tile(const Geom& g, const S& src, unsigned char* lds, int x0, int y0, int za,
                                          int zb, const Read& read) {
    using R = typename S::R;
    using C = typename S::C;
    constexpr int TY = pull_rows<S>();
    const RecPlanes<C, S::NC, TY> rp{reinterpret_cast<C*>(lds)};
    const int lane = threadIdx.x & 63;
    const int ty = wave_uniform(threadIdx.x >> 6);
    const int x = x0 + lane, y = y0 + ty;
    const bool site_in = x < g.nx && y < g.ny;
    const int xc = min(x, g.nx - 1), yc = min(y, g.ny - 1);
    const LeanLane ln = lean_lane(g, W, xc, lane, ty);
    const LeanRowSet<W> rows(g, yc);
    const RecStage<S, TY> recs(g, x0, y0, lane, ty,
                               (unsigned)(halo_coord(y, g.ny, g.wy) * g.nx + halo_coord(x, g.nx, g.wx)));
    typename RecStage<S, TY>::Regs next;
    typename S::Pre pre;
    {
        typename RecStage<S, TY>::Regs a, b;
        recs.load(g, src, za - 1, a);
        recs.load(g, src, za, b);
        recs.load(g, src, za + 1, next);
        src.template fetch<W, false>(g, rows.at(za), ln, pre);
        recs.put(rp, 0, a);
        recs.put(rp, 1, b);
    }
    for (int cz = za; cz < zb; ++cz) {
        const int k = (cz - za) & (kPullSlots - 1);  // slot of plane cz - 1
        const int k1 = (k + 1) & (kPullSlots - 1), k2 = (k + 2) & (kPullSlots - 1);
        recs.put(rp, k2, next);
        __syncthreads();
        const LeanRows rw = rows.at(cz);
        R t[Q], d[Q];
        MovingTerms<R> mt;
        if constexpr (W && MV) mt.template init<S, TY>(g, src, rw, ln, rp, k1);
        src.template values<W, TY>(g, rw, ln, rp, k, k1, k2, pre, [&](int i, R ti, R di) {
            if constexpr (W && MV) mt.add(g, i, rw, ln, yc, cz, ti, di);
            t[i] = ti;
            d[i] = di;
        });
        recs.load(g, src, cz + 2, next);
        src.template fetch<W, false>(g, rows.at(min(cz + 1, g.nz - 1)), ln, pre);
        if (site_in) read((int)(rw.own() + ln.c0), t, d);
    }
}

template <typename S, bool W, bool MV, typename Out>
__global__ __launch_bounds__(kTileX * pull_rows<S>()) void pull_moments_kernel(Geom g, S src, FusedShape fs, Out* rr,
                                                                              Out* rb, Out* j) {
    using R = typename S::R;
    extern __shared__ unsigned char lds_raw[];
    int x0, y0, za, zb;
    tile_of_block(fs, kTileX, g.nz, x0, y0, za, zb);
    pull_tile<S, W, MV>(g, src, lds_raw, x0, y0, za, zb, [&](int s, const R (&t)[Q], const R (&d)[Q]) {
        put_moments<R>(g, s, t, d, rr, rb, j);
    });
}

template <typename S, bool W, typename Out>
__global__ __launch_bounds__(kTileX * pull_rows<S>()) void pull_export_kernel(Geom g, S src, FusedShape fs, Out* out) {
    using R = typename S::R;
    extern __shared__ unsigned char lds_raw[];
    int x0, y0, za, zb;
    tile_of_block(fs, kTileX, g.nz, x0, y0, za, zb);
    pull_tile<S, W, false>(g, src, lds_raw, x0, y0, za, zb, [&](int s, const R (&t)[Q], const R (&d)[Q]) {
        const size_t N = (size_t)g.N;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            double fr, fb;
            from_shifted<double>(i, double(t[i]), double(d[i]), fr, fb);
            out[(size_t)i * N + s] = Out(fr);
            out[(size_t)(Q + i) * N + s] = Out(fb);
        }
    });
}

// Compensated totals: workgroup b sums tiles b, b + gridDim, ... in that order,
// each thread its column; the grid is fixed by the lattice, so the result is
// bitwise reproducible.
template <typename S, bool W>
__global__ __launch_bounds__(kTileX * pull_rows<S>()) void pull_totals_kernel(Geom g, S src, FusedShape fs,
                                                                             Neu* __restrict__ partial) {
    using R = typename S::R;
    extern __shared__ unsigned char lds_raw[];
    __shared__ Neu sums[pull_rows<S>() * NTOT];
    Neu acc[NTOT];
#pragma unroll
    for (int q = 0; q < NTOT; ++q) acc[q] = Neu{0.0, 0.0};
    const int tiles = fs.tiles_x * fs.tiles_y;
    for (int b = blockIdx.x; b < fs.nblocks; b += gridDim.x) {
        const int tile = b % tiles, za = (b / tiles) * fs.TZ;
        pull_tile<S, W, false>(g, src, lds_raw, (tile % fs.tiles_x) * kTileX, (tile / fs.tiles_x) * fs.TY, za,
                               min(za + fs.TZ, g.nz),
                               [&](int, const R (&t)[Q], const R (&d)[Q]) { add_site_totals<R>(t, d, acc); });
        __syncthreads();  // the next tile restages the ring
    }
    block_reduce(acc, sums);
    if (threadIdx.x == 0)
        for (int q = 0; q < NTOT; ++q) partial[blockIdx.x * NTOT + q] = acc[q];
}

}  // namespace lbm
