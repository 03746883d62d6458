// lb_lean.hpp -- the tile of the one-read step.
//
// A workgroup owns 64 x TY columns of a z-chunk and marches it plane by plane,
// one tile row per wavefront (64-wide wavefronts, so the row's y and the plane's
// z are wave-uniform and every row offset is scalar).  Per plane a wavefront
//   - stores the phase field of plane z + H and the colour records of plane
//     z + 1, loaded a plane ahead, into their LDS rings;
//   - pulls its sites: the totals t_i come from memory (loaded a plane ahead),
//     the colour differences are decoded from the source sites' records in LDS
//     (packed and 16-bit storage; the first step of a state reads pair arrays);
//   - takes the colour gradient and the near-contact probe from the ring,
//     collides and stores;
//   - gathers the phase sums of the next state: each row adds what it sends to
//     the rows above, beside and below it (neighbouring columns by DPP shifts
//     that read zero beyond the wavefront's end), and hands the six sums for
//     other rows over through LDS.
// A site whose sources all lie in the tile gets its phase field here; face sites
// keep their own sums for the assembly.
//
// What bounds it: at 256^3 FP32 moves 3.34 GB (92 B per site each way, the phase
// field, halos of records), 0.59 ms at the rate its access pattern reaches
// without arithmetic (lb_pattern_ms), and issues 0.40 ms of vector instructions
// per SIMD: 16 rows, four wavefronts per SIMD, take 0.70 ms, 4.8 TB/s (0.77 with
// 8 rows of 64 x 128 planes).  Left out in turn, probe, decode, phase sums and
// collision give 4 % each: memory bounds it.  16-bit storage moves 2.78 GB, 0.53
// ms, and issues 0.46: with droplets over a twentieth of the volume 12 rows, three
// wavefronts, take 0.71 ms, 8 rows 0.79, and a probe less is 10 % less; with 30 %,
// the emulsion of bench.py, whose probes are the more, 12 rows take 0.80 ms.
// Everything a plane needs from memory is loaded while the plane before it is
// collided.
#pragma once
#include "lb_pack.hpp"
#include "lb_single.hpp"

namespace lbm {

__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Values per buffer resource of the raw forms: the 19 arrays t_i as two
// resources of 9 and 10, the 19 pair arrays as five of up to four (a direction and its
// opposite in one), so that a load or store is one buffer access
// with a scalar row offset and a per-lane column offset and needs no 64-bit
// address arithmetic.  Needs 10 raw_stride(N) sizeof(T) < 2^32 for the totals and
// 8 raw_stride(N) sizeof(T) < 2^32 for the pairs (checked on the host): the pairs of
// every lattice whose 16-bit form fits its offsets (113 million sites) fit theirs.
constexpr int kResArrays = 10;
constexpr int kResPairs = 4;
constexpr unsigned kRsrcWord3 = 0x00020000;  // raw 32-bit buffer on gfx9-family targets
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// (t, d) pair loads
__device__ __forceinline__ void res_load_pair(float& t, float& d, __amdgpu_buffer_rsrc_t r, unsigned voff,
                                              unsigned soff) {
    const auto v = __builtin_bit_cast(RawPair<float>::type, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    t = v.x;
    d = v.y;
}
__device__ __forceinline__ void res_load_pair(double& t, double& d, __amdgpu_buffer_rsrc_t r, unsigned voff,
                                              unsigned soff) {
    const auto v = __builtin_bit_cast(RawPair<double>::type, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
    t = v.x;
    d = v.y;
}
__device__ __forceinline__ float res_load(float, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ double res_load(double, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
// non-temporal store (aux = 2: nt)
__device__ __forceinline__ void res_store(float v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 2);
}
__device__ __forceinline__ void res_store(double v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, voff, soff, 2);
}

// Resource of an array, its range all 32-bit offsets (every access is in range
// by its clamped coordinates or masked).  The pointer is made opaque first: the
// resource is then rebuilt where it is used, from two scalar registers and two
// constants, instead of holding four registers across the loop, whose resources
// together would spill.
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t array_res(const T* p) {
    asm volatile("" : "+s"(p));
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, -1, (int)kRsrcWord3);
}
// phase-sum pair (own sums of a face site), 8 or 16 bytes
__device__ __forceinline__ void res_store(const Part2<float>& v, __amdgpu_buffer_rsrc_t r, unsigned voff,
                                          unsigned soff) {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, voff, soff, 0);
}
// (16-byte stores take the whole offset per lane and none in a scalar register:
// the compiler keeps the instruction after such a store from overwriting its
// data only in that form, and with a scalar offset a record's first value was
// seen replaced by the next instruction's result in the last quarter of every
// 16 lanes)
__device__ __forceinline__ void res_store(const Part2<double>& v, __amdgpu_buffer_rsrc_t r, unsigned voff,
                                          unsigned soff) {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(V, v), r, voff + soff, 0, 0);
}
__device__ __forceinline__ void res_store_cached(float v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 0);
}
__device__ __forceinline__ void res_store_cached(double v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, voff, soff, 0);
}

// Value of lane l-1 of the wavefront (0 in lane 0) and of lane l+1 (0 in
// lane 63): DPP wave_shr:1 / wave_shl:1 with out-of-range lanes reading zero.
__device__ __forceinline__ float from_left(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ double from_left(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x138, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double from_right(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x130, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// FP32 rows of whole 128-byte lines are stored past the caches; others through
// them, so that a line two rows or two tiles share is completed before it goes to
// memory (201x77x59: a step 98 us against 104; aligned rows lose 4 % through them.
// In FP64 and 16 bits the second form costs small lattices 4 to 6 %).
__device__ __forceinline__ bool whole_lines(const Geom& g) { return ((unsigned)g.nx & 31u) == 0; }

// 16-byte pieces of a record
typedef double d2 __attribute__((ext_vector_type(2)));
template <typename T>
struct Chunk;
template <>
struct Chunk<float> {
    typedef f4 type;
};
template <>
struct Chunk<double> {
    typedef d2 type;
};
template <typename C>
__device__ __forceinline__ C res_load_chunk(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(C, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
template <typename C>
__device__ __forceinline__ void res_store_chunk(C v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, voff + soff, 0, 2);
}

// Rows a site's pulls read: r[1 + dz][1 + dy] = first site of the row
// (y + dy, z + dz) with the periodic wrap, and the walls its row lies next to.
// All of it is scalar.
struct LeanRows {
    unsigned r[3][3];
    bool ylo, yhi, zlo, zhi;
    __device__ __forceinline__ unsigned own() const { return r[1][1]; }
    // the source of direction i lies beyond a y or z wall
    __device__ __forceinline__ bool beyond(int i) const {
        using L = Lattice;
        return (L::cy[i] > 0 && ylo) || (L::cy[i] < 0 && yhi) || (L::cz[i] > 0 && zlo) || (L::cz[i] < 0 && zhi);
    }
    __device__ __forceinline__ unsigned from(int i) const { return r[1 - Lattice::cz[i]][1 - Lattice::cy[i]]; }
};
// Per-lane context: columns x, x - 1, x + 1 (periodic wrap; beyond an x wall x
// itself) and the x walls next to the lane's site.
struct LeanLane {
    unsigned c0, cm, cp;
    bool wx, xlo, xhi;
    int lane, ty, x;
    __device__ __forceinline__ unsigned col(int i) const {
        return Lattice::cx[i] > 0 ? cm : (Lattice::cx[i] < 0 ? cp : c0);
    }
    __device__ __forceinline__ bool beyond(int i) const {
        return (Lattice::cx[i] > 0 && xlo) || (Lattice::cx[i] < 0 && xhi);
    }
};
// Clamped coordinates (xc, yc): lanes and rows beyond the lattice compute on a
// valid site and store nothing.
__device__ __forceinline__ LeanLane lean_lane(const Geom& g, bool walls, int xc, int lane, int ty) {
    LeanLane o;
    o.wx = walls && g.wx;
    o.c0 = (unsigned)xc;
    o.cm = (unsigned)(xc == 0 ? (o.wx ? 0 : g.nx - 1) : xc - 1);
    o.cp = (unsigned)(xc == g.nx - 1 ? (o.wx ? xc : 0) : xc + 1);
    o.xlo = o.wx && xc == 0;
    o.xhi = o.wx && xc == g.nx - 1;
    o.lane = lane;
    o.ty = ty;
    o.x = xc;
    return o;
}
// The rows around row yc of any plane, from loop-invariant parts.
template <bool W>
struct LeanRowSet {
    unsigned yr[3], nxy;
    bool ylo, yhi, wz;
    int nz;
    __device__ __forceinline__ LeanRowSet(const Geom& g, int yc)
        : yr{(unsigned)(yc == 0 ? g.ny - 1 : yc - 1) * (unsigned)g.nx, (unsigned)(yc * g.nx),
             (unsigned)(yc == g.ny - 1 ? 0 : yc + 1) * (unsigned)g.nx},
          nxy((unsigned)g.nxy), ylo(W && g.wy && yc == 0), yhi(W && g.wy && yc == g.ny - 1), wz(W && g.wz), nz(g.nz) {}
    __device__ __forceinline__ LeanRows at(int z) const {  // z in [0, nz)
        LeanRows o;
        const unsigned zr[3] = {(unsigned)(z == 0 ? nz - 1 : z - 1) * nxy, (unsigned)z * nxy,
                                (unsigned)(z == nz - 1 ? 0 : z + 1) * nxy};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) o.r[a][b] = zr[a] + yr[b];
        o.ylo = ylo;
        o.yhi = yhi;
        o.zlo = wz && z == 0;
        o.zhi = wz && z == nz - 1;
        return o;
    }
};
// Offsets of direction i's source value: site = row (scalar) + column (lane),
// in array a.  Off a y or z wall the wavefront reads the opposite direction of
// its own row; off an x wall the lanes next to it do.  Lattices with walls (W) take
// the lane offsets of c_x != 0 whether x is walled or not: behind a branch, the loads
// of either side were waited for one by one (256x256x128 FP32 between walls on every
// axis, 8 rows: 773 us a step against 489).  BRANCH keeps the branch, for tiles whose
// registers spill either way (FP64 between moving walls with a near-contact halo:
// 1140 us without it, 1038 with it).
//   load(a, row, col): the value at that row and column of array a
//   load_at(site_and_array offset per lane)
template <bool W, bool BRANCH, typename Load, typename LoadLane>
__device__ __forceinline__ void source_of(int i, const LeanRows& rw, const LeanLane& ln, const Load& load,
                                          const LoadLane& load_lane) {
    using L = Lattice;
    if constexpr (W) {
        const bool bb = rw.beyond(i);
        const int a = bb ? L::opp[i] : i;
        const unsigned row = bb ? rw.own() : rw.from(i);
        const unsigned col = bb ? ln.c0 : ln.col(i);
        if (L::cx[i] != 0 && (!BRANCH || ln.wx)) load_lane(a, row, col, L::opp[i], rw.own(), ln.c0, ln.beyond(i));
        else load(a, row, col);
    } else {
        load(i, rw.from(i), ln.col(i));
    }
}

// halo_coord along z for a plane at most a few halos beyond the lattice, without
// a division (the scalar unit has none).
__device__ __forceinline__ int halo_plane(int z, int n, int wall) {
    if (wall) {
        const int m = z < 0 ? -1 - z : (z >= n ? 2 * n - 1 - z : z);
        return m < 0 ? 0 : (m >= n ? n - 1 : m);
    }
    while (z < 0) z += n;
    while (z >= n) z -= n;
    return z;
}

// The decode reads a source record from LDS per direction; left free, the
// compiler has all 19 in flight (76 or 152 registers) and fewer wavefronts fit a
// SIMD.  After the tenth direction the running sums pass through an empty
// statement that the later reads stay behind: 16 rows of FP32 then fit the 128
// registers of four wavefronts per SIMD without spilling (256^3, tile: 701 us
// against 894), 12 rows of 16-bit storage the 168 of three (384^3 bf16: 2.10 ms;
// 2.19 with a stop every fourth direction, 7.8 without).  The wall tests take more
// registers: there the statement stands after every sixth.
template <bool W, typename R>
__device__ __forceinline__ void settle(SiteSums<R>& m, int i) {
    if (W ? i % 6 == 5 : i == 9)
        asm volatile("" : "+v"(m.drho), "+v"(m.dif), "+v"(m.rc), "+v"(m.jx), "+v"(m.jy), "+v"(m.jz)::"memory");
}

// LDS ring of the source records of planes z - 1, z, z + 1 (tile plus one site
// around it): per plane NC runs of 16-byte pieces, so consecutive lanes read
// consecutive pieces, free of bank conflicts.
constexpr int kRecRow = kTileX + 2;
template <typename C, int NC, int TY>
struct RecPlanes {
    C* base;
    static constexpr int half = (TY + 2) * kRecRow;
    static constexpr int plane = NC * half;
    static constexpr size_t plane_bytes = (size_t)plane * sizeof(C);
    // piece k of ring entry e of slot s
    __device__ __forceinline__ C& at(int s, int k, int e) const { return base[s * plane + k * half + e]; }
};

// Staging of the record ring: every thread loads its own site's record of a
// plane and, the first RE of them, one of the halo around the tile.
template <typename S, int TY>
struct RecStage {
    using C = typename S::C;
    static constexpr int NC = S::NC, NCA = NC > 0 ? NC : 1;
    static constexpr int RE = 2 * kRecRow + 2 * TY;
    static_assert(RE <= kTileX * TY, "a tile's record halo exceeds its threads");
    using Planes = RecPlanes<C, NCA, TY>;
    unsigned main_at, halo_at;  // sites within a plane
    int main_lds, halo_lds;
    bool halo_on;
    struct Regs {
        C m[NCA], h[NCA];
    };
    __device__ __forceinline__ RecStage(const Geom& g, int x0, int y0, int lane, int ty, unsigned own_at)
        : main_at(own_at), halo_at(0), main_lds((ty + 1) * kRecRow + lane + 1), halo_lds(0),
          halo_on(NC > 0 && (int)threadIdx.x < RE) {
        if (NC == 0) return;
        const int e = min((int)threadIdx.x, RE - 1);
        int r, q;
        if (e < 2 * kRecRow) {
            r = e < kRecRow ? 0 : TY + 1;
            q = e < kRecRow ? e : e - kRecRow;
        } else {
            const int e2 = e - 2 * kRecRow;
            r = 1 + (e2 >> 1);
            q = (e2 & 1) ? kTileX + 1 : 0;
        }
        halo_at = (unsigned)(halo_coord(y0 - 1 + r, g.ny, g.wy) * g.nx + halo_coord(x0 - 1 + q, g.nx, g.wx));
        halo_lds = r * kRecRow + q;
    }
    __device__ __forceinline__ void load(const Geom& g, const S& src, int plane, Regs& s) const {
        if constexpr (NC > 0) {
            constexpr unsigned RB = 16u * NC;
            const __amdgpu_buffer_rsrc_t rr = src.rec_res();
            const unsigned so = (unsigned)halo_plane(plane, g.nz, g.wz) * (unsigned)g.nxy * RB;
#pragma unroll
            for (int k = 0; k < NC; ++k) s.m[k] = res_load_chunk<C>(rr, main_at * RB + 16u * k, so);
            if (halo_on) {
#pragma unroll
                for (int k = 0; k < NC; ++k) s.h[k] = res_load_chunk<C>(rr, halo_at * RB + 16u * k, so);
            }
        }
    }
    __device__ __forceinline__ void put(const Planes& rp, int slot, const Regs& s) const {
        if constexpr (NC > 0) {
#pragma unroll
            for (int k = 0; k < NC; ++k) rp.at(slot, k, main_lds) = s.m[k];
            if (halo_on) {
#pragma unroll
                for (int k = 0; k < NC; ++k) rp.at(slot, k, halo_lds) = s.h[k];
            }
        }
    }
};

// ------------------------------------------------------------- pair arrays
// Source of a state's first step: pairs (t_i, d_i), read where they are needed.
template <typename T>
struct LeanPairs {
    using R = T;
    using C = typename Chunk<T>::type;
    static constexpr int NC = 0;
    const T* f;
    struct Pre {};
    // five resources of up to four arrays: 0-2, 3-6, ... 15-18
    struct Res {
        __amdgpu_buffer_rsrc_t r[5];
    };
    static __device__ __forceinline__ constexpr int part(int i) { return (i + 1) / kResPairs; }
    static __device__ __forceinline__ constexpr int first(int k) { return k == 0 ? 0 : kResPairs * k - 1; }
    // offset of a site in array i of its resource
    static __device__ __forceinline__ unsigned off(int i, unsigned S, unsigned site) {
        return ((unsigned)(i - first(part(i))) * S + site) * 2u * (unsigned)sizeof(T);
    }
    __device__ __forceinline__ Res res(unsigned N) const {
        const unsigned S = N + kRawPad;
        Res o;
#pragma unroll
        for (int k = 0; k < 5; ++k) o.r[k] = array_res(f + (size_t)first(k) * 2 * S);
        return o;
    }
    template <bool W, bool BR>
    __device__ __forceinline__ void fetch(const Geom&, const LeanRows&, const LeanLane&, Pre&) const {}

    // The own post-collision phase from the pairs of the site itself.
    template <int TY>
    __device__ __forceinline__ T own_phase(const Geom& g, unsigned own, const LeanLane& ln,
                                           const RecPlanes<C, 1, TY>&, int) const {
        const Res rs = res((unsigned)g.N);
        constexpr unsigned SZ = 2 * (unsigned)sizeof(T);
        const unsigned S = (unsigned)g.N + kRawPad;
        T st = T(0), sd = T(0);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            T tj, dj;
            res_load_pair(tj, dj, rs.r[part(j)], ln.c0 * SZ, off(j, S, own));
            st += weight<T>(j) + tj;
            sd += dj;
        }
        return sd / st;
    }
    template <bool W, int TY, typename Visit>
    __device__ __forceinline__ void values(const Geom& g, const LeanRows& rw, const LeanLane& ln,
                                           const RecPlanes<C, 1, TY>&, int, int, int, const Pre&,
                                           const Visit& visit) const {
        T t[Q], d[Q];
        const Res rs = res((unsigned)g.N);
        constexpr unsigned SZ = 2 * (unsigned)sizeof(T);
        const unsigned S = (unsigned)g.N + kRawPad;
#pragma unroll
        for (int i = 0; i < Q; ++i)
            source_of<W, false>(
                i, rw, ln,
                [&](int a, unsigned row, unsigned col) {
                    res_load_pair(t[i], d[i], rs.r[part(i)], col * SZ, off(a, S, row));
                },
                [&](int a, unsigned row, unsigned col, int o, unsigned own, unsigned c0, bool refl) {
                    res_load_pair(t[i], d[i], rs.r[part(i)],
                                  refl ? off(o, S, own) + c0 * SZ : off(a, S, row) + col * SZ, 0);
                });
#pragma unroll
        for (int i = 0; i < Q; ++i) visit(i, t[i], d[i]);
    }
};

// ------------------------------------------------------------------ packed
template <typename T>
struct LeanPack {
    using R = T;
    using C = typename Chunk<T>::type;
    static constexpr int NC = (int)(sizeof(T) / 4);  // pieces of a record
    static constexpr bool kSplit = false;
    T* rec;
    T* tot;
    struct Pre {
        T v[Q];
    };
    static constexpr int kFirst = 9;  // arrays of the first resource
    static __device__ __forceinline__ int part(int i) { return i < kFirst ? 0 : 1; }
    static __device__ __forceinline__ unsigned off(int i, unsigned S, unsigned site) {
        return ((unsigned)(i < kFirst ? i : i - kFirst) * S + site) * (unsigned)sizeof(T);
    }
    struct Res {
        __amdgpu_buffer_rsrc_t t[2];
    };
    __device__ __forceinline__ Res res(unsigned N) const {
        return Res{{array_res(tot), array_res(tot + (size_t)kFirst * (N + kRawPad))}};
    }
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rec_res() const { return array_res(rec); }
    template <bool W, bool BR>
    __device__ __forceinline__ void fetch(const Geom& g, const LeanRows& rw, const LeanLane& ln, Pre& p) const {
        const Res rs = res((unsigned)g.N);
        const unsigned S = (unsigned)g.N + kRawPad;
        unsigned step = S * (unsigned)sizeof(T), at = 0;  // array offset, accumulated (re-read each plane:
        asm volatile("" : "+s"(step));                    // 19 loop-invariant offsets would spill)
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            if (i == kFirst) at = 0;
            source_of<W, BR>(
                i, rw, ln,
                [&](int a, unsigned row, unsigned col) {
                    if constexpr (W)
                        p.v[i] = res_load(T(0), rs.t[part(i)], col * (unsigned)sizeof(T), off(a, S, row));
                    else
                        p.v[i] = res_load(T(0), rs.t[part(i)], col * (unsigned)sizeof(T),
                                          at + row * (unsigned)sizeof(T));
                },
                [&](int a, unsigned row, unsigned col, int o, unsigned own, unsigned c0, bool refl) {
                    const unsigned v = refl ? off(o, S, own) + c0 * (unsigned)sizeof(T)
                                            : off(a, S, row) + col * (unsigned)sizeof(T);
                    p.v[i] = res_load(T(0), rs.t[part(i)], v, 0);
                });
            at += step;
        }
    }
    template <int TY>
    static __device__ __forceinline__ Colour<T> colour(const RecPlanes<C, NC, TY>& rp, int s, int e) {
        if constexpr (NC == 1) {
            const C a = rp.at(s, 0, e);
            return Colour<T>{a.x, a.y, a.z, a.w};
        } else {
            const C a = rp.at(s, 0, e), b = rp.at(s, 1, e);
            return Colour<T>{a.x, a.y, b.x, b.y};
        }
    }
    // The own post-collision phase, summed as RawPop sums its pairs; s0: slot of
    // the site's plane.
    template <int TY>
    __device__ __forceinline__ T own_phase(const Geom& g, unsigned own, const LeanLane& ln,
                                           const RecPlanes<C, NC, TY>& rp, int s0) const {
        const Res rs = res((unsigned)g.N);
        const Colour<T> q = colour<TY>(rp, s0, (ln.ty + 1) * kRecRow + ln.lane + 1);
        const unsigned S = (unsigned)g.N + kRawPad;
        T st = T(0), sd = T(0);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const T v = res_load(T(0), rs.t[part(j)], ln.c0 * (unsigned)sizeof(T), off(j, S, own));
            st += weight<T>(j) + v;
            sd += recoloured<T>(j, weight<T>(j) + v, q);
        }
        return sd / st;
    }
    // Colour difference of a value arriving in direction i, read from the
    // opposite direction where refl.
    static __device__ __forceinline__ T diff(int i, T wt, const Colour<T>& q, bool refl) {
#pragma clang fp contract(off)
        if (i == 0) return q.phi * wt;
        const T cs = cdot3<T>(i, q.sx, q.sy, q.sz);
        constexpr T k = weight<T>(1) / (weight<T>(7) * inv_clen<T>(7));
        const T v = Lattice::len2(i) == 1 ? k * cs : cs;
        return fma_of(q.phi, wt, refl ? -v : v);
    }
    // visit(i, t_i, d_i) of the lane's site in ascending direction; sm, s0, sp:
    // slots of planes z - 1, z, z + 1
    template <bool W, int TY, typename Visit>
    __device__ __forceinline__ void values(const Geom&, const LeanRows& rw, const LeanLane& ln,
                                           const RecPlanes<C, NC, TY>& rp, int sm, int s0, int sp, const Pre& p,
                                           const Visit& visit) const {
        using L = Lattice;
        const int own = (ln.ty + 1) * kRecRow + ln.lane + 1;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            int s = L::cz[i] > 0 ? sm : (L::cz[i] < 0 ? sp : s0), e = own - L::cy[i] * kRecRow - L::cx[i];
            bool refl = false;
            if constexpr (W) {
                refl = rw.beyond(i) || (L::cx[i] != 0 && ln.beyond(i));
                s = refl ? s0 : s;
                e = refl ? own : e;
            }
            visit(i, p.v[i], diff(i, weight<T>(i) + p.v[i], colour<TY>(rp, s, e), refl));
        }
    }
    // Destination: store the site and keep what a later pull reads of it.
    struct Kept {
        Colour<T> q;
        T phase;
    };
    __device__ __forceinline__ void store(const Geom& g, unsigned own, const LeanLane& ln, T (&t)[Q],
                                          const SiteTotals<T>& tot_, bool site_in, Kept& k) const {
        k.q = colour_of(tot_);
        if (site_in) {
            const Res rs = res((unsigned)g.N);
            const __amdgpu_buffer_rsrc_t rr = rec_res();
            const unsigned S = (unsigned)g.N + kRawPad;
            constexpr unsigned RB = 4 * (unsigned)sizeof(T);
            if constexpr (NC == 1) {
                res_store_chunk(C{k.q.phi, k.q.sx, k.q.sy, k.q.sz}, rr, ln.c0 * RB, own * RB);
            } else {
                res_store_chunk(C{k.q.phi, k.q.sx}, rr, ln.c0 * RB, own * RB);
                res_store_chunk(C{k.q.sy, k.q.sz}, rr, ln.c0 * RB + 16u, own * RB);
            }
            unsigned step = S * (unsigned)sizeof(T);
            asm volatile("" : "+s"(step));
            auto put = [&](auto store_one) {
                unsigned at = own * (unsigned)sizeof(T);
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    if (i == kFirst) at = own * (unsigned)sizeof(T);
                    store_one(t[i], rs.t[part(i)], ln.c0 * (unsigned)sizeof(T), at);
                    at += step;
                }
            };
            auto past = [](T v, __amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) { res_store(v, r, vo, so); };
            auto through = [](T v, __amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) { res_store_cached(v, r, vo, so); };
            if constexpr (NC == 1) {
                if (whole_lines(g)) put(past);
                else put(through);
            } else {
                put(past);
            }
        }
    }
    __device__ __forceinline__ T kept_diff(int i, T wt, const Kept& k) const { return recoloured<T>(i, wt, k.q); }
    static __device__ __forceinline__ void clear(Kept& k) { k.q = Colour<T>{T(0), T(0), T(0), T(0)}; }
    // phase a moving wall's term is shared by: from the stored values
    __device__ __forceinline__ T kept_phase(const T (&t)[Q], const Kept& k) const {
        T st = T(0), sd = T(0);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            st += weight<T>(j) + t[j];
            sd += recoloured<T>(j, weight<T>(j) + t[j], k.q);
        }
        return sd / st;
    }
};

// ------------------------------------------------- 16-bit moment-split form
// (the codec of SplitPop): per site an FP32 record of 8 values, per direction a
// 16-bit deviation.
template <typename H>
struct LeanSplit {
    using R = float;
    using C = f4;
    static constexpr int NC = 2;
    static constexpr bool kSplit = true;
    float* rec;
    H* dev;
    SplitPop<H> codec;  // scale and the record arithmetic
    struct Pre {
        unsigned dv[Q];  // one per register (two per register would make every load wait
                         // at once for the packing)
    };
    static __device__ __forceinline__ H dev_of(unsigned v) { return __builtin_bit_cast(H, (unsigned short)v); }
    static __device__ __forceinline__ unsigned off(int i, unsigned S, unsigned site) {
        return ((unsigned)i * S + site) * 2u;
    }
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rec_res() const { return array_res(rec); }
    template <bool W, bool BR>
    __device__ __forceinline__ void fetch(const Geom& g, const LeanRows& rw, const LeanLane& ln, Pre& p) const {
        const __amdgpu_buffer_rsrc_t rd = array_res(dev);
        const unsigned S = (unsigned)g.N + kDevPad;
        unsigned step = 2u * S, at = 0;
        asm volatile("" : "+s"(step));
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            source_of<W, BR>(
                i, rw, ln,
                [&](int a, unsigned row, unsigned col) {
                    p.dv[i] = __builtin_amdgcn_raw_buffer_load_b16(rd, col * 2u, W ? off(a, S, row) : at + 2u * row, 0);
                },
                [&](int a, unsigned row, unsigned col, int o, unsigned own, unsigned c0, bool refl) {
                    const unsigned v = refl ? off(o, S, own) + c0 * 2u : off(a, S, row) + col * 2u;
                    p.dv[i] = __builtin_amdgcn_raw_buffer_load_b16(rd, v, 0, 0);
                });
            at += step;
        }
    }
    template <bool W, int TY, typename Visit>
    __device__ __forceinline__ void values(const Geom&, const LeanRows& rw, const LeanLane& ln,
                                           const RecPlanes<C, NC, TY>& rp, int sm, int s0, int sp, const Pre& p,
                                           const Visit& visit) const {
        using L = Lattice;
        const int own = (ln.ty + 1) * kRecRow + ln.lane + 1;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            int s = L::cz[i] > 0 ? sm : (L::cz[i] < 0 ? sp : s0), e = own - L::cy[i] * kRecRow - L::cx[i];
            float sg = 1.0f;
            if constexpr (W) {
                const bool refl = rw.beyond(i) || (L::cx[i] != 0 && ln.beyond(i));
                s = refl ? s0 : s;
                e = refl ? own : e;
                sg = refl ? -1.0f : 1.0f;
            }
            const f4 ra = rp.at(s, 0, e), rb = rp.at(s, 1, e);
            float t, d;
            codec.finish(i, sg, SplitPop<H>::excess(i, sg, ra), rb, dev_of(p.dv[i]), t, d);
            visit(i, t, d);
        }
    }
    // The phase of the site's own record.
    template <int TY>
    __device__ __forceinline__ float own_phase(const Geom&, unsigned, const LeanLane& ln,
                                               const RecPlanes<C, NC, TY>& rp, int s0) const {
        return rp.at(s0, 1, (ln.ty + 1) * kRecRow + ln.lane + 1).x;
    }
    // Destination: encode and store the record and the deviations, and keep in
    // t the totals a later pull decodes (exactly: the same codec arithmetic).
    struct Kept {
        f4 rb;
    };
    __device__ __forceinline__ void store(const Geom& g, unsigned own, const LeanLane& ln, float (&t)[Q],
                                          const SiteTotals<float>& tot, bool site_in, Kept& k) const {
#pragma clang fp contract(off)
        const f4 ra = {tot.drho, tot.jx, tot.jy, tot.jz};
        k.rb = f4{tot.phi, tot.vx, tot.vy, tot.vz};
        H h[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const float wX = weight<float>(i) * SplitPop<H>::excess(i, 1.0f, ra);
            h[i] = Half<H>::from_f((t[i] - wX) * codec.scale);
            t[i] = fma_of(Half<H>::to_f(h[i]), codec.inv_scale, wX);
        }
        if (site_in) {
            const unsigned S = (unsigned)g.N + kDevPad;
            const __amdgpu_buffer_rsrc_t rr = rec_res(), rd = array_res(dev);
            res_store_chunk(ra, rr, ln.c0 * 32u, own * 32u);
            res_store_chunk(k.rb, rr, ln.c0 * 32u + 16u, own * 32u);
            unsigned step = 2u * S, at = 2u * own;
            asm volatile("" : "+s"(step));
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, h[i]), rd, ln.c0 * 2u, at, 2);
                at += step;
            }
        }
    }
    __device__ __forceinline__ float kept_diff(int i, float wt, const Kept& k) const {
        return SplitPop<H>::colour_diff(i, 1.0f, wt, k.rb);
    }
    static __device__ __forceinline__ void clear(Kept& k) { k.rb = f4{0.0f, 0.0f, 0.0f, 0.0f}; }
    __device__ __forceinline__ float kept_phase(const float (&)[Q], const Kept& k) const { return k.rb.x; }
};

// Off a moving wall each reflected direction of the pulled site gains the wall
// term, shared between the components by the site's own phase.
template <typename R>
struct MovingTerms {
    bool on = false;
    R ph = R(0);
    // s0: record slot of the site's plane
    template <typename S, int TY, typename Planes>
    __device__ __forceinline__ void init(const Geom& g, const S& src, const LeanRows& rw, const LeanLane& ln,
                                         const Planes& rp, int s0) {
        const bool wyz = rw.ylo || rw.yhi || rw.zlo || rw.zhi;
        on = g.moving && (wyz || ln.xlo || ln.xhi);
        if (on) ph = src.template own_phase<TY>(g, rw.own(), ln, rp, s0);
    }
    __device__ __forceinline__ void add(const Geom& g, int i, const LeanRows& rw, const LeanLane& ln, int yc, int cz,
                                        R& t, R& d) const {
#pragma clang fp contract(off)
        if (i == 0 || !on || !(rw.beyond(i) || ln.beyond(i))) return;
        const R a = wall_term<R>(g, i, ln.x, yc, cz);
        t += a;
        d = fma_of(a, ph, d);
    }
};

// ------------------------------------------------------------ phase sums
// What a row sends to the rows above and below it, summed over the columns it
// comes from: slot (e, f) for direction velocities c_y = e, c_z = f.  Between
// rows r and r + 1 lie the sums r sends up (e = 1) and those r + 1 sends down;
// what the first and last row send out of the tile is another box's.
__host__ __device__ constexpr int xch_slot(int e, int f) { return (e > 0 ? 0 : 3) + (f == 0 ? 0 : (f > 0 ? 1 : 2)); }
constexpr int kXchSlots = 6;
constexpr int kXchRow = kTileX + 2;  // a row's 64 columns and one beyond each end (x-face terms)

// LDS of a tile with source S: phase ring, record ring, exchange rows (D and R
// sums at once, or one after the other where both do not fit), x-face sums.
template <typename S, int TY, int H>
struct LeanLds {
    using R = typename S::R;
    static constexpr size_t phi = (phi_ring_bytes<R, kTileX, H>(TY) + 15) & ~size_t(15);
    static constexpr size_t rec = 3 * RecPlanes<typename S::C, S::NC, TY>::plane_bytes;
    static constexpr size_t half = (size_t)(TY - 1) * kXchSlots * kXchRow * sizeof(R);
    static constexpr size_t vs = (size_t)2 * 3 * TY * sizeof(Part2<R>);
    static constexpr int rounds = phi + rec + 2 * half + vs <= kLdsBytes ? 1 : 2;
    static constexpr size_t xch = rounds == 1 ? 2 * half : half;
    static constexpr size_t bytes = phi + rec + xch + vs;
};

// x-face sums the edge lanes of a tile column accumulate for the face sites of
// the neighbouring columns: the lo edge lane (c_x = -1) feeds the hi face of the
// column on its left, the hi edge lane (c_x = +1) the lo face of the one on its
// right (periodic wrap; none beyond an x wall).  Both lanes run the same code,
// each on its side's directions; where one lane is both (a column one site wide)
// it runs twice.  The running sums of the destination planes z-1, z, z+1 of a row
// live in LDS, vs[side][plane mod 3][row].
template <typename R, int TY>
struct XEdge {
    int passes;
    bool lo_on, hi_on, hi;    // this lane feeds a column, and from which side
    unsigned lo_at, hi_at;    // entries of its destinations in plane 0
    int width;
    __device__ __forceinline__ XEdge(const Geom& g, int x0, int x1, int y, bool row_in, int lane)
        : passes(x1 - x0 == 1 ? 2 : 1), width(x1 - x0) {
        int bd_lo = 0, bd_hi = 0;
        const bool has_lo = xface_dest<kTileX>(g, x0, x1, -1, bd_lo), has_hi = xface_dest<kTileX>(g, x0, x1, 1, bd_hi);
        lo_on = row_in && lane == 0 && has_lo;
        hi_on = row_in && lane == x1 - x0 - 1 && has_hi;
        hi = lane != 0;
        lo_at = xface_at(g, bd_lo, 1, y, 0);
        hi_at = xface_at(g, bd_hi, 0, y, 0);
    }
    __device__ __forceinline__ bool is_hi(int pass) const { return passes == 1 ? hi : pass != 0; }
    __device__ __forceinline__ bool active(bool h) const {
        const bool l = lo_on, r = hi_on;
        return (h && r) || (!h && l);
    }
    __device__ __forceinline__ unsigned dest(bool h) const {  // byte offset in plane 0
        const unsigned l = lo_at, r = hi_at;
        return (h ? r : l) * (unsigned)sizeof(Part2<R>);
    }

    // Before the exchange: the lane's own terms of plane cz close the sum of
    // destination plane cz - 1 (stored), add the first in-plane term of plane cz
    // and open the sum of plane cz + 1; the terms its row sends across the face
    // into the rows above and below go to the pads of its exchange rows.
    // val(i): w_i + t_i and d_i of direction i; pad(e, column, terms): stores one.
    template <typename V, typename Pad>
    __device__ __forceinline__ void own(const Geom& g, const V& val, const Pad& pad, Part2<R>* __restrict__ vs, int ty,
                                        int cz, int k0, int za, int zb, __amdgpu_buffer_rsrc_t xf) const {
        const int km = k0 == 0 ? 2 : k0 - 1, kp = k0 == 2 ? 0 : k0 + 1;
#pragma unroll 1
        for (int pass = 0; pass < passes; ++pass) {
            const bool h = is_hi(pass);
            if (!active(h)) continue;
            auto side = [&](int cy, int cz_) {
                const Part2<R> l = val(dir_of(-1, cy, cz_)), r = val(dir_of(1, cy, cz_));
                return Part2<R>{h ? r.dn : l.dn, h ? r.rc : l.rc};
            };
            Part2<R>* v = vs + (h ? 3 * TY : 0) + ty;
            auto plus = [](const Part2<R>& p, const Part2<R>& q) { return Part2<R>{p.dn + q.dn, p.rc + q.rc}; };
            if (cz - 1 >= za)
                res_store(plus(v[km * TY], side(0, -1)), xf, dest(h),
                          (unsigned)((cz - 1) * g.ny) * (unsigned)sizeof(Part2<R>));
            v[k0 * TY] = plus(cz == za ? Part2<R>{R(0), R(0)} : v[k0 * TY], side(0, 0));
            if (cz + 1 < zb) v[kp * TY] = side(0, 1);
            const int column = h ? 1 + width : 0;
            pad(1, column, side(1, 0));
            pad(-1, column, side(-1, 0));
        }
    }
    // The pads alone, for a second exchange round.
    template <typename V, typename Pad>
    __device__ __forceinline__ void pads(const V& val, const Pad& pad) const {
#pragma unroll 1
        for (int pass = 0; pass < passes; ++pass) {
            const bool h = is_hi(pass);
            if (!active(h)) continue;
#pragma unroll
            for (int e = 1; e >= -1; e -= 2) {
                const Part2<R> l = val(dir_of(-1, e, 0)), r = val(dir_of(1, e, 0));
                pad(e, h ? 1 + width : 0, Part2<R>{h ? r.dn : l.dn, h ? r.rc : l.rc});
            }
        }
    }
    // After the exchange: the in-plane terms the rows below and above send across
    // the face, in ascending direction (7 from below then 9 from above; 8 from
    // above then 10 from below); the chunk's last plane is then complete.
    // got(e, column): what the row y - e left at that pad, zero if it is not in
    // the tile.
    // round: of `rounds` exchange rounds, the R sums in the first, the D sums in
    // the last.
    template <typename Got>
    __device__ __forceinline__ void rows(const Geom& g, int round, int rounds, const Got& got, Part2<R>* __restrict__ vs,
                                         int ty, int cz, int k0, int zb, __amdgpu_buffer_rsrc_t xf) const {
        const bool do_rc = round == 0, do_dn = round == rounds - 1;
#pragma unroll 1
        for (int pass = 0; pass < passes; ++pass) {
            const bool h = is_hi(pass);
            if (!active(h)) continue;
            Part2<R>* v = vs + (h ? 3 * TY : 0) + ty;
            const int column = h ? 1 + width : 0;
            const Part2<R> below = got(1, column), above = got(-1, column);
            Part2<R> P = v[k0 * TY];
            if (do_rc) P.rc = (P.rc + (h ? below.rc : above.rc)) + (h ? above.rc : below.rc);
            if (do_dn) P.dn = (P.dn + (h ? below.dn : above.dn)) + (h ? above.dn : below.dn);
            if (do_dn && cz == zb - 1)
                res_store(P, xf, dest(h),
                          (unsigned)(cz * g.ny) * (unsigned)sizeof(P));
            else
                v[k0 * TY] = P;
        }
    }
};

// One tile of the one-read step: columns [x0, x0+64) x [y0, y0+TY), planes
// [za, zb); blockDim.x == 64 TY; source S, destination D (the same form, or
// pair arrays into either).  W: the lattice has walls (an all-periodic lattice
// carries none of their tests), MV: some may move.
template <typename S, typename D, int TY, int H, bool W, bool MV>
__device__ __forceinline__ void lean_tile(const Geom& g, const S& src, const D& dst, const Coeffs<typename S::R>& c,
                                          unsigned char* __restrict__ lds, int x0, int y0, int za, int zb,
                                          const typename S::R* __restrict__ phi_in,
                                          Part2<typename S::R>* __restrict__ part_out,
                                          typename S::R* __restrict__ phi_out, int moving_next) {
#pragma clang fp contract(off)
    using L = Lattice;
    using R = typename S::R;
    using C = typename S::C;
    using Lds = LeanLds<S, TY, H>;
    constexpr int TX = kTileX, NT = TX * TY;
    constexpr int LX = TX + 2 * H, LY = TY + 2 * H, NP = 2 * H + 1, PLANE = LY * LX;
    constexpr int NCA = S::NC > 0 ? S::NC : 1;
    constexpr bool BR = MV && H > 1 && sizeof(R) == 8;
    R* const ring = reinterpret_cast<R*>(lds);
    const RecPlanes<C, NCA, TY> rp{reinterpret_cast<C*>(lds + Lds::phi)};
    R* const xch = reinterpret_cast<R*>(lds + Lds::phi + Lds::rec);
    Part2<R>* const vs = reinterpret_cast<Part2<R>*>(lds + Lds::phi + Lds::rec + Lds::xch);

    const int lane = threadIdx.x & 63;
    const int ty = wave_uniform(threadIdx.x >> 6);
    const int x = x0 + lane, y = y0 + ty;
    const int x1 = min(x0 + TX, g.nx), y1 = min(y0 + TY, g.ny);
    const int nrows = y1 - y0;
    const bool xin = x < g.nx, row_in = y < g.ny, site_in = xin && row_in;
    const bool ragged = x1 - x0 < TX;
    const int xc = xin ? x : g.nx - 1, yc = row_in ? y : g.ny - 1;
    const LeanLane ln = lean_lane(g, W, xc, lane, ty);
    const unsigned nxy = (unsigned)g.nxy;
    const LeanRowSet<W> rows(g, yc);

    // ---- staging of the rings: every thread loads its own site's entry and its
    // share of the halo entries around the tile
    constexpr int PE = LY * LX - TX * TY, NE = (PE + NT - 1) / NT;  // phase halo
    const unsigned main_at = (unsigned)(halo_coord(y0 + ty, g.ny, g.wy) * g.nx + halo_coord(x, g.nx, g.wx));
    const int main_lds = (ty + H) * LX + lane + H;
    unsigned pe_at[NE];
    int pe_lds[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int e = min((int)threadIdx.x + k * NT, PE - 1);  // (surplus threads repeat the last entry)
        int r, q;
        if (e < 2 * H * LX) {
            r = e / LX;
            q = e - r * LX;
            r = r < H ? r : TY + r;
        } else {
            const int e2 = e - 2 * H * LX;
            r = H + e2 / (2 * H);
            q = e2 % (2 * H);
            q = q < H ? q : TX + q;
        }
        pe_at[k] = (unsigned)(halo_coord(y0 - H + r, g.ny, g.wy) * g.nx + halo_coord(x0 - H + q, g.nx, g.wx));
        pe_lds[k] = r * LX + q;
    }
    const RecStage<S, TY> recs(g, x0, y0, lane, ty, main_at);
    struct Stage {
        R m, e[NE];
        typename RecStage<S, TY>::Regs rec;
    };
    auto load_phi = [&](int q, Stage& s) {
        const unsigned so = (unsigned)halo_plane(q, g.nz, g.wz) * nxy * (unsigned)sizeof(R);
        const __amdgpu_buffer_rsrc_t rphi = array_res(phi_in);
        s.m = res_load(R(0), rphi, main_at * (unsigned)sizeof(R), so);
#pragma unroll
        for (int k = 0; k < NE; ++k) s.e[k] = res_load(R(0), rphi, pe_at[k] * (unsigned)sizeof(R), so);
    };
    auto put_phi = [&](int slot, const Stage& s) {
        R* p = ring + slot * PLANE;
        p[main_lds] = s.m;
#pragma unroll
        for (int k = 0; k < NE; ++k) p[pe_lds[k]] = s.e[k];
    };
    const XEdge<R, TY> xedge(g, x0, x1, y, row_in, lane);
    // a site on an x or y face of the box keeps its own sums for the assembly
    const bool face_xy = lane == 0 || lane == TX - 1 || x == g.nx - 1 || ty == 0 || ty == TY - 1 || y == g.ny - 1;

    // ---- prologue: the planes below the first one, all in flight together
    Stage st;
    typename S::Pre pre;
    {
        Stage s[2 * H];
#pragma unroll
        for (int k = 0; k < 2 * H; ++k) load_phi(za - H + k, s[k]);
        recs.load(g, src, za - 1, s[0].rec);
        recs.load(g, src, za, s[1].rec);
        load_phi(za + H, st);
        recs.load(g, src, za + 1, st.rec);
        const LeanRows rw = rows.at(za);
        src.template fetch<W, BR>(g, rw, ln, pre);
#pragma unroll
        for (int k = 0; k < 2 * H; ++k) put_phi(k, s[k]);
        recs.put(rp, 0, s[0].rec);
        recs.put(rp, 1, s[1].rec);
    }
    R prev_dn = R(0), prev_rc = R(0), cur_dn = R(0), cur_rc = R(0);
    int s0 = H;  // ring slot of plane cz
    int k0 = 0;  // (cz - za) mod 3: x-face sums; record slots of cz - 1, cz, cz + 1 are k0, k0 + 1, k0 + 2

    for (int cz = za; cz < zb; ++cz) {
        const int r1 = k0 == 2 ? 0 : k0 + 1, r2 = k0 == 0 ? 2 : k0 - 1;
        {
            int sh = s0 + H;
            sh = sh >= NP ? sh - NP : sh;
            put_phi(sh, st);
            recs.put(rp, r2, st.rec);
        }
        __syncthreads();
        // ---- colour gradient and near contact from the ring (before the pull: the
        // probe's addresses then do not add to the pulled values in registers)
        const int sm = s0 == 0 ? NP - 1 : s0 - 1, sp = s0 == NP - 1 ? 0 : s0 + 1;
        R gx, gy, gz;
        {
            const int b = (ty + H - 1) * LX + lane + H - 1;
            const R* pm = ring + sm * PLANE + b;
            const R* p0 = ring + s0 * PLANE + b;
            const R* pp = ring + sp * PLANE + b;
            stencil_gradient<R>(
                [&](int i) {
                    const R* pl = L::cz[i] < 0 ? pm : (L::cz[i] > 0 ? pp : p0);
                    return pl[(1 + L::cy[i]) * LX + 1 + L::cx[i]];
                },
                gx, gy, gz);
        }
        R Fx = c.fx, Fy = c.fy, Fz = c.fz;
        if (H > 1 && c.nc_range > 0) {
            const PhiRing<R, TX, H> pr{ring, LY};
            ring_near_contact<R, TX, H>(g, pr, s0, xc, yc, cz, ty + H, lane + H, gx, gy, gz, c, Fx, Fy, Fz);
        }
        // ---- pull (x, y, cz), then load what the next plane needs: always, at
        // the same point and for a plane clamped into the lattice, so that a
        // value the loop carries has one source and nothing at the loop head
        // waits for its load
        const LeanRows rw = rows.at(cz);
        const unsigned own = rw.own();
        R t[Q];
        SiteSums<R> m;
        MovingTerms<R> mt;
        if constexpr (W && MV) mt.template init<S, TY>(g, src, rw, ln, rp, r1);
        src.template values<W, TY>(g, rw, ln, rp, k0, r1, r2, pre, [&](int i, R ti, R di) {
            if constexpr (W && MV) mt.add(g, i, rw, ln, yc, cz, ti, di);
            t[i] = ti;
            m.add(i, ti, weight<R>(i) + ti, di);
            settle<W>(m, i);
        });
        {
            const int zn = min(cz + 1, g.nz - 1);
            load_phi(cz + 1 + H, st);
            recs.load(g, src, cz + 2, st.rec);
            const LeanRows rn = rows.at(zn);
            src.template fetch<W, BR>(g, rn, ln, pre);
        }
        SiteTotals<R> tot;
        collide_totals<R>(t, m, gx, gy, gz, Fx, Fy, Fz, c, tot);
        typename D::Kept kept;
        dst.store(g, own, ln, t, tot, site_in, kept);
        if (ragged) {
            asm volatile("");  // (a branch: selects would cost every full tile 23 instructions)
            // lanes beyond the lattice hand nothing to their neighbours
            if (!xin) {
#pragma unroll
                for (int i = 0; i < Q; ++i) t[i] = -weight<R>(i);
                D::clear(kept);
            }
        }
        // ---- phase sums of the next state.  val(i): what direction i carries
        auto val = [&](int i) {
            const R a = weight<R>(i) + t[i];
            return Part2<R>{dst.kept_diff(i, a, kept), a};
        };
        auto add = [](Part2<R>& p, const Part2<R>& q) {
            p.dn += q.dn;
            p.rc += q.rc;
        };
        // sum over the columns of what this row sends in (c_y, c_z) = (e, f):
        // c_x = 0, then from the left, then from the right
        auto row_sum = [&](int e, int f) {
            Part2<R> p = val(dir_of(0, e, f));
            if (e == 0 || f == 0) {
                const Part2<R> l = val(dir_of(1, e, f)), r = val(dir_of(-1, e, f));
                add(p, Part2<R>{from_left(l.dn), from_left(l.rc)});
                add(p, Part2<R>{from_right(r.dn), from_right(r.rc)});
            }
            return p;
        };
        // bounce-backs into this site: its own values, before the in-plane group
        // (off a moving wall, as the next pull reads them)
        if constexpr (W) {
            R ph = R(0);
            bool mv = false;
            if constexpr (MV) {
                mv = moving_next && (rw.ylo || rw.yhi || rw.zlo || rw.zhi || ln.xlo || ln.xhi);
                if (mv) ph = dst.kept_phase(t, kept);
            }
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                if (!(rw.beyond(i) || ln.beyond(i))) continue;
                const R tv = t[L::opp[i]];
                R dv = dst.kept_diff(L::opp[i], weight<R>(i) + tv, kept);
                R wa = weight<R>(i) + tv;
                if (mv) {
                    const R ad = wall_term<R>(g, i, xc, yc, cz);
                    wa = weight<R>(i) + (tv + ad);
                    dv = fma_of(ad, ph, dv);
                }
                cur_rc += wa;
                cur_dn += dv;
            }
        }
        // by destination plane cz - 1, cz, cz + 1: the running sum, then this row's
        // terms, those of the row below (c_y = 1) and of the row above
        Part2<R> to_m{prev_dn, prev_rc}, to_0{cur_dn, cur_rc}, to_p{R(0), R(0)};
        add(to_m, row_sum(0, -1));
        add(to_0, row_sum(0, 0));
        add(to_p, row_sum(0, 1));
        constexpr int STEP = Lds::rounds == 1 ? 2 : 1;  // D beside R, or in a second round
        constexpr int XROW = STEP * kXchSlots * kXchRow;
#pragma unroll
        for (int round = 0; round < Lds::rounds; ++round) {
            if (round) __syncthreads();
            // of row ty to row ty + e; from row ty - e
            auto to_row = [&](int e) { return xch + (e > 0 ? ty : ty - 1) * XROW; };
            auto row_at = [&](int e) { return xch + (e > 0 ? ty - 1 : ty) * XROW; };
            const bool up = ty + 1 < nrows, down = ty > 0 && ty < nrows;  // (uniform)
            auto sends = [&](int e) { return e > 0 ? up : down; };
            auto put = [&](int e, int f, int column, const Part2<R>& p) {
                R* o = to_row(e) + xch_slot(e, f) * kXchRow + column;
                if (STEP == 2 || round == 0) o[0] = p.rc;
                if (STEP == 2) o[kXchSlots * kXchRow] = p.dn;
                else if (round == 1) o[0] = p.dn;
            };
            if (up) {
                put(1, -1, 1 + lane, row_sum(1, -1));
                put(1, 0, 1 + lane, row_sum(1, 0));
                put(1, 1, 1 + lane, row_sum(1, 1));
            }
            if (down) {
                put(-1, -1, 1 + lane, row_sum(-1, -1));
                put(-1, 0, 1 + lane, row_sum(-1, 0));
                put(-1, 1, 1 + lane, row_sum(-1, 1));
            }
            auto pad = [&](int e, int column, const Part2<R>& p) {
                if (sends(e)) put(e, 0, column, p);
            };
            if (round == 0) xedge.own(g, val, pad, vs, ty, cz, k0, za, zb, array_res(part_out + g.N));
            else xedge.pads(val, pad);
            __syncthreads();
            auto have = [&](int e) { return e > 0 ? down : up; };  // (a row beyond the tile: another box's terms)
            auto take = [&](int e, int f, Part2<R>& p) {
                const R* o = row_at(e) + xch_slot(e, f) * kXchRow + 1 + lane;
                if (STEP == 2 || round == 0) p.rc += o[0];
                if (STEP == 2) p.dn += o[kXchSlots * kXchRow];
                else if (round == 1) p.dn += o[0];
            };
            if (have(1)) {
                take(1, -1, to_m);
                take(1, 0, to_0);
                take(1, 1, to_p);
            }
            if (have(-1)) {
                take(-1, -1, to_m);
                take(-1, 0, to_0);
                take(-1, 1, to_p);
            }
            xedge.rows(
                g, round, Lds::rounds,
                [&](int e, int column) {
                    const R* o = row_at(e) + xch_slot(e, 0) * kXchRow + column;
                    const R a = have(e) ? o[0] : R(0);
                    return Part2<R>{STEP == 2 ? (have(e) ? o[kXchSlots * kXchRow] : R(0)) : a, a};
                },
                vs, ty, cz, k0, zb, array_res(part_out + g.N));
        }
        // destination cz - 1 is complete: sources in plane cz are its last group
        if (cz - 1 >= za && site_in) {
            const unsigned row = (unsigned)(cz - 1) * nxy + (unsigned)(y * g.nx);
            if (cz - 1 == za || face_xy)
                res_store(to_m, array_res(part_out), (unsigned)x * (unsigned)sizeof(Part2<R>), row * (unsigned)sizeof(Part2<R>));
            else
                res_store_cached(to_m.dn / to_m.rc, array_res(phi_out), (unsigned)x * (unsigned)sizeof(R),
                                 row * (unsigned)sizeof(R));
        }
        prev_dn = to_0.dn;
        prev_rc = to_0.rc;
        cur_dn = to_p.dn;
        cur_rc = to_p.rc;
        // the chunk's last plane has no own sources above it
        if (cz == zb - 1 && site_in)
            res_store(to_0, array_res(part_out), (unsigned)x * (unsigned)sizeof(Part2<R>), own * (unsigned)sizeof(Part2<R>));
        // no barrier here: the next staging overwrites ring slots that only this
        // plane's pull and collide read, before the exchange's barrier, and the
        // exchange rows are next written after the next staging's barrier
        s0 = sp;
        k0 = r1;
    }
}

template <typename S, typename D, int TY, int H, bool W, bool MV>
__global__ __launch_bounds__(kTileX * TY) void lean_kernel(Geom g, S src, D dst, Coeffs<typename S::R> c, FusedShape fs,
                                                           const Part2<typename S::R>* __restrict__ part_in,
                                                           Part2<typename S::R>* __restrict__ part_out,
                                                           int moving_next) {
    using R = typename S::R;
    extern __shared__ unsigned char lds_raw[];
    int x0, y0, za, zb;
    tile_of_block(fs, kTileX, g.nz, x0, y0, za, zb);
    lean_tile<S, D, TY, H, W, MV>(g, src, dst, c, lds_raw, x0, y0, za, zb,
                                  phi_of<kTileX>(const_cast<Part2<R>*>(part_in), g), part_out,
                                  phi_of<kTileX>(part_out, g), moving_next);
}

}  // namespace lbm
