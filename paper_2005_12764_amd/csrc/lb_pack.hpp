// lb_pack.hpp -- packed raw (FP64/FP32) storage: what a one-read step writes.
//
// After recolouring the 19 colour differences of a site follow from its 19
// totals, its phase and its recolouring vector (recoloured()), so a state that
// a step has collided is 23 values per site instead of the 38 of the pair
// arrays: FP32 moves 184 B per site and step instead of 304.  The pair arrays
// (RawPop) remain the form of states that no collision made (initial, imported,
// loaded from a checkpoint), which hold 38 independent values, and of saved
// states.
//
// Layout: the colour records [N] (phi, s_x, s_y, s_z), 16 bytes per value of
// four FP32, then 19 arrays t_i, raw_stride(N) values apart (the padding of the
// pair arrays).  A packed state fits the buffer of the pair arrays.
#pragma once
#include "lb_kernels.hpp"

namespace lbm {

template <typename T>
__host__ __device__ constexpr size_t pack_t_offset(size_t N) { return 4 * N; }

template <typename T, bool MW = false>
struct PackPop {
    const T* rec;
    const T* tot;
    size_t N;

    __device__ __forceinline__ Colour<T> colour(int s) const {
        const T* r = rec + 4 * (size_t)s;
        return Colour<T>{r[0], r[1], r[2], r[3]};
    }
    // t, d that direction i takes from the stored direction dir of site src
    template <typename R>
    __device__ __forceinline__ void pull_one(int i, int src, int dir, R& t, R& d) const {
#pragma clang fp contract(off)
        const T v = tot[(size_t)dir * raw_stride(N) + src];
        const Colour<T> q = colour(src);
        const T cs = dir == i ? recoloured<T>(i, weight<T>(i) + v, q)
                              : recoloured<T>(Lattice::opp[i], weight<T>(i) + v, q);
        t = R(v);
        d = R(cs);
    }
    // The site's 19 values, for kernels whose consecutive lanes take consecutive
    // sites: of the 19 source records a lane loads one per source row and takes those
    // beside it from its neighbours' (lanes at the ends of a row or of the wavefront
    // load theirs), and a value is addressed by one 32-bit offset.  Issue bound these
    // readings: 1x2048x2048 FP32, totals 302 -> 154 us, moments 150 -> 118, export 292
    // -> 248 against 19 record loads and 64-bit addresses (pair arrays: 152, 145, 247).
    template <typename R>
    __device__ __forceinline__ void pull(const Geom& g, int s, int x, int y, int z, R (&t)[Q], R (&d)[Q]) const {
        if (MW || g.wx || g.wy || g.wz) pull_rows<true, R>(g, s, x, y, z, t, d);
        else pull_rows<false, R>(g, s, x, y, z, t, d);
    }
    template <bool W, typename R>
    __device__ __forceinline__ void pull_rows(const Geom& g, int s, int x, int y, int z, R (&t)[Q], R (&d)[Q]) const {
#pragma clang fp contract(off)
        using L = Lattice;
        const int lane = threadIdx.x & 63;
        const int xm = x == 0 ? g.nx - 1 : x - 1, xp = x == g.nx - 1 ? 0 : x + 1;
        const bool first = lane == 0 || x == 0, last = lane == 63 || x == g.nx - 1;
        const bool xlo = W && g.wx && x == 0, xhi = W && g.wx && x == g.nx - 1;
        const Colour<T> own = colour(s);
#pragma unroll
        for (int row = 0; row < 9; ++row) {
            const int e = row % 3 - 1, f = row / 3 - 1;  // c_y, c_z of the row's directions
            bool beyond = false;
            const int ys = e ? step_back(y, e, g.ny, g.wy, beyond) : y;
            const int zs = f ? step_back(z, f, g.nz, g.wz, beyond) : z;
            const int base = site_of(g, 0, ys, zs);
            Colour<T> q[3] = {own, own, own};  // from the left, the own column, the right
            if (e || f) q[1] = colour(W && beyond ? s : base + x);
            if (!e || !f) {
                q[0] = beside<0x138>(q[1]);
                q[2] = beside<0x130>(q[1]);
                if (first) q[0] = colour(base + xm);
                if (last) q[2] = colour(base + xp);
            }
#pragma unroll
            for (int cx = 1; cx >= -1; --cx) {
                if (cx && e && f) continue;
                const int i = dir_at(cx, e, f);
                const bool refl = W && (beyond || (cx > 0 && xlo) || (cx < 0 && xhi));
                // (of two runs of arrays, a direction and its opposite in one: a packed
                // lattice is one whose 10 arrays span less than 2^32 bytes)
                const int run = i < 9 ? 0 : 9;
                const unsigned S = (unsigned)raw_stride(N);
                const unsigned src = (unsigned)(base + (cx > 0 ? xm : (cx < 0 ? xp : x)));
                const unsigned at = refl ? (unsigned)(L::opp[i] - run) * S + (unsigned)s : (unsigned)(i - run) * S + src;
                const T v = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(tot + (size_t)run * S) +
                                                        (size_t)(at * (unsigned)sizeof(T)));
                const Colour<T>& c = q[1 - cx];
                t[i] = R(v);
                d[i] = R(recoloured<T>(i, weight<T>(i) + v,
                                       refl ? Colour<T>{own.phi, -own.sx, -own.sy, -own.sz} : c));
            }
        }
        if constexpr (MW) {
            const bool ylo = g.wy && y == 0, yhi = g.wy && y == g.ny - 1, zlo = g.wz && z == 0, zhi = g.wz && z == g.nz - 1;
            if (g.moving && (xlo || xhi || ylo || yhi || zlo || zhi)) {
                const R ph = own_phase<R>(s);  // shares the walls' terms between the components
#pragma unroll
                for (int i = 1; i < Q; ++i) {
                    const bool refl = (L::cx[i] > 0 && xlo) || (L::cx[i] < 0 && xhi) || (L::cy[i] > 0 && ylo) ||
                                      (L::cy[i] < 0 && yhi) || (L::cz[i] > 0 && zlo) || (L::cz[i] < 0 && zhi);
                    const R add = refl ? wall_term<R>(g, i, x, y, z) : R(0);
                    t[i] = refl ? t[i] + add : t[i];
                    d[i] = refl ? fma_of(add, ph, d[i]) : d[i];
                }
            }
        }
    }
    // the colour of the lane before (DPP 0x138) or after (0x130)
    template <int DPP>
    static __device__ __forceinline__ Colour<T> beside(const Colour<T>& q) {
        return Colour<T>{shifted<DPP>(q.phi), shifted<DPP>(q.sx), shifted<DPP>(q.sy), shifted<DPP>(q.sz)};
    }
    template <int DPP>
    static __device__ __forceinline__ T shifted(T v) {
        if constexpr (sizeof(T) == 4) {
            return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), DPP, 0xf, 0xf, true));
        } else {
            const long long b = __double_as_longlong(v);
            const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), DPP, 0xf, 0xf, true);
            const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), DPP, 0xf, 0xf, true);
            return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
        }
    }
    static constexpr int dir_at(int cx, int cy, int cz) {
        for (int i = 0; i < Q; ++i)
            if (Lattice::cx[i] == cx && Lattice::cy[i] == cy && Lattice::cz[i] == cz) return i;
        return -1;
    }
    // The site's own post-collision phase, summed as RawPop sums its pairs.
    template <typename R>
    __device__ __forceinline__ R own_phase(int s) const {
        R st = R(0), sd = R(0);
        const Colour<T> q = colour(s);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const T v = tot[(size_t)j * raw_stride(N) + s];
            st += weight<R>(j) + R(v);
            sd += R(recoloured<T>(j, weight<T>(j) + v, q));
        }
        return sd / st;
    }
    static constexpr bool ring = false;
    static constexpr bool moving = MW;
};

// The pair arrays of a packed state (what a checkpoint holds), the unused pairs after
// each array as zeros, so that equal states are saved as equal bytes.  Bound by
// memory: 92 B read and 152 written per site in FP32.  256x256x128 into the caller's
// buffer 390 us; 882 through a population buffer and a copy, 500 the copy of a state
// held in pairs.
template <typename T>
__global__ __launch_bounds__(256) void unpack_kernel(int n, PackPop<T> src, T* __restrict__ f) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n + kRawPad) return;
    if (s >= n) {
#pragma unroll
        for (int i = 0; i < Q; ++i) raw_put(f, src.N, i, s, T(0), T(0));
        return;
    }
    const Colour<T> q = src.colour(s);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const T t = src.tot[(size_t)i * raw_stride(src.N) + s];
        raw_put(f, src.N, i, s, t, recoloured<T>(i, weight<T>(i) + t, q));
    }
}

// Zeros in the unused pairs after each pair array.
template <typename T>
__global__ __launch_bounds__(kRawPad * Q) void clear_pads_kernel(size_t N, T* __restrict__ f) {
    raw_put(f, N, (int)(threadIdx.x / kRawPad), (int)(N + threadIdx.x % kRawPad), T(0), T(0));
}

}  // namespace lbm
