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
    template <typename R>
    __device__ __forceinline__ void pull(const Geom& g, int s, int x, int y, int z, R (&t)[Q], R (&d)[Q]) const {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            int dir;
            const int src = pull_source(g, i, x, y, z, s, dir);
            pull_one<R>(i, src, dir, t[i], d[i]);
        }
        if constexpr (MW) {
            if (g.moving) raw_wall_terms<R>(*this, g, s, x, y, z, t, d);
        }
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
