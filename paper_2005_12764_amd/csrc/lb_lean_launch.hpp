// lb_lean_launch.hpp -- host-side launch of the one-read tile kernel for a
// source and a destination form (shared by the translation units that
// instantiate it).
#pragma once
#include <hip/hip_runtime.h>

#include <string>

#include "lb_internal.hpp"
#include "lb_lean.hpp"

namespace lbm {

// Tile policies of a population buffer.
template <typename T>
__host__ __device__ __forceinline__ LeanPack<T> lean_pack(void* buf, size_t N) {
    return LeanPack<T>{(T*)buf, (T*)buf + pack_t_offset<T>(N)};
}
template <typename H>
LeanSplit<H> lean_split(void* buf, size_t N, int scale_log2) {
    const SplitPop<H> s = split_view<H>(buf, N, scale_log2);
    return LeanSplit<H>{s.rec, s.dev, s};
}

namespace lean_launch {

template <typename S, typename D, int TY, int HALO, bool W, bool MV>
int launch_h(const LatticeView& v, const S& src, const D& dst, const Coeffs<typename S::R>& c, const FusedShape& fs) {
    using R = typename S::R;
    const size_t lds = LeanLds<S, TY, HALO>::bytes;
    auto kern = lean_kernel<S, D, TY, HALO, W, MV>;
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return set_error(LB_EDEVICE, (std::string("lean_kernel LDS: ") + hipGetErrorString(e)).c_str());
    }
    // the next step's pull adds moving-wall terms even when this one (the
    // first after a state was set) does not: the gathered sums follow the next
    const int moving_next = make_geom(*v.p).moving;
    hipLaunchKernelGGL(kern, dim3(fs.nblocks), dim3(kTX * TY), lds, v.stream, v.g, src, dst, c, fs,
                       (const Part2<R>*)v.part_in, (Part2<R>*)v.part_out, moving_next);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(LB_EDEVICE, (std::string("lean_kernel: ") + hipGetErrorString(e)).c_str());
    return LB_OK;
}

template <typename S, typename D, int TY, int HALO>
int launch_w(const LatticeView& v, const S& src, const D& dst, const Coeffs<typename S::R>& c, const FusedShape& fs) {
    // walls at rest and moving walls take separate instantiations (the
    // resting-wall kernel holds none of the wall-term code); the first step of a
    // state, taken once, has one for every kind of wall
    const bool walls = v.g.wx || v.g.wy || v.g.wz;
    if (!walls) return launch_h<S, D, TY, HALO, false, false>(v, src, dst, c, fs);
    if (S::NC == 0 || v.g.moving || make_geom(*v.p).moving)
        return launch_h<S, D, TY, HALO, true, true>(v, src, dst, c, fs);
    if constexpr (S::NC > 0) return launch_h<S, D, TY, HALO, true, false>(v, src, dst, c, fs);
    return LB_EINVAL;
}

// Halos and rows whose rings fit a workgroup's LDS are instantiated (tile_rows
// picks no others).
template <typename S, typename D, int TY, int HALO>
int launch_halo(const LatticeView& v, const S& src, const D& dst, const Coeffs<typename S::R>& c,
                const FusedShape& fs) {
    if constexpr (LeanLds<D, TY, HALO>::bytes <= kLdsBytes) return launch_w<S, D, TY, HALO>(v, src, dst, c, fs);
    return set_error(LB_EINVAL, "one-read tile does not fit in LDS");
}

template <typename S, typename D, int TY>
int launch_ty(const LatticeView& v, const S& src, const D& dst, const Coeffs<typename S::R>& c, const FusedShape& fs) {
    switch (tile_halo(*v.p)) {
        case 1: return launch_halo<S, D, TY, 1>(v, src, dst, c, fs);
        case 2: return launch_halo<S, D, TY, 2>(v, src, dst, c, fs);
        case 3: return launch_halo<S, D, TY, 3>(v, src, dst, c, fs);
        case 4: return launch_halo<S, D, TY, 4>(v, src, dst, c, fs);
        case 5: return launch_halo<S, D, TY, 5>(v, src, dst, c, fs);
    }
    return set_error(LB_EINVAL, "near-contact range outside the tile kernels' halo");
}

template <typename S, typename D>
int launch(const LatticeView& v, const S& src, const D& dst, const Coeffs<typename S::R>& c, const FusedShape& fs) {
    switch (fs.TY) {
        case kSingleTYSmall: return launch_ty<S, D, kSingleTYSmall>(v, src, dst, c, fs);
        case kSingleTY: return launch_ty<S, D, kSingleTY>(v, src, dst, c, fs);
        case kSingleTYLarge: return launch_ty<S, D, kSingleTYLarge>(v, src, dst, c, fs);
        case kSingleTYSplit:
            if constexpr (D::kSplit) return launch_ty<S, D, kSingleTYSplit>(v, src, dst, c, fs);
    }
    return set_error(LB_EINVAL, "one-read tile rows outside the storage's choices");
}

// 32-bit byte offsets within the buffer resources.
template <typename T>
bool raw_fits(size_t N) {
    return (uint64_t)kResArrays * sizeof(T) * (uint64_t)raw_stride(N) < ((uint64_t)1 << 32);
}
template <typename T>
bool pairs_fit(size_t N) {
    return (uint64_t)2 * kResPairs * sizeof(T) * (uint64_t)raw_stride(N) < ((uint64_t)1 << 32);
}
inline bool split_fits(size_t N) {
    return (uint64_t)32 * N < ((uint64_t)1 << 32) && (uint64_t)2 * Q * (uint64_t)dev_stride(N) < ((uint64_t)1 << 32);
}
inline int too_large() { return set_error(LB_EINVAL, "lattice too large for the one-read step's 32-bit offsets"); }

}  // namespace lean_launch
}  // namespace lbm
