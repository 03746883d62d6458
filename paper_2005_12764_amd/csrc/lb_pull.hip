// lb_pull.hip -- moments, export and totals of packed and 16-bit states.
#include <algorithm>

#include "lb_lean_launch.hpp"
#include "lb_pull.hpp"

namespace lbm {
namespace {

int status(const char* what) {
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) return LB_OK;
    return set_error(LB_EDEVICE, (std::string(what) + ": " + hipGetErrorString(e)).c_str());
}

// Do tiles read this state sooner than a thread per site?  They read each record
// once, but march planes and leave lanes beyond the lattice idle, so it depends on the
// share of their lanes that are sites, and on the size.  16-bit states, whose decode
// is long: from a quarter (16x512x512 fp16 moments 251 us against 625 site by site;
// at an eighth 470 against 595, at a sixteenth it turns).  Raw states site by site
// keep up with memory, and tiles save the records' traffic.  Moments and totals of
// large lattices: from 0.7 (256^3 FP32 393 us against 442 and 375 against 555;
// 80x458x458, 0.62, 591 against 447); smaller ones: moments from 0.8 without walls
// (128x91x91 26 against 29, between walls 34 against 30; full rows of 2^18 sites, 64^3
// 7.9 against 8.6), FP64 totals (64^3 45 against 53).  Export is bound by its stores: from 0.9 (64x256x256 208 against 229;
// 80x229x229 354 against 254).
enum Reading { MOMENTS, EXPORT, TOTALS };
bool tiles_pay(const LatticeView& v, Reading what) {
    const bool split = v.p->storage >= LB_STORE_F16, f64 = v.p->storage == LB_STORE_F64;
    const int rows = v.p->storage == LB_STORE_F32 ? pull_rows<LeanPack<float>>() : pull_rows<LeanPack<double>>();
    auto share = [](int n, int T) { return double(n) / (double(T) * ((n + T - 1) / T)); };
    const double used = share(v.g.nx, kTX) * share(v.g.ny, rows);
    if (split) return used >= 0.25;
    if (what == EXPORT) return v.g.N >= 1 << 20 && used >= 0.9;
    if (v.g.N >= 1 << 21) return used >= 0.7;
    if (what == TOTALS) return f64 && v.g.N >= 1 << 18 && used >= 0.8;
    return v.g.N >= 1 << 18 && used >= (f64 || v.g.N >= 1 << 19 ? 0.8 : 1.0) && !(v.g.wx || v.g.wy || v.g.wz);
}

// fn(policy) of the current state; taken = false where the state is in pair arrays,
// beyond the policies' 32-bit offsets or read sooner site by site.
template <typename Fn>
int with_policy(const LatticeView& v, Reading what, bool& taken, Fn&& fn) {
    const size_t N = (size_t)v.g.N;
    taken = !v.pending && tiles_pay(v, what);
    if (taken) switch (v.p->storage) {
            case LB_STORE_F64:
                if ((taken = v.packed && lean_launch::raw_fits<double>(N))) return fn(lean_pack<double>(v.cur, N));
                break;
            case LB_STORE_F32:
                if ((taken = v.packed && lean_launch::raw_fits<float>(N))) return fn(lean_pack<float>(v.cur, N));
                break;
            case LB_STORE_F16:
                if ((taken = lean_launch::split_fits(N))) return fn(lean_split<__half>(v.cur, N, v.p->scale_log2));
                break;
            default:
                if ((taken = lean_launch::split_fits(N)))
                    return fn(lean_split<__hip_bfloat16>(v.cur, N, v.p->scale_log2));
        }
    return LB_OK;
}

template <typename K>
int raise_lds(K kern, size_t lds) {
    if (lds <= 65536) return LB_OK;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e == hipSuccess) return LB_OK;
    return set_error(LB_EDEVICE, (std::string("pull kernel LDS: ") + hipGetErrorString(e)).c_str());
}

template <typename S, bool W, bool MV, typename Out>
int run_moments(const LatticeView& v, const S& src, Out* rr, Out* rb, Out* j) {
    const FusedShape fs = pull_shape(v.g, pull_rows<S>());
    auto kern = pull_moments_kernel<S, W, MV, Out>;
    int rc = raise_lds(kern, pull_lds<S>());
    if (rc) return rc;
    hipLaunchKernelGGL(kern, dim3(fs.nblocks), dim3(kTX * fs.TY), pull_lds<S>(), v.stream, v.g, src, fs, rr, rb, j);
    return status("pull_moments_kernel");
}
template <typename S, typename Out>
int moments_of(const LatticeView& v, const S& src, Out* rr, Out* rb, Out* j) {
    if (v.g.moving) return run_moments<S, true, true>(v, src, rr, rb, j);
    if (v.g.wx || v.g.wy || v.g.wz) return run_moments<S, true, false>(v, src, rr, rb, j);
    return run_moments<S, false, false>(v, src, rr, rb, j);
}

template <typename S, bool W, typename Out>
int run_export(const LatticeView& v, const S& src, Out* out) {
    const FusedShape fs = pull_shape(v.g, pull_rows<S>());
    auto kern = pull_export_kernel<S, W, Out>;
    int rc = raise_lds(kern, pull_lds<S>());
    if (rc) return rc;
    hipLaunchKernelGGL(kern, dim3(fs.nblocks), dim3(kTX * fs.TY), pull_lds<S>(), v.stream, v.g, src, fs, out);
    return status("pull_export_kernel");
}

template <typename S, bool W>
int run_totals(const LatticeView& v, const S& src, Neu* partial, int& blocks) {
    const FusedShape fs = pull_shape(v.g, pull_rows<S>());
    auto kern = pull_totals_kernel<S, W>;
    int rc = raise_lds(kern, pull_lds<S>());
    if (rc) return rc;
    blocks = std::min(kTotalsBlocks, fs.nblocks);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kTX * fs.TY), pull_lds<S>(), v.stream, v.g, src, fs, partial);
    return status("pull_totals_kernel");
}

bool walls(const LatticeView& v) { return v.g.wx || v.g.wy || v.g.wz; }

}  // namespace

int pull_moments(const LatticeView& v, void* rr, void* rb, void* j, int dtype, bool& taken) {
    return with_policy(v, MOMENTS, taken, [&](auto src) {
        if (dtype == LB_DTYPE_F64) return moments_of(v, src, (double*)rr, (double*)rb, (double*)j);
        return moments_of(v, src, (float*)rr, (float*)rb, (float*)j);
    });
}

// (off moving walls the export adds the wall terms in FP64 and the totals in the
// storage's arithmetic: those lattices keep the per-site kernels)
int pull_export(const LatticeView& v, void* out, int dtype, bool& taken) {
    if ((taken = !v.g.moving) == false) return LB_OK;
    return with_policy(v, EXPORT, taken, [&](auto src) {
        using S = decltype(src);
        if (dtype == LB_DTYPE_F64)
            return walls(v) ? run_export<S, true>(v, src, (double*)out) : run_export<S, false>(v, src, (double*)out);
        return walls(v) ? run_export<S, true>(v, src, (float*)out) : run_export<S, false>(v, src, (float*)out);
    });
}

int pull_totals(const LatticeView& v, Neu* partial, int& blocks, bool& taken) {
    if ((taken = !v.g.moving) == false) return LB_OK;
    return with_policy(v, TOTALS, taken, [&](auto src) {
        using S = decltype(src);
        return walls(v) ? run_totals<S, true>(v, src, partial, blocks) : run_totals<S, false>(v, src, partial, blocks);
    });
}

}  // namespace lbm
