// lb_lean.hip -- one-read tile kernel for packed FP32 storage, and the LDS of
// the tiles.
#include "lb_lean_launch.hpp"

namespace lbm {

template <>
int launch_lean_raw<float>(const LatticeView& v, const Coeffs<float>& c, const FusedShape& fs) {
    const size_t N = (size_t)v.g.N;
    if (!lean_launch::raw_fits<float>(N)) return lean_launch::too_large();
    return lean_launch::launch(v, lean_pack<float>(v.cur, N), lean_pack<float>(v.nxt, N), c, fs);
}

namespace {
template <typename S, int TY>
size_t lds_of(int H) {
    switch (H) {
        case 1: return LeanLds<S, TY, 1>::bytes;
        case 2: return LeanLds<S, TY, 2>::bytes;
        case 3: return LeanLds<S, TY, 3>::bytes;
        case 4: return LeanLds<S, TY, 4>::bytes;
        default: return LeanLds<S, TY, 5>::bytes;
    }
}
template <typename S>
size_t lds_of(int TY, int H) {
    switch (TY) {
        case kSingleTYSmall: return lds_of<S, kSingleTYSmall>(H);
        case kSingleTY: return lds_of<S, kSingleTY>(H);
        case kSingleTYSplit: return lds_of<S, kSingleTYSplit>(H);
        default: return lds_of<S, kSingleTYLarge>(H);
    }
}
}  // namespace

size_t lean_tile_lds(const lb_params& p, int TY) {
    const int H = tile_halo(p);
    if (p.storage == LB_STORE_F64) return lds_of<LeanPack<double>>(TY, H);
    if (p.storage == LB_STORE_F32) return lds_of<LeanPack<float>>(TY, H);
    return lds_of<LeanSplit<__half>>(TY, H);
}

}  // namespace lbm
