// lb_lean_first.hip -- the first one-read step of a state that no collision
// made: from its pair arrays into the form the lattice's steps write.
#include "lb_lean_launch.hpp"

namespace lbm {

// (the pairs a first step reads fit wherever the form it writes does)
bool one_read_fits(int storage, size_t N) {
    switch (storage) {
        case LB_STORE_F64: return lean_launch::raw_fits<double>(N) && lean_launch::pairs_fit<double>(N);
        case LB_STORE_F32: return lean_launch::raw_fits<float>(N) && lean_launch::pairs_fit<float>(N);
    }
    return lean_launch::split_fits(N) && lean_launch::pairs_fit<float>(N);
}

template <>
int launch_lean_first<float>(const LatticeView& v, const Coeffs<float>& c, const FusedShape& fs) {
    const size_t N = (size_t)v.g.N;
    const LeanPairs<float> src{(const float*)v.pending};
    if (!one_read_fits(v.p->storage, N)) return lean_launch::too_large();
    switch (v.p->storage) {
        case LB_STORE_F32: return lean_launch::launch(v, src, lean_pack<float>(v.nxt, N), c, fs);
        case LB_STORE_F16: return lean_launch::launch(v, src, lean_split<__half>(v.nxt, N, v.p->scale_log2), c, fs);
        case LB_STORE_BF16:
            return lean_launch::launch(v, src, lean_split<__hip_bfloat16>(v.nxt, N, v.p->scale_log2), c, fs);
    }
    return set_error(LB_EINVAL, "unknown storage");
}

template <>
int launch_lean_first<double>(const LatticeView& v, const Coeffs<double>& c, const FusedShape& fs) {
    const size_t N = (size_t)v.g.N;
    if (!one_read_fits(v.p->storage, N)) return lean_launch::too_large();
    return lean_launch::launch(v, LeanPairs<double>{(const double*)v.pending}, lean_pack<double>(v.nxt, N), c, fs);
}

}  // namespace lbm
