// lb_lean64.hip -- one-read tile kernel for packed FP64 storage.
#include "lb_lean_launch.hpp"

namespace lbm {

template <>
int launch_lean_raw<double>(const LatticeView& v, const Coeffs<double>& c, const FusedShape& fs) {
    const size_t N = (size_t)v.g.N;
    if (!lean_launch::raw_fits<double>(N)) return lean_launch::too_large();
    return lean_launch::launch(v, lean_pack<double>(v.cur, N), lean_pack<double>(v.nxt, N), c, fs);
}

}  // namespace lbm
