// lb_lean16.hip -- one-read tile kernel for the 16-bit moment-split storage
// (fp16, bf16).
#include "lb_lean_launch.hpp"

namespace lbm {

template <typename H>
int launch_lean_split(const LatticeView& v, const Coeffs<float>& c, const FusedShape& fs) {
    const size_t N = (size_t)v.g.N;
    if (!lean_launch::split_fits(N)) return lean_launch::too_large();
    return lean_launch::launch(v, lean_split<H>(v.cur, N, v.p->scale_log2), lean_split<H>(v.nxt, N, v.p->scale_log2), c,
                               fs);
}

template int launch_lean_split<__half>(const LatticeView&, const Coeffs<float>&, const FusedShape&);
template int launch_lean_split<__hip_bfloat16>(const LatticeView&, const Coeffs<float>&, const FusedShape&);

}  // namespace lbm
