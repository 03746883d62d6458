// lb_internal.hpp -- declarations shared by the host translation units.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <string>
#include <type_traits>

#include "lb.h"
#include "lb_pack.hpp"
#include "lb_single.hpp"

namespace lbm {

// Blocks of the compensated-reduction kernel (fixed, so totals are bitwise
// reproducible for a given lattice).
constexpr int kTotalsBlocks = 512;
// Most of the one that reads packed states site by site: as many as are resident at
// once, four wavefronts per SIMD in FP32 (1x4096x4096 497 us, 560 with 512 blocks),
// three off moving walls, two in FP64.  The partial sums' buffers hold as many.
constexpr int kPackTotalsBlocks = 1024;

// What a launch needs to know about one lattice.
struct LatticeView {
    const lb_params* p = nullptr;
    Geom g;
    hipStream_t stream = nullptr;
    void* cur = nullptr;       // post-collision buffer holding the current state
    void* nxt = nullptr;       // buffer the next step writes
    void* pending = nullptr;   // pair arrays of a state no collision made, of a lattice whose steps
                               // write another form (else null)
    bool packed = false;       // raw storage: steps write (and, unless pending, cur holds) the packed form
    void* phi = nullptr;       // phase-field scratch of the two-pass step
    void* part_in = nullptr;   // phase sums and phase field of the current state (one-read step)
    void* part_out = nullptr;  // the same, written by the one-read step for the next state
    bool part_valid = false;   // part_in holds the current state's sums
    FusedShape shape{};        // tile shape of the one-read step
    Coeffs<double> cd;
    Coeffs<float> cf;
};

int set_error(int code, const char* msg);
int validate_params(const lb_params* p, std::string& why);
template <typename R>
Coeffs<R> make_coeffs(const lb_params& p);
Geom make_geom(const lb_params& p);
size_t pop_bytes(int storage, size_t N);

// Views of a population buffer.
template <typename T, bool MW = false>
PackPop<T, MW> pack_view(void* buf, size_t N) {
    return PackPop<T, MW>{(const T*)buf, (const T*)buf + pack_t_offset<T>(N), N};
}
template <typename H, bool MW = false>
SplitPop<H, MW> split_view(void* buf, size_t N, int scale_log2) {
    SplitPop<H, MW> s;
    s.rec = (float*)buf;
    s.dev = (H*)((float*)buf + 8 * N);
    s.N = N;
    const float sc = std::is_same<H, __half>::value ? std::ldexp(1.0f, scale_log2) : 1.0f;
    s.scale = sc;
    s.inv_scale = 1.0f / sc;
    return s;
}

// Tile kernels: 64-wide tiles of TY rows marching z-chunks of TZ planes.
constexpr int kTX = kTileX;
enum TileKind { TILE_COLLIDE = 0, TILE_SINGLE = 1, TILE_PHASE = 2, TILE_BATCH = 3 };
// Tile shape set through lb_set_tiles for (kind, storage): 0 = unset.
struct TileSetting {
    int ty, tz;
};
TileSetting tile_setting(int kind, int storage);
void set_tile_setting(int kind, int storage, int ty, int tz);
int env_int(const char* name, int dflt);
int tile_halo(const lb_params& p);
size_t tile_lds(const lb_params& p, int kind, int TY);
int tile_rows(const lb_params& p, int kind);
FusedShape tile_shape(const lb_params& p, int kind);
// A shape of this kind was asked for (lb_set_tiles or the environment).
bool tile_shape_asked(const lb_params& p, int kind);

int choose_kernel(const lb_params& p);
// Events recorded around the passes of one step (null = no timing):
// ev[0] before the step, ev[1] between the phase and the collide pass (equal
// to ev[0] for the fused kernel), ev[2] after the step.
struct StepEvents {
    hipEvent_t ev[3];
};
int launch_step(const LatticeView& v, int kernel, const StepEvents* t = nullptr);
// Tile kernel of the one-read step (lb_lean*.hip): collide and stream the
// current state into v.nxt, gathering the next state's own phase sums.  raw:
// packed storage; split: 16-bit moment-split storage; first: from pair arrays
// (v.pending) into either.
template <typename T>
int launch_lean_raw(const LatticeView& v, const Coeffs<T>& c, const FusedShape& fs);
template <typename H>
int launch_lean_split(const LatticeView& v, const Coeffs<float>& c, const FusedShape& fs);
template <typename T>
int launch_lean_first(const LatticeView& v, const Coeffs<T>& c, const FusedShape& fs);
size_t lean_tile_lds(const lb_params& p, int TY);
// The buffer offsets of the one-read step and of a state's first one fit 32 bits.
bool one_read_fits(int storage, size_t N);
// Pair arrays of the current packed state (a checkpoint's form) into f.
int launch_unpack(const LatticeView& v, void* f);
// Zeros between the pair arrays of f.
int launch_clear_pads(const LatticeView& v, void* f);
// Moments, export and totals of a packed or 16-bit state through marching tiles
// (lb_pull.hip); taken = false: the state has another form, nothing was done.
int pull_moments(const LatticeView& v, void* rr, void* rb, void* j, int dtype, bool& taken);
int pull_export(const LatticeView& v, void* out, int dtype, bool& taken);
int pull_totals(const LatticeView& v, Neu* partial, int& blocks, bool& taken);
int launch_init(const LatticeView& v, const void* rr, const void* rb, const void* u, int dtype);
int launch_import(const LatticeView& v, const void* f, int dtype);
int launch_export(const LatticeView& v, void* out, int dtype);
int launch_moments(const LatticeView& v, void* rr, void* rb, void* j, int dtype);
int launch_korteweg(const LatticeView& v, double lam, int b, void* kout, void* pout, int dtype, int accumulate);
int launch_totals(const LatticeView& v, Neu* partial, double* dtot);
int launch_droplets(hipStream_t st, const Geom& g, const double* cen, const double* rad, int n, double width,
                    double background, double rho0, double* rr, double* rb);

}  // namespace lbm
