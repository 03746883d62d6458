// lb_launch.hip -- kernel instantiation and dispatch over storage types.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cmath>
#include <string>
#include <type_traits>

#include "lb_internal.hpp"
#include "lb_korteweg.hpp"
#include "lb_lean.hpp"
#include "lb_shanchen.hpp"
#include "lb_single.hpp"

namespace lbm {

namespace {

constexpr int kBlock = 256;
int max_lds_bytes();
int device_lds_bytes();
size_t real_size(const lb_params& p);
bool split_storage(const lb_params& p);

int launch_status(const char* what) {
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) return LB_OK;
    std::string m = std::string(what) + ": " + hipGetErrorString(e);
    return set_error(LB_EDEVICE, m.c_str());
}

unsigned grid_for(int N) { return (unsigned)((N + kBlock - 1) / kBlock); }

// Calls fn(R{}, src, coeffs) with the compute type and a view of the current
// state in its storage; lattices with moving walls get the storage types that
// add the moving-wall terms (the first state of a 16-bit lattice is never pulled
// with them).
template <bool MW, typename Fn>
int with_state_mw(const LatticeView& v, Fn&& fn) {
    const size_t N = (size_t)v.g.N;
    switch (v.p->storage) {
        case LB_STORE_F64:
            if (v.packed && !v.pending) return fn(double(0), pack_view<double, MW>(v.cur, N), v.cd);
            return fn(double(0), RawPop<double, MW>{(double*)(v.pending ? v.pending : v.cur), N}, v.cd);
        case LB_STORE_F32:
            if (v.packed && !v.pending) return fn(float(0), pack_view<float, MW>(v.cur, N), v.cf);
            return fn(float(0), RawPop<float, MW>{(float*)(v.pending ? v.pending : v.cur), N}, v.cf);
        case LB_STORE_F16:
            if (v.pending) return fn(float(0), RawPop<float>{(float*)v.pending, N}, v.cf);
            return fn(float(0), split_view<__half, MW>(v.cur, N, v.p->scale_log2), v.cf);
        case LB_STORE_BF16:
            if (v.pending) return fn(float(0), RawPop<float>{(float*)v.pending, N}, v.cf);
            return fn(float(0), split_view<__hip_bfloat16, MW>(v.cur, N, v.p->scale_log2), v.cf);
    }
    return set_error(LB_EINVAL, "unknown storage");
}

template <typename Fn>
int with_state(const LatticeView& v, Fn&& fn) {
    if (v.g.moving) return with_state_mw<true>(v, fn);
    return with_state_mw<false>(v, fn);
}

// LDS per workgroup the device allows (160 KiB on gfx950).
int device_lds_bytes() {
    static int cached = -1;
    if (cached < 0) {
        int dev = 0, v = 0;
        (void)hipGetDevice(&dev);
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
            v = 65536;
        cached = v;
    }
    return cached;
}

// Budget of the two-pass tile kernels (64 KiB: more LDS per workgroup would
// cost them occupancy).
int max_lds_bytes() { return std::min(device_lds_bytes(), 65536); }

size_t real_size(const lb_params& p) { return p.storage == LB_STORE_F64 ? 8 : 4; }

bool split_storage(const lb_params& p) { return p.storage >= LB_STORE_F16; }

// Collide pass of the two-pass step: z-marching tiles reading the phase
// pass's phi through an LDS ring.
template <typename R, typename Src, typename Dst, int H>
int zmarch_h(const LatticeView& v, const Src& src, const Dst& dst, const Coeffs<R>& c, const R* phi_in) {
    const FusedShape fs = tile_shape(*v.p, TILE_COLLIDE);
    const size_t lds = tile_lds(*v.p, TILE_COLLIDE, fs.TY);
    hipLaunchKernelGGL((fused_kernel<R, Src, Dst, kTX, H>), dim3(fs.nblocks), dim3(kBlock), lds, v.stream, v.g, src,
                       dst, c, fs, phi_in);
    return launch_status("collide pass");
}

template <typename R, typename Src, typename Dst>
int zmarch(const LatticeView& v, const Src& src, const Dst& dst, const Coeffs<R>& c, const R* phi_in) {
    switch (tile_halo(*v.p)) {
        case 1: return zmarch_h<R, Src, Dst, 1>(v, src, dst, c, phi_in);
        case 2: return zmarch_h<R, Src, Dst, 2>(v, src, dst, c, phi_in);
        case 3: return zmarch_h<R, Src, Dst, 3>(v, src, dst, c, phi_in);
        case 4: return zmarch_h<R, Src, Dst, 4>(v, src, dst, c, phi_in);
        case 5: return zmarch_h<R, Src, Dst, 5>(v, src, dst, c, phi_in);
    }
    return set_error(LB_EINVAL, "near-contact range outside the tile kernels' halo");
}

// One-read step: the own partial sums of the current state (and phi where
// they are complete) come from the previous one-read step, or from
// part_kernel when no such step made them; assemble_kernel adds the
// cross-tile terms into phi of the face sites; the tile kernel collides,
// streams and gathers the next state's sums and interior phi.
int lean_step(const LatticeView& v, const FusedShape& fs) {
    switch (v.p->storage) {
        case LB_STORE_F64: return v.pending ? launch_lean_first<double>(v, v.cd, fs) : launch_lean_raw<double>(v, v.cd, fs);
        case LB_STORE_F32: return v.pending ? launch_lean_first<float>(v, v.cf, fs) : launch_lean_raw<float>(v, v.cf, fs);
        case LB_STORE_F16: return v.pending ? launch_lean_first<float>(v, v.cf, fs) : launch_lean_split<__half>(v, v.cf, fs);
        case LB_STORE_BF16:
            return v.pending ? launch_lean_first<float>(v, v.cf, fs) : launch_lean_split<__hip_bfloat16>(v, v.cf, fs);
    }
    return set_error(LB_EINVAL, "unknown storage");
}

// phi of the face sites of a one-read state (its interior phi is already in
// the phase-sum buffer).
template <typename R, typename Src, int TY>
int assemble_phase(const LatticeView& v, const Src& src, const FusedShape& fs) {
    const FaceSet faces = face_set(v.g, kTX, TY, fs.TZ);
    hipLaunchKernelGGL((assemble_kernel<R, Src, kTX, TY>), dim3(grid_for(faces.row_sites + faces.edge_sites)),
                       dim3(kBlock), 0, v.stream, v.g, src, faces, (Part2<R>*)v.part_in);
    return launch_status("assemble_kernel");
}

template <typename R, typename Src, int TY>
int single_ty(const LatticeView& v, const Src& src, const FusedShape& fs, const StepEvents* t) {
    if (!v.part_valid) {
        hipLaunchKernelGGL((part_kernel<R, Src, kTX, TY>), dim3(grid_for(v.g.N)), dim3(kBlock), 0, v.stream, v.g,
                           src, fs.TZ, (Part2<R>*)v.part_in);
        int rc = launch_status("part_kernel");
        if (rc) return rc;
    }
    int rc = assemble_phase<R, Src, TY>(v, src, fs);
    if (rc) return rc;
    if (t) (void)hipEventRecord(t->ev[1], v.stream);
    return lean_step(v, fs);
}

template <typename R, typename Src>
int single_pass(const LatticeView& v, const Src& src, const StepEvents* t) {
    if (!v.part_in || !v.part_out) return set_error(LB_EINVAL, "one-read step without its phase buffers");
    const FusedShape fs = v.shape;
    if (t) (void)hipEventRecord(t->ev[0], v.stream);
    if (fs.TY <= 0) return set_error(LB_EINVAL, "one-read tile does not fit in LDS");
    const int rc = with_rows(fs.TY, [&](auto ty) { return single_ty<R, Src, decltype(ty)::value>(v, src, fs, t); });
    if (rc) return rc;
    if (t) (void)hipEventRecord(t->ev[2], v.stream);
    return LB_OK;
}

// Phase pass: raw storage pulls site by site; 16-bit moment-split storage
// runs z-marching tiles with the source records staged in LDS.
template <typename R, typename Src>
int phase_pass(const LatticeView& v, const Src& src) {
    if constexpr (Src::ring) {
        if (tile_rows(*v.p, TILE_PHASE) > 0) {
            const FusedShape fs = tile_shape(*v.p, TILE_PHASE);
            hipLaunchKernelGGL((phase_tile_kernel<R, Src, kTX>), dim3(fs.nblocks), dim3(kBlock),
                               tile_lds(*v.p, TILE_PHASE, fs.TY), v.stream, v.g, src, (R*)v.phi, fs);
            return launch_status("phase_tile_kernel");
        }
    }
    hipLaunchKernelGGL((phase_kernel<R, Src>), dim3(grid_for(v.g.N)), dim3(kBlock), 0, v.stream, v.g, src, (R*)v.phi);
    return launch_status("phase_kernel");
}

// Tiles of the one-pass Shan-Chen step: one workgroup per CU (a workgroup pulls
// two planes more than it writes; 128^3: 162 us with 16 planes, 174 with 8, 207
// with 12, 236 with 32; 256^3: 1.07 ms with 128, 1.16 with 16).
FusedShape sc_shape(const Geom& g) {
    FusedShape fs;
    fs.TY = kScRows;
    fs.tiles_x = (g.nx + kTX - 1) / kTX;
    fs.tiles_y = (g.ny + kScRows - 1) / kScRows;
    const int tiles = fs.tiles_x * fs.tiles_y;
    const int chunks = std::max(1, 256 / tiles);
    fs.TZ = (g.nz + chunks - 1) / chunks;
    fs.chunks = (g.nz + fs.TZ - 1) / fs.TZ;
    fs.nblocks = tiles * fs.chunks;
    return fs;
}
// Does one pass beat two?  Within the 32-bit offsets of its row loads, where chunks are
// three planes or more, two of full rows (48^3 two planes 22 us against 17 with two
// passes, 64^3 25.5 against 27, 512x512x1 one plane 33 against 26), and more lanes than
// about half are sites (8x256x256 173 against 141, 33x154x225, 0.52, 132 against 122;
// 70x90x300, 0.55, 222 against 234, 40x160x160 98 against 113).
bool sc_one(const Geom& g) {
    const bool fits = (uint64_t)kResArrays * sizeof(float) * (uint64_t)raw_stride((size_t)g.N) < ((uint64_t)1 << 32);
    const double lanes = double(g.nx) / (kTX * ((g.nx + kTX - 1) / kTX));
    return fits && lanes >= 0.53 && sc_shape(g).TZ >= (lanes == 1.0 ? 2 : 3);
}

// Shan-Chen step (raw storage): density pass, then the collide tiles with the
// density pairs in an LDS ring.
template <typename R, typename Src, typename Dst>
int sc_two_pass(const LatticeView& v, const Src& src, const Dst& dst, const Coeffs<R>& c, const StepEvents* t) {
    RhoPair<R>* rho2 = (RhoPair<R>*)v.phi;
    hipLaunchKernelGGL((sc_density_kernel<R, Src>), dim3(grid_for(v.g.N)), dim3(kBlock), 0, v.stream, v.g, src, rho2);
    int rc = launch_status("sc_density_kernel");
    if (rc) return rc;
    if (t) (void)hipEventRecord(t->ev[1], v.stream);
    const FusedShape fs = tile_shape(*v.p, TILE_COLLIDE);
    const size_t lds = sc_ring_bytes<R>(fs.TY, kTX);
    hipLaunchKernelGGL((sc_collide_kernel<R, Src, Dst, kTX>), dim3(fs.nblocks), dim3(kBlock), lds, v.stream, v.g, src,
                       dst, c, fs, (const RhoPair<R>*)rho2);
    return launch_status("sc_collide_kernel");
}

template <typename R, typename Src, typename Dst, bool W>
int sc_one_pass(const LatticeView& v, const Src& src, const Dst& dst, const Coeffs<R>& c) {
    const FusedShape fs = sc_shape(v.g);
    hipLaunchKernelGGL((sc_step_kernel<R, Src, Dst, W>), dim3(fs.nblocks), dim3(kTX * kScRows), sc_step_bytes<R>(),
                       v.stream, v.g, src, LeanPairs<R>{(const R*)v.cur}, dst, c, fs);
    return launch_status("sc_step_kernel");
}

// One pass for FP32 without moving walls where it pays; two passes otherwise.  (In FP64 the values of two sites and a third's in
// flight exceed the registers, 440 B spill and 128^3 takes 636 us against 387; the
// terms of moving walls spill too.)
template <typename R, typename Src, typename Dst>
int sc_step(const LatticeView& v, const Src& src, const Dst& dst, const Coeffs<R>& c, const StepEvents* t) {
    if constexpr (Src::ring || Dst::ring) {
        return set_error(LB_EINVAL, "the Shan-Chen model needs raw storage");
    } else {
        if (t) (void)hipEventRecord(t->ev[0], v.stream);
        int rc = LB_OK;
        bool one = false;
        if constexpr (sizeof(R) == 4 && !Src::moving) {
            one = sc_one(v.g);
            if (one) {
                if (t) (void)hipEventRecord(t->ev[1], v.stream);  // (no pass before the collide pass)
                rc = v.g.wx || v.g.wy || v.g.wz ? sc_one_pass<R, Src, Dst, true>(v, src, dst, c)
                                                : sc_one_pass<R, Src, Dst, false>(v, src, dst, c);
            }
        }
        if (!one) rc = sc_two_pass<R>(v, src, dst, c, t);
        if (t) (void)hipEventRecord(t->ev[2], v.stream);
        return rc;
    }
}

// Two passes: the phase pass writes phi; the collide pass z-marches tiles
// with phi in an LDS ring (or, when the ring does not fit, reads phi from
// global memory site by site).
template <typename R, typename Src, typename Dst>
int two_pass(const LatticeView& v, const Src& src, const Dst& dst, const Coeffs<R>& c, const StepEvents* t) {
    if (!v.phi) return set_error(LB_EINVAL, "two-pass step without a phase-field buffer");
    if (v.p->model == LB_MODEL_SHAN_CHEN) return sc_step<R>(v, src, dst, c, t);
    if (t) (void)hipEventRecord(t->ev[0], v.stream);
    int rc = phase_pass<R>(v, src);
    if (rc) return rc;
    if (t) (void)hipEventRecord(t->ev[1], v.stream);
    if (tile_rows(*v.p, TILE_COLLIDE) > 0) {
        rc = zmarch<R>(v, src, dst, c, (const R*)v.phi);
    } else {
        hipLaunchKernelGGL((collide_kernel<R, Src, Dst>), dim3(grid_for(v.g.N)), dim3(kBlock), 0, v.stream, v.g, src,
                           dst, (const R*)v.phi, c);
        rc = launch_status("collide_kernel");
    }
    if (t) (void)hipEventRecord(t->ev[2], v.stream);
    return rc;
}

}  // namespace

int env_int(const char* name, int dflt) {
    const char* e = std::getenv(name);
    return (e && *e) ? std::atoi(e) : dflt;
}

namespace {
TileSetting g_tiles[4][4] = {};  // [kind][storage]
}  // namespace

TileSetting tile_setting(int kind, int storage) {
    if (kind < 0 || kind > 3 || storage < 0 || storage > 3) return TileSetting{0, 0};
    return g_tiles[kind][storage];
}
void set_tile_setting(int kind, int storage, int ty, int tz) { g_tiles[kind][storage] = TileSetting{ty, tz}; }

int tile_halo(const lb_params& p) {
    return 1 + ((p.nc_strength > 0.0 && p.model == LB_MODEL_COLOUR_GRADIENT) ? p.nc_range : 0);
}

size_t tile_lds(const lb_params& p, int kind, int TY) {
    const int H = tile_halo(p);
    const size_t phi = (size_t)(2 * H + 1) * (TY + 2 * H) * (kTX + 2 * H) * real_size(p);
    const size_t rec = (size_t)3 * (TY + 2) * (kTX + 2) * 32;
    const bool split = split_storage(p);
    switch (kind) {
        case TILE_PHASE: return rec;
        case TILE_COLLIDE: return ((phi + 15) & ~size_t(15)) + (split ? rec : 0);
        default: return lean_tile_lds(p, TY);
    }
}

// Rows asked for by lb_set_tiles or the environment (0 = none).
static int wanted_rows(const lb_params& p, int kind) {
    const int set = tile_setting(kind, p.storage).ty;
    if (set > 0) return set;
    return env_int(kind == TILE_SINGLE ? "LB_SINGLE_TY" : (kind == TILE_PHASE ? "LB_PHASE_TY" : "LB_COLLIDE_TY"), 0);
}
static int wanted_planes(const lb_params& p, int kind) {
    const int set = tile_setting(kind, p.storage).tz;
    if (set > 0) return set;
    return env_int(kind == TILE_PHASE ? "LB_PHASE_TZ" : "LB_TZ", 0);
}

static bool single_rows_fit(const lb_params& p, int ty) {
    return (ty == kSingleTY || ty == kSingleTYSmall || ty == kSingleTYLarge ||
            (ty == kSingleTYSplit && split_storage(p))) &&
           tile_lds(p, TILE_SINGLE, ty) <= (size_t)device_lds_bytes();
}

// Estimated microseconds of a one-read step with TY rows and chunks of TZ
// planes: workgroups run in rounds of as many as the 256 CUs hold at once (LDS
// and registers); a workgroup starts its rings in s + s1 w and then takes a plane in
// max(a + b w, f w) with w wavefronts per SIMD (a + b: the latency of a row that
// nothing overlaps, f: its share of issue and memory); the assembly takes 8 us,
// or 9 and 17 ns per thousand face sites.  Fitted to 360 shapes of lattices from
// 32^3 to 384^3 in each storage, of which it finds one within 7% of the best; over 14
// lattices from 32^3 to 256x256x128, near-contact ranges 0, 2, 3 and 4 and walls on
// two and three axes, its choice is 1.5% above the best on average at rest, 1 to 3%
// between moving walls, at most 34% (256^3 FP32: 757 us with 16 rows and 64 planes, 793 with 8 rows and 32, 1170
// with 16 rows and 128, half the CUs; 384^3 bf16: 2.21 ms with 12 rows and 48
// planes, 2.61 with 8 rows; 256^3 fp16: 793 us with 12 rows, 833 with 8; 128^3
// FP64: 220 us with 8 rows and 16 planes, 273 with 4; 64^3 FP32: 32 us with 2
// planes, 50 with 4).
static double single_cost(const lb_params& p, int TY, int TZ) {
    const int H = tile_halo(p);
    const bool f64 = p.storage == LB_STORE_F64, split = split_storage(p), walls = p.bc[0] || p.bc[1] || p.bc[2];
    const double s = f64 ? 3.4 : (split ? 7.9 : 5.5), s1 = f64 ? 3.3 : (split ? 0.3 : 0.6);
    const double a = f64 ? 3.4 : (split ? 1.9 : 3.1), b = f64 ? 3.2 : (split ? 1.65 : 1.0);
    const double f = f64 ? 3.0 : (split ? 1.2 : 2.4), scale = walls ? 1.2 : 1.0;
    // a SIMD holds, by registers
    const int waves = f64 || make_geom(p).moving ? 2 : (split || walls ? 3 : 4);
    const int hold =
        std::max(1, std::min((int)(kLdsBytes / tile_lds(p, TILE_SINGLE, TY)), waves * 4 / TY));
    const double tiles = double((p.nx + kTX - 1) / kTX) * ((p.ny + TY - 1) / TY);
    const int chunks = (p.nz + TZ - 1) / TZ;
    const double per_cu = std::ceil(tiles * chunks / 256.0);
    const double resident = std::min<double>(hold, per_cu);
    // (rounds beyond the second start as CUs become free)
    const double rounds = per_cu <= 2 * hold ? std::ceil(per_cu / resident) : per_cu / resident;
    const double w = 0.25 * TY * resident;
    const double tile = rounds * (s + s1 * w + TZ * scale * std::max(a + b * w, f * w));
    auto faces = [](double n, int T) { return std::min(n, 2.0 * std::ceil(n / T)); };
    const double fx = faces(p.nx, kTX) / p.nx, fy = faces(p.ny, TY) / p.ny, fz = faces(p.nz, TZ) / p.nz;
    const double sites = double(p.nx) * p.ny * p.nz * (1.0 - (1.0 - fx) * (1.0 - fy) * (1.0 - fz));
    return tile + std::max(8.0, 9.0 + sites * 1.66e-5);
}

// Rows and planes of the one-read step nothing else was asked for: the least
// estimated step over the rows that measured best somewhere (16 of FP32 unless walls
// move, 12 of 16 bits, 8 and 4 of all) and the plane counts that divide the lattice
// into equal chunks.  Some of them spill and are worth it: 16 rows of FP32 between
// walls at rest 8 to 24 B a lane (256x256x128 421 us, 489 with 8 rows; moving walls
// 220 B, 646 us against 563 with 8), 12 rows of 16 bits between moving walls 56 B
// (541 us against 564), 8 rows of FP64 there 72 to 104 B (1024 us, 1200 with 4).
static void single_auto(const lb_params& p, int ty_wanted, int tz_wanted, int& ty, int& tz) {
    const bool moving = make_geom(p).moving;
    auto offered = [&](int r) {
        if (r == kSingleTYSplit) return split_storage(p);
        return r != kSingleTYLarge || (p.storage == LB_STORE_F32 && !moving);
    };
    double best = -1.0;
    for (int r : {kSingleTY, kSingleTYSmall, kSingleTYSplit, kSingleTYLarge}) {
        if (!single_rows_fit(p, r)) continue;
        if (ty_wanted > 0 ? r != ty_wanted : !offered(r)) continue;
        for (int chunks = 1; chunks <= p.nz; chunks += chunks < 16 ? 1 : chunks / 8) {
            const int planes = tz_wanted > 0 ? std::min(tz_wanted, p.nz) : (p.nz + chunks - 1) / chunks;
            const double cost = single_cost(p, r, planes);
            if (best < 0.0 || cost < best) {
                best = cost;
                ty = r;
                tz = planes;
            }
            if (tz_wanted > 0) break;
        }
    }
}

// Tile rows: what was asked for or is preferred per kind and storage (measured
// on MI355X), else the largest that keeps the LDS rings within the budget; 0
// when none fits.
int tile_rows(const lb_params& p, int kind) {
    int want = wanted_rows(p, kind);
    if (kind == TILE_SINGLE) {
        for (int ty : {want, kSingleTY, kSingleTYSmall})
            if (single_rows_fit(p, ty)) return ty;
        return 0;
    }
    if (want <= 0) {
        // the autotuner's choices for the 256^3 emulsion on MI355X
        if (kind == TILE_PHASE) want = 4;
        else if (split_storage(p)) want = kind == TILE_COLLIDE ? 4 : 8;
        else want = p.storage == LB_STORE_F64 ? 8 : 4;
    }
    for (int ty = want; ty >= 1; ty /= 2)
        if (tile_lds(p, kind, ty) <= (size_t)max_lds_bytes()) return ty;
    return 0;
}

FusedShape tile_shape(const lb_params& p, int kind) {
    FusedShape fs;
    int tz = wanted_planes(p, kind);
    fs.TY = tile_rows(p, kind);
    if (kind == TILE_SINGLE && fs.TY > 0) {
        const int want = wanted_rows(p, kind);
        single_auto(p, single_rows_fit(p, want) ? want : 0, tz, fs.TY, tz);
    }
    fs.tiles_x = (p.nx + kTX - 1) / kTX;
    fs.tiles_y = (p.ny + fs.TY - 1) / fs.TY;
    const int tiles = fs.tiles_x * fs.tiles_y;
    // the autotuner's choices for the 256^3 emulsion on MI355X: 16-plane chunks
    // for the 16-bit phase pass and the raw-storage two-pass collide, the latter
    // shorter where that leaves less than 2048 tile rows (two-pass steps: 32^3
    // FP32 91 -> 25 us, FP64 173 -> 31; 64^3 101 -> 37, 191 -> 57; 128^3 and
    // larger take 16 planes, FP64 387 us against 404 with 8).  The Shan-Chen collide,
    // whose ring holds densities alone, takes 4 planes in FP32 and 2 in FP64: with 16,
    // 200x96x72 FP64 takes 341 us a step against 254, between moving walls FP32 266
    // against 197, 8x256x256 there 381 against 284; 128^3 FP64 388 either way
    const int most = p.model == LB_MODEL_SHAN_CHEN ? (p.storage == LB_STORE_F64 ? 2 : 4) : 16;
    if (tz <= 0 && kind == TILE_PHASE) tz = 16;
    if (tz <= 0 && kind == TILE_COLLIDE && !split_storage(p))
        tz = (int)std::min<int64_t>(most, std::max<int64_t>(1, (int64_t)p.nz * tiles * fs.TY / 2048));
    if (tz <= 0) {
        // aim for 1024 workgroups, keeping chunks a few halos deep
        const int want_chunks = std::max(1, 1024 / std::max(1, tiles));
        tz = std::max(4 * tile_halo(p), (p.nz + want_chunks - 1) / want_chunks);
    }
    fs.TZ = std::min(std::max(tz, 1), p.nz);
    fs.chunks = (p.nz + fs.TZ - 1) / fs.TZ;
    fs.nblocks = tiles * fs.chunks;
    return fs;
}

bool tile_shape_asked(const lb_params& p, int kind) { return wanted_rows(p, kind) > 0 || wanted_planes(p, kind) > 0; }

int choose_kernel(const lb_params& p) {
    const bool fits = tile_rows(p, TILE_SINGLE) > 0;
    if (p.kernel == LB_KERNEL_TWOPASS) return LB_KERNEL_TWOPASS;
    if (p.kernel == LB_KERNEL_FUSED) return fits ? LB_KERNEL_FUSED : -1;
    // automatic: the one-read step (measured faster than two passes for raw
    // and 16-bit storage); the Shan-Chen model and lattices too large for
    // 32-bit buffer offsets take two passes
    // (the one-read step's 32-bit byte offsets need 10 x raw_stride(sites) x value size < 2^32)
    const bool small =
        (uint64_t)kResArrays * real_size(p) * (uint64_t)raw_stride((size_t)p.nx * p.ny * p.nz) < ((uint64_t)1 << 32);
    if (!fits || !small || p.model != LB_MODEL_COLOUR_GRADIENT) return LB_KERNEL_TWOPASS;
    // FP64 between moving walls with the widest near-contact halo has tiles of 4 rows
    // and one wavefront per SIMD left: two passes are faster where a tenth of the lanes
    // or more lie beyond the lattice (30x100x100 82 us against 124, 201x77x59 203
    // against 226; 128^3 440 against 372), and on large lattices with an x wall too
    // (512x128x64 874 against 947; 128^3 545 against 491)
    const double lanes = double(p.nx) / (kTX * ((p.nx + kTX - 1) / kTX)), sites = double(p.nx) * p.ny * p.nz;
    if (p.storage == LB_STORE_F64 && tile_halo(p) > LB_MAX_NC_RANGE && make_geom(p).moving &&
        (lanes < 0.9 || (p.bc[0] && sites >= 1 << 22)))
        return LB_KERNEL_TWOPASS;
    return LB_KERNEL_FUSED;
}

// Source/destination storage pairs a two-pass step may combine: same storage,
// or the raw FP32 initial state of a 16-bit lattice into its moment-split
// storage.
template <typename Src, typename Dst>
struct StepPair : std::false_type {};
template <typename T, bool MW>
struct StepPair<RawPop<T, MW>, RawPop<T>> : std::true_type {};
template <typename H, bool MW>
struct StepPair<RawPop<float, MW>, SplitPop<H>> : std::true_type {};
template <typename H, bool MW>
struct StepPair<SplitPop<H, MW>, SplitPop<H>> : std::true_type {};

template <typename Dst>
int two_pass_into(const LatticeView& v, const Dst& dst, const StepEvents* t) {
    return with_state(v, [&](auto rt, auto src, const auto& c) {
        using R = decltype(rt);
        using S = decltype(src);
        if constexpr (StepPair<S, Dst>::value) return two_pass<R>(v, src, dst, c, t);
        return set_error(LB_EINVAL, "storage/compute mismatch");
    });
}

int launch_step(const LatticeView& v, int kernel, const StepEvents* t) {
    const size_t N = (size_t)v.g.N;
    if (kernel == LB_KERNEL_FUSED)
        return with_state(v, [&](auto rt, auto src, const auto&) { return single_pass<decltype(rt)>(v, src, t); });
    switch (v.p->storage) {
        case LB_STORE_F64: return two_pass_into(v, RawPop<double>{(double*)v.nxt, N}, t);
        case LB_STORE_F32: return two_pass_into(v, RawPop<float>{(float*)v.nxt, N}, t);
        case LB_STORE_F16: return two_pass_into(v, split_view<__half>(v.nxt, N, v.p->scale_log2), t);
        case LB_STORE_BF16: return two_pass_into(v, split_view<__hip_bfloat16>(v.nxt, N, v.p->scale_log2), t);
    }
    return set_error(LB_EINVAL, "unknown storage");
}

int launch_unpack(const LatticeView& v, void* f) {
    const unsigned grid = grid_for(v.g.N + kRawPad);
    const size_t N = (size_t)v.g.N;
    if (v.p->storage == LB_STORE_F64)
        hipLaunchKernelGGL(unpack_kernel<double>, dim3(grid), dim3(kBlock), 0, v.stream, v.g.N,
                           pack_view<double>(v.cur, N), (double*)f);
    else
        hipLaunchKernelGGL(unpack_kernel<float>, dim3(grid), dim3(kBlock), 0, v.stream, v.g.N,
                           pack_view<float>(v.cur, N), (float*)f);
    return launch_status("unpack_kernel");
}

int launch_clear_pads(const LatticeView& v, void* f) {
    const size_t N = (size_t)v.g.N;
    if (v.p->storage == LB_STORE_F64)
        hipLaunchKernelGGL(clear_pads_kernel<double>, dim3(1), dim3(kRawPad * Q), 0, v.stream, N, (double*)f);
    else
        hipLaunchKernelGGL(clear_pads_kernel<float>, dim3(1), dim3(kRawPad * Q), 0, v.stream, N, (float*)f);
    return launch_status("clear_pads_kernel");
}

// Initial state goes to raw storage: the current buffer for F64/F32, the
// pending FP32 buffer for 16-bit lattices.
template <typename In>
static int init_typed(const LatticeView& v, const In* rr, const In* rb, const In* u) {
    const unsigned grid = grid_for(v.g.N);
    if (v.p->storage == LB_STORE_F64) {
        hipLaunchKernelGGL((init_raw_kernel<double, In>), dim3(grid), dim3(kBlock), 0, v.stream, v.g,
                           (double*)(v.pending ? v.pending : v.cur), rr, rb, u);
    } else {
        float* dst = (float*)(v.pending ? v.pending : v.cur);
        hipLaunchKernelGGL((init_raw_kernel<float, In>), dim3(grid), dim3(kBlock), 0, v.stream, v.g, dst, rr, rb, u);
    }
    return launch_status("init_raw_kernel");
}

int launch_init(const LatticeView& v, const void* rr, const void* rb, const void* u, int dtype) {
    if (dtype == LB_DTYPE_F64) return init_typed<double>(v, (const double*)rr, (const double*)rb, (const double*)u);
    return init_typed<float>(v, (const float*)rr, (const float*)rb, (const float*)u);
}

template <typename In>
static int import_typed(const LatticeView& v, const In* f) {
    const unsigned grid = grid_for(v.g.N);
    if (v.p->storage == LB_STORE_F64) {
        hipLaunchKernelGGL((import_raw_kernel<double, In>), dim3(grid), dim3(kBlock), 0, v.stream, v.g,
                           (double*)(v.pending ? v.pending : v.cur), f);
    } else {
        float* dst = (float*)(v.pending ? v.pending : v.cur);
        hipLaunchKernelGGL((import_raw_kernel<float, In>), dim3(grid), dim3(kBlock), 0, v.stream, v.g, dst, f);
    }
    return launch_status("import_raw_kernel");
}

int launch_import(const LatticeView& v, const void* f, int dtype) {
    if (dtype == LB_DTYPE_F64) return import_typed<double>(v, (const double*)f);
    return import_typed<float>(v, (const float*)f);
}

int launch_export(const LatticeView& v, void* out, int dtype) {
    bool taken = false;
    const int rc = pull_export(v, out, dtype, taken);
    if (rc || taken) return rc;
    const unsigned grid = grid_for(v.g.N);
    return with_state(v, [&](auto rt, auto src, const auto&) {
        using R = decltype(rt);
        using S = decltype(src);
        if (dtype == LB_DTYPE_F64)
            hipLaunchKernelGGL((export_kernel<R, S, double>), dim3(grid), dim3(kBlock), 0, v.stream, v.g, src, (double*)out);
        else
            hipLaunchKernelGGL((export_kernel<R, S, float>), dim3(grid), dim3(kBlock), 0, v.stream, v.g, src, (float*)out);
        return launch_status("export_kernel");
    });
}

int launch_moments(const LatticeView& v, void* rr, void* rb, void* j, int dtype) {
    bool taken = false;
    const int rc = pull_moments(v, rr, rb, j, dtype, taken);
    if (rc || taken) return rc;
    const unsigned grid = grid_for(v.g.N);
    return with_state(v, [&](auto rt, auto src, const auto&) {
        using R = decltype(rt);
        using S = decltype(src);
        if (dtype == LB_DTYPE_F64)
            hipLaunchKernelGGL((moments_kernel<R, S, double>), dim3(grid), dim3(kBlock), 0, v.stream, v.g, src,
                               (double*)rr, (double*)rb, (double*)j);
        else
            hipLaunchKernelGGL((moments_kernel<R, S, float>), dim3(grid), dim3(kBlock), 0, v.stream, v.g, src,
                               (float*)rr, (float*)rb, (float*)j);
        return launch_status("moments_kernel");
    });
}

int launch_korteweg(const LatticeView& v, double lam, int b, void* kout, void* pout, int dtype, int accumulate) {
    return with_state(v, [&](auto rt, auto src, const auto&) {
        using R = decltype(rt);
        using S = decltype(src);
        // phase field of the current state, as the next collision sees it: a
        // one-read state completes the field its phase-sum buffer holds (the
        // next step repeats that, with the same result); otherwise a phase
        // pass writes it into the scratch field
        const R* field = (const R*)v.phi;
        int rc;
        if (v.part_valid && v.part_in) {
            const FusedShape fs = v.shape;
            rc = with_rows(fs.TY, [&](auto ty) { return assemble_phase<R, S, decltype(ty)::value>(v, src, fs); });
            field = phi_of<kTX>((Part2<R>*)v.part_in, v.g);
        } else {
            rc = phase_pass<R>(v, src);
        }
        if (rc) return rc;
        const dim3 grid((unsigned)(((v.g.nx + 63) / 64) * ((v.g.ny + kKortewegRows - 1) / kKortewegRows) *
                                   ((v.g.nz + kKortewegChunk - 1) / kKortewegChunk)));
        const dim3 block(64 * kKortewegRows);
        if (dtype == LB_DTYPE_F64)
            hipLaunchKernelGGL((korteweg_kernel<R, double>), grid, block, 0, v.stream, v.g, field, R(lam),
                               b, (double*)kout, (double*)pout, accumulate);
        else
            hipLaunchKernelGGL((korteweg_kernel<R, float>), grid, block, 0, v.stream, v.g, field, R(lam),
                               b, (float*)kout, (float*)pout, accumulate);
        return launch_status("korteweg_kernel");
    });
}

int launch_droplets(hipStream_t st, const Geom& g, const double* cen, const double* rad, int n, double width,
                    double background, double rho0, double* rr, double* rb) {
    hipLaunchKernelGGL(droplet_fields_kernel, dim3(grid_for(g.N)), dim3(kBlock), 0, st, g, cen, rad, n, width,
                       background, rho0, rr, rb);
    return launch_status("droplet_fields_kernel");
}

int launch_totals(const LatticeView& v, Neu* partial, double* dtot) {
    const bool pack = v.packed && !v.pending;
    const int fill = v.p->storage == LB_STORE_F64 ? 512 : (v.g.moving ? 768 : kPackTotalsBlocks);
    int grid = std::min<int>(pack ? fill : kTotalsBlocks, (int)grid_for(v.g.N));
    bool taken = false;
    int rc = pull_totals(v, partial, grid, taken);
    if (!rc && !taken) rc = with_state(v, [&](auto rt, auto src, const auto&) {
        using R = decltype(rt);
        using S = decltype(src);
        hipLaunchKernelGGL((totals_kernel<R, S>), dim3(grid), dim3(kBlock), 0, v.stream, v.g, src, partial);
        return launch_status("totals_kernel");
    });
    if (rc) return rc;
    hipLaunchKernelGGL(totals_final_kernel, dim3(1), dim3(kBlock), 0, v.stream, partial, grid, dtot);
    return launch_status("totals_final_kernel");
}

}  // namespace lbm
