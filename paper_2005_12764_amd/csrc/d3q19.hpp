// d3q19.hpp -- device-side lattice tables and the local colour-gradient
// collision for gfx950.  Device code only; every loop over directions is
// fully unrolled so the lattice vectors and weights fold into immediates.
//
// Method (arXiv 2005.12764):
//   equilibrium w_i rho (1 + u_i + q_i)                     Sec. 2, eq:equil
//   BGK with mixture rate w_eff and harmonic nu_bar          Sec. 2.1, eq:twobgk
//   exact-difference source f^eq(u + F/rho) - f^eq(u)        Sec. 2.1, eq:edm
//   near-contact force F_rep = -A_h[h] n delta_I             Sec. 4
// plus the colour-gradient perturbation (Reis-Phillips, D3Q19 coefficients
// of Liu-Valocchi-Kang) and Latva-Kokko-Rothman recolouring, which the paper
// uses but does not write out.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbm {

constexpr int Q = 19;

// Direction order: rest, +x,-x,+y,-y,+z,-z, then the 12 face diagonals in
// opposite pairs.  This order is part of the library's state layout.
struct Lattice {
    static constexpr int cx[Q] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
    static constexpr int cy[Q] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
    static constexpr int cz[Q] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
    static constexpr int opp[Q] = {0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17};
    static constexpr int len2(int i) { return cx[i] * cx[i] + cy[i] * cy[i] + cz[i] * cz[i]; }
};

template <typename R>
__host__ __device__ constexpr R weight(int i) {
    return Lattice::len2(i) == 0 ? R(1) / R(3) : (Lattice::len2(i) == 1 ? R(1) / R(18) : R(1) / R(36));
}
// 1/|c_i| (0 for the rest vector, whose recolouring term vanishes).
template <typename R>
__host__ __device__ constexpr R inv_clen(int i) {
    return Lattice::len2(i) == 0 ? R(0)
                                 : (Lattice::len2(i) == 1 ? R(1) : R(0.70710678118654752440084436210485));
}

// Per-lattice constants in the compute type, prepared on the host.
template <typename R>
struct Coeffs {
    R inv_nu_r, inv_nu_b;  // 1 / nu_k, nu_k = (tau_k - 1/2)/3
    R omega;               // the mixture rate when tau_r == tau_b (then 1/tau at every site)
    R half_A;              // A/2 of the perturbation
    R beta;
    R eps_g, eps_g2;       // |G| at or below which n = 0, and its square
    R g_iface, g_iface2;   // interface threshold of the near-contact probe, and its square
    R nc_strength, nc_hmin;
    R fx, fy, fz;          // body force density
    int nc_range;          // 0 = near-contact off
    int same_tau;          // tau_r == tau_b: omega above holds everywhere
    int model;             // 0 colour gradient, 1 Shan-Chen
    R g_sc;                // Shan-Chen coupling G_C
};

// c_i . a for a lattice velocity c_i (components -1, 0, 1): the sum of the
// non-zero components' terms only (a product by a zero component is not
// dropped by the compiler, since 0 * a is not 0 for every float a).
template <typename R>
__device__ __forceinline__ R cdot3(int i, R ax, R ay, R az) {
    using L = Lattice;
    R v = R(0);
    bool any = false;
    if (L::cx[i]) { v = L::cx[i] > 0 ? ax : -ax; any = true; }
    if (L::cy[i]) { const R b = L::cy[i] > 0 ? ay : -ay; v = any ? v + b : b; any = true; }
    if (L::cz[i]) { const R b = L::cz[i] > 0 ? az : -az; v = any ? v + b : b; }
    return v;
}

// Reciprocal and reciprocal square root.  FP32: the hardware estimates
// (v_rcp_f32, v_rsq_f32, within 1 ulp), used where an FP32 result only feeds
// further rounding-level arithmetic; FP64: correctly rounded.
__device__ __forceinline__ float rcp_of(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_of(double x) { return 1.0 / x; }
__device__ __forceinline__ float rsq_of(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq_of(double x) { return 1.0 / sqrt(x); }

__device__ __forceinline__ float fma_of(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_of(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename R>
__device__ __forceinline__ R dot3(R ax, R ay, R az, R bx, R by, R bz) {
#pragma clang fp contract(off)
    return fma_of(az, bz, fma_of(ay, by, ax * bx));
}

// Is |G| (G with squared length g2) above the threshold e (squared e2)?
// FP32 compares squares; FP64 compares the root, as the definition reads.
__device__ __forceinline__ bool above(float g2, float e, float e2) { (void)e; return g2 > e2; }
__device__ __forceinline__ bool above(double g2, double e, double e2) { (void)e2; return sqrt(g2) > e; }
__device__ __forceinline__ bool at_least(float g2, float e, float e2) { (void)e; return g2 >= e2; }
__device__ __forceinline__ bool at_least(double g2, double e, double e2) { (void)e2; return sqrt(g2) >= e; }
// 1/|G| for a G known to be non-zero.
__device__ __forceinline__ float inv_norm(float g2) { return rsq_of(g2); }
__device__ __forceinline__ double inv_norm(double g2) { return 1.0 / sqrt(g2); }

// Outputs of one site's collision that the 16-bit storage keeps per site.
template <typename R>
struct SiteTotals {
    R drho;                // post-collision density - 1
    R jx, jy, jz;          // 3 (j + F) = 3 rho v: the linear term of the equilibrium
    R phi;                 // phase x_r - x_b
    R vx, vy, vz;          // recolouring vector beta (rho_r rho_b/rho) G/|G|
};

// Local collision of one site, in shifted variables: t_i = f^r_i + f^b_i - w_i
// (the total's deviation from the rest equilibrium at unit density) and
// d_i = f^r_i - f^b_i (the colour difference).  Carrying the small t_i keeps
// FP32 rounding relative to the deviations that hold the flow, not to the
// O(w_i) populations (a per-step force increment is ~1e-7 of those).
// t (and d) hold the pulled (post-streaming) values on entry and the
// post-collision, recoloured values on exit.  (gx,gy,gz) is the colour gradient
// at the site, (Fx,Fy,Fz) the total force.
//
// Equilibrium, source and perturbation are all w_i times a polynomial of second
// degree in c_i, so they are summed once per site as
//   w_i (a + c.b + c.M c),   b = 3 (w j + F),
//   M = 4.5 rho (v v - (1 - w) u u) + (A/2)|G| n n,   v = u + F/rho,
//   a = w drho - 1.5 rho (|v|^2 - (1 - w)|u|^2) -+ (A/2)|G|
// (u u of the equilibrium and u du + du u + du du of the source together are
// v v - (1 - w) u u; -B_i is -w_i for the moving directions and +w_0 at rest),
// and each direction then costs (1 - w) t_i + w_i (even +- odd part).  The
// linear term of the force enters through F itself, not through a difference
// of equilibria.  Fused multiply-adds are written out and the compiler forms
// none itself: a sum of two products can be fused either way, and every kernel
// that collides a site (single tiles, batch tiles) has to round alike.
//
// Sums of a site's pulled values that the collision needs, each in ascending
// direction.  rc = sum_i (w_i + t_i) is rounded term by term as dif = sum_i d_i
// is: a pure component (d_i = +-(w_i + t_i)) then gives phi = dif/rc = +-1 and
// x_r, x_b = 1, 0 exactly, and stays pure.
template <typename R>
struct SiteSums {
    R drho = R(0), dif = R(0), rc = R(0), jx = R(0), jy = R(0), jz = R(0);
    // direction i: t_i, w_i + t_i, d_i
    __device__ __forceinline__ void add(int i, R t, R wt, R d) {
        using L = Lattice;
        drho += t;
        dif += d;
        rc += wt;
        if (L::cx[i]) jx += L::cx[i] > 0 ? t : -t;
        if (L::cy[i]) jy += L::cy[i] > 0 ? t : -t;
        if (L::cz[i]) jz += L::cz[i] > 0 ? t : -t;
    }
};

// t_i becomes the post-collision total of direction i; the recoloured colour
// differences follow from it and the phase and recolouring vector left in tot
// (recoloured()).
template <typename R>
__device__ __forceinline__ void collide_totals(R (&t)[Q], const SiteSums<R>& m, R gx, R gy, R gz, R Fx, R Fy, R Fz,
                                               const Coeffs<R>& c, SiteTotals<R>& tot) {
#pragma clang fp contract(off)
    using L = Lattice;
    const R drho = m.drho, rc = m.rc, jx = m.jx, jy = m.jy, jz = m.jz;
    const R rho = R(1) + drho;            // sum of the weights is 1
    const R phi = m.dif / rc;             // x_r - x_b (a divided, not multiplied, quotient)
    const R xr = fma_of(R(0.5), phi, R(0.5)), xb = fma_of(R(-0.5), phi, R(0.5));
    const R inv_rho = rcp_of(rho);
    const R ux = jx * inv_rho, uy = jy * inv_rho, uz = jz * inv_rho;
    // v = u + du, the exact-difference velocity shift du = F^k/rho_k with
    // F^k = (rho_k/rho) F; rho v = j + F
    const R px = jx + Fx, py = jy + Fy, pz = jz + Fz;
    const R vx = px * inv_rho, vy = py * inv_rho, vz = pz * inv_rho;
    // mixture relaxation: 1/nu_bar = x_r/nu_r + x_b/nu_b, w = 2 cs2/(2 nu_bar + cs2)
    R omega = c.omega;
    if (!c.same_tau) {
        const R nubar = rcp_of(fma_of(xb, c.inv_nu_b, xr * c.inv_nu_r));
        omega = R(2) * rcp_of(fma_of(R(6), nubar, R(1)));
    }
    const R om1 = R(1) - omega;

    const R g2 = dot3(gx, gy, gz, gx, gy, gz);
    const bool has_n = above(g2, c.eps_g, c.eps_g2);
    const R inv_gm = has_n ? inv_norm(g2) : R(0);
    const R gm = g2 * inv_gm;
    // perturbation amplitude (A/2)|G| and recolouring strength
    // beta rho_r rho_b / rho = beta x_r x_b rc
    const R pa = c.half_A * gm;
    const R seg = has_n ? c.beta * xr * xb * rc : R(0);
    const R nx = gx * inv_gm, ny = gy * inv_gm, nz = gz * inv_gm;

    // T = rho (v v - (1 - w) u u)
    const R kx = om1 * jx, ky = om1 * jy, kz = om1 * jz;
    const R Txx = fma_of(px, vx, -(kx * ux)), Tyy = fma_of(py, vy, -(ky * uy)), Tzz = fma_of(pz, vz, -(kz * uz));
    const R Txy = fma_of(px, vy, -(kx * uy)), Txz = fma_of(px, vz, -(kx * uz)), Tyz = fma_of(py, vz, -(ky * uz));
    constexpr R w0 = weight<R>(0), w1 = weight<R>(1), w2 = weight<R>(7);
    const R a = fma_of(omega, drho, R(-1.5) * ((Txx + Tyy) + Tzz));
    // times the weight of a diagonal direction (the axis weight is twice it)
    const R pw = w2 * pa;
    const R qx = pw * nx, qy = pw * ny, qz = pw * nz;
    constexpr R k45 = R(4.5) * w2, k9 = R(9) * w2;
    const R mxx = fma_of(qx, nx, k45 * Txx), myy = fma_of(qy, ny, k45 * Tyy), mzz = fma_of(qz, nz, k45 * Tzz);
    const R hx = R(2) * qx, hy = R(2) * qy;
    const R mxy = fma_of(hx, ny, k9 * Txy), mxz = fma_of(hx, nz, k9 * Txz), myz = fma_of(hy, nz, k9 * Tyz);
    constexpr R k3 = R(3) * w2;
    const R bx = k3 * fma_of(omega, jx, Fx), by = k3 * fma_of(omega, jy, Fy), bz = k3 * fma_of(omega, jz, Fz);
    const R a2 = fma_of(w2, a, -pw);
    t[0] = fma_of(om1, t[0], w0 * (a + pa));
    auto pair = [&](int i, R even, R odd) {
        const int o = L::opp[i];
        t[i] = fma_of(om1, t[i], even + odd);
        t[o] = fma_of(om1, t[o], even - odd);
    };
    pair(1, R(2) * (a2 + mxx), R(2) * bx);
    pair(3, R(2) * (a2 + myy), R(2) * by);
    pair(5, R(2) * (a2 + mzz), R(2) * bz);
    const R exy = a2 + (mxx + myy), exz = a2 + (mxx + mzz), eyz = a2 + (myy + mzz);
    pair(7, exy + mxy, bx + by);
    pair(9, exy - mxy, bx - by);
    pair(11, exz + mxz, bx + bz);
    pair(13, exz - mxz, bx - bz);
    pair(15, eyz + myz, by + bz);
    pair(17, eyz - myz, by - bz);
    tot.drho = drho;
    tot.jx = R(3) * px;  // 3 rho v = 3 (j + F)
    tot.jy = R(3) * py;
    tot.jz = R(3) * pz;
    tot.phi = phi;
    tot.vx = seg * nx;
    tot.vy = seg * ny;
    tot.vz = seg * nz;
}

// Recolouring f^r = x_r f* + rec, f^b = x_b f* - rec, f* = w_i + t*_i, rec =
// w_i (c_i . v)/|c_i|: the colour difference d_i = phi f* + 2 rec of a direction
// from wt = w_i + t*_i and the site's phase and recolouring vector, which are
// kept as s = 2 w_7 v/|c_7| so that the twelve diagonal directions need no
// factor.
template <typename R>
struct Colour {
    R phi, sx, sy, sz;
};
template <typename R>
__device__ __forceinline__ Colour<R> colour_of(const SiteTotals<R>& tot) {
#pragma clang fp contract(off)
    constexpr R k = R(2) * weight<R>(7) * inv_clen<R>(7);
    return Colour<R>{tot.phi, k * tot.vx, k * tot.vy, k * tot.vz};
}
template <typename R>
__device__ __forceinline__ R recoloured(int i, R wt, const Colour<R>& q) {
#pragma clang fp contract(off)
    if (i == 0) return q.phi * wt;
    const R cs = cdot3<R>(i, q.sx, q.sy, q.sz);
    constexpr R k = weight<R>(1) / (weight<R>(7) * inv_clen<R>(7));
    return fma_of(q.phi, wt, Lattice::len2(i) == 1 ? k * cs : cs);
}

// The collision with the colour differences held per direction.
template <typename R>
__device__ __forceinline__ void collide(R (&t)[Q], R (&d)[Q], R gx, R gy, R gz, R Fx, R Fy, R Fz,
                                        const Coeffs<R>& c, SiteTotals<R>* tot) {
    SiteSums<R> m;
#pragma unroll
    for (int i = 0; i < Q; ++i) m.add(i, t[i], weight<R>(i) + t[i], d[i]);
    collide_totals<R>(t, m, gx, gy, gz, Fx, Fy, Fz, c, *tot);
    const Colour<R> q = colour_of(*tot);
#pragma unroll
    for (int i = 0; i < Q; ++i) d[i] = recoloured<R>(i, weight<R>(i) + t[i], q);
}

// Local collision of one site in the Shan-Chen model (Sec. 2.1: the
// inter-component force of eq. shanchen_force entering each component's
// exact-difference source, eq:edm), in the shifted variables of collide().
// (bx,by,bz) = sum_i w_i rho_b(x + c_i) c_i and (rx,ry,rz) the same of rho_r.
// Component k gets the velocity shift du_k = F^k/rho_k with
// F^k = -G_C rho_k sum_i w_i rho_k'(x + c_i) c_i + (rho_k/rho) F_body, i.e.
// du_k = -G_C (that sum) + F_body/rho, with no division by rho_k; both relax
// with the mixture rate toward f^eq(rho_k, u), u = j/rho.  No perturbation
// and no recolouring: the force alone keeps the components apart.
template <typename R>
__device__ __forceinline__ void collide_sc(R (&t)[Q], R (&d)[Q], R bx, R by, R bz, R rx, R ry, R rz,
                                           const Coeffs<R>& c) {
    using L = Lattice;
    R drho = R(0), dif = R(0), rc = R(0), jx = R(0), jy = R(0), jz = R(0);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        drho += t[i];
        dif += d[i];
        rc += weight<R>(i) + t[i];
        if (L::cx[i]) jx += L::cx[i] > 0 ? t[i] : -t[i];
        if (L::cy[i]) jy += L::cy[i] > 0 ? t[i] : -t[i];
        if (L::cz[i]) jz += L::cz[i] > 0 ? t[i] : -t[i];
    }
    const R rho = R(1) + drho;
    const R rr = R(0.5) * (rc + dif), rb = R(0.5) * (rc - dif);
    const R inv_rho = R(1) / rho;
    const R ux = jx * inv_rho, uy = jy * inv_rho, uz = jz * inv_rho;
    const R fx = c.fx * inv_rho, fy = c.fy * inv_rho, fz = c.fz * inv_rho;
    // velocity shifts of the red (R) and blue (B) components
    const R Rx = fx - c.g_sc * bx, Ry = fy - c.g_sc * by, Rz = fz - c.g_sc * bz;
    const R Bx = fx - c.g_sc * rx, By = fy - c.g_sc * ry, Bz = fz - c.g_sc * rz;
    // s_k = u + (u + du_k): f^eq(rho_k, u + du_k) - f^eq(rho_k, u)
    //   = rho_k w_i [3 c.du_k + 4.5 (c.du_k)(c.s_k) - 1.5 du_k.s_k]
    const R sRx = R(2) * ux + Rx, sRy = R(2) * uy + Ry, sRz = R(2) * uz + Rz;
    const R sBx = R(2) * ux + Bx, sBy = R(2) * uy + By, sBz = R(2) * uz + Bz;
    const R dsR = Rx * sRx + Ry * sRy + Rz * sRz;
    const R dsB = Bx * sBx + By * sBy + Bz * sBz;
    R omega = c.omega;
    if (!c.same_tau) {
        const R phi = dif / rc;
        const R xr = R(0.5) + R(0.5) * phi, xb = R(0.5) - R(0.5) * phi;
        const R nubar = R(1) / (xr * c.inv_nu_r + xb * c.inv_nu_b);
        omega = R(2) / (R(6) * nubar + R(1));
    }
    const R uu = ux * ux + uy * uy + uz * uz;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const R w = weight<R>(i);
        const R cu = cdot3<R>(i, ux, uy, uz);
        const R q = R(3) * cu + R(4.5) * cu * cu - R(1.5) * uu;
        const R teq = w * (drho + rho * q);          // f^eq(rho_r) + f^eq(rho_b) - w
        const R deq = w * dif * (R(1) + q);          // f^eq(rho_r) - f^eq(rho_b)
        const R cdR = cdot3<R>(i, Rx, Ry, Rz);
        const R csR = cdot3<R>(i, sRx, sRy, sRz);
        const R cdB = cdot3<R>(i, Bx, By, Bz);
        const R csB = cdot3<R>(i, sBx, sBy, sBz);
        const R SR = rr * w * (R(3) * cdR + R(4.5) * cdR * csR - R(1.5) * dsR);
        const R SB = rb * w * (R(3) * cdB + R(4.5) * cdB * csB - R(1.5) * dsB);
        t[i] = t[i] - omega * (t[i] - teq) + (SR + SB);
        d[i] = d[i] - omega * (d[i] - deq) + (SR - SB);
    }
}

// The two components from the shifted variables.
template <typename R>
__device__ __forceinline__ void from_shifted(int i, R t, R d, R& fr, R& fb) {
    const R f = weight<R>(i) + t;
    fr = R(0.5) * (f + d);
    fb = R(0.5) * (f - d);
}

// G = 3 sum_i w_i phi_i c_i from the 18 neighbour values, phi(i) the value at
// x + c_i: differences of opposite neighbours, the diagonal ones added before
// their weight (a uniform field gives exactly zero).
template <typename R, typename Phi>
__device__ __forceinline__ void stencil_gradient(const Phi& phi, R& gx, R& gy, R& gz) {
#pragma clang fp contract(off)
    using L = Lattice;
    R e[Q];
#pragma unroll
    for (int i = 1; i < Q; i += 2) e[i] = phi(i) - phi(L::opp[i]);
    // (the axis weight is twice the diagonal one)
    constexpr R k = R(3) * weight<R>(7);
    gx = k * fma_of(R(2), e[1], (e[7] + e[9]) + (e[11] + e[13]));
    gy = k * fma_of(R(2), e[3], (e[7] - e[9]) + (e[15] + e[17]));
    gz = k * fma_of(R(2), e[5], (e[11] - e[13]) + (e[15] - e[17]));
}

// Near-contact amplitude A_h(h): full strength up to h_min, h^-3 beyond,
// zero outside 1..K.
template <typename R>
__device__ __forceinline__ R nc_amplitude(int h, const Coeffs<R>& c) {
    if (h < 1 || h > c.nc_range) return R(0);
    if (R(h) <= c.nc_hmin) return c.nc_strength;
    const R r = c.nc_hmin / R(h);
    return c.nc_strength * r * r * r;
}

}  // namespace lbm
