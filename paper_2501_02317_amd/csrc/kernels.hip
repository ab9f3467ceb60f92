// Device kernels of the Godunov hydro step for gfx950 (CDNA4, wave64).
//
// Method (Wang, arXiv 2501.02317, Sec. 3): conserved -> primitive in FP64
// (Sec. 3.1), ghost cells from the boundary rules of Sec. 3.1.1 resolved at
// load time, PLM with minmod on primitive variables (eq. minmod), HLLC with
// the subtraction-safe wave speeds (eqs. hllc-contact-spd, hllc-mixed-dvel),
// flux-divergence update and Heun combine in FP64 (Sec. 3.3), CFL dt
// reduction (Sec. 3.1).
//
// Layout: SoA FP64 U[c][k][j][i], interior only.  The stage kernel is a
// 2.5-D sweep: a work-group owns a TX x TY tile of the (kernel) x-y plane and
// marches along the kernel z axis over a chunk of kz planes.  The z stencil
// (five planes of primitive variables) lives in registers, the in-plane
// stencil in an LDS plane with a two-cell halo.  Every face flux is computed
// once per work-group and is one value shared by both neighbouring cells.
//
// Floating point: the compiler contracts nothing on its own (contraction is
// off), but the code fuses by hand where it pays -- explicit fused
// multiply-adds, FP64 reciprocals and reciprocal square roots from the
// hardware estimates refined by Newton steps (two, about 1 ulp, in the
// conversions and the time step; one, about 2^-45 relative, in the HLLC
// solve), and algebraically equal rearrangements of the written formulas.
// The FP64 path therefore agrees with a plain serial evaluation of the same
// formulas to rounding, not bitwise.
#include <hip/hip_runtime.h>

#include <type_traits>

#include <cfloat>
#include <cmath>

#include "hydro_internal.h"

// The part of this file that a translation unit compiles: 0 everything but
// the stage kernels, 1 .. 6 the stage kernels of one dimensionality and
// precision (see the dispatch below).
#ifndef HYDRO_PART
#define HYDRO_PART 0
#endif

#pragma clang fp contract(off)

namespace hydro {
namespace {

enum { BC_PERIODIC = 0, BC_FREE = 1, BC_OUTFLOW = 2, BC_REFLECT = 3 };
enum { VM_NONE = 0, VM_NEG = 1, VM_CLIP_LO = 2, VM_CLIP_HI = 3 };


__device__ __forceinline__ double dabs(double x) { return __builtin_fabs(x); }
__device__ __forceinline__ float dabs(float x) { return __builtin_fabsf(x); }

// Velocity component (index into W/U) along kernel axis ax.
template <int NDIM>
__device__ __forceinline__ constexpr int vcomp(int ax) {
    return ax == 0 ? 1 : (ax == 1 ? 2 : NDIM);
}

// Arithmetic policy.  FP32 (the mixed path's reconstruction and Riemann
// solve): the hardware reciprocal and reciprocal square root (1 ulp), which
// the FP32 tolerance of that path absorbs.  FP64: the hardware estimates
// (relative error up to about 2^-23) refined by Newton steps instead of the
// longer correctly rounded division and square-root sequences -- two steps
// (about 1 ulp) for the conversions and the time step, one step (relative
// error about 2^-45) for the six per HLLC face (rcp1, rsq1), well inside the
// 1e-12 agreement the FP64 path keeps with a plain evaluation.
template <typename R>
struct Ops;

template <>
struct Ops<double> {
    static __device__ __forceinline__ double fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
    static __device__ __forceinline__ double rcp(double x) {
        double r = __builtin_amdgcn_rcp(x);
        double e = __builtin_fma(-x, r, 1.0);
        r = __builtin_fma(r, e, r);
        e = __builtin_fma(-x, r, 1.0);
        return __builtin_fma(r, e, r);
    }
    static __device__ __forceinline__ double rsq(double x) {
        double y = __builtin_amdgcn_rsq(x);
        double e = __builtin_fma(-x * y, y, 1.0);
        y = __builtin_fma(0.5 * y, e, y);
        e = __builtin_fma(-x * y, y, 1.0);
        return __builtin_fma(0.5 * y, e, y);
    }
    static __device__ __forceinline__ double rcp1(double x) {
        const double r = __builtin_amdgcn_rcp(x);
        return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    }
    static __device__ __forceinline__ double rsq1(double x) {
        const double y = __builtin_amdgcn_rsq(x);
        return __builtin_fma(0.5 * y, __builtin_fma(-x * y, y, 1.0), y);
    }
    static __device__ __forceinline__ double max0(double x) { return __builtin_fmax(x, 0.0); }
    // median of (a, b, 0): the minmod of eq. minmod
    static __device__ __forceinline__ double minmod(double a, double b) {
        return __builtin_fmax(__builtin_fmin(a, b), __builtin_fmin(__builtin_fmax(a, b), 0.0));
    }
    // The slopes of the two cells beside a face, minmod(a, m) and
    // minmod(m, b), with m the difference across the face: the median of
    // (x, m, 0) is x clamped to [min(m, 0), max(m, 0)], and the two bounds
    // serve both slopes (FP64 min and max issue at half rate).
    static __device__ __forceinline__ void minmod2(double a, double m, double b, double& sa, double& sb) {
        const double lo = __builtin_fmin(m, 0.0), hi = __builtin_fmax(m, 0.0);
        sa = __builtin_fmin(__builtin_fmax(a, lo), hi);
        sb = __builtin_fmin(__builtin_fmax(b, lo), hi);
    }
};

template <>
struct Ops<float> {
    static __device__ __forceinline__ float fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
    static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
    static __device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
    static __device__ __forceinline__ float rcp1(float x) { return __builtin_amdgcn_rcpf(x); }
    static __device__ __forceinline__ float rsq1(float x) { return __builtin_amdgcn_rsqf(x); }
    static __device__ __forceinline__ float max0(float x) { return __builtin_fmaxf(x, 0.0f); }
    static __device__ __forceinline__ float minmod(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }
    static __device__ __forceinline__ void minmod2(float a, float m, float b, float& sa, float& sb) {
        sa = __builtin_amdgcn_fmed3f(a, m, 0.0f);
        sb = __builtin_amdgcn_fmed3f(m, b, 0.0f);
    }
};

// Gas constants in the compute precision.
template <typename R>
struct Gas {
    R g;          // gamma
    R z;          // (gamma + 1) / (2 gamma)
    R inv_gm1;    // 1 / (gamma - 1)
    R inv_g_gm1;  // 1 / (gamma (gamma - 1))
};

template <typename R>
__device__ __forceinline__ Gas<R> make_gas(double g) {
    Gas<R> o;
    o.g = (R)g;
    o.z = (R)((g + 1.0) / (2.0 * g));
    o.inv_gm1 = (R)(1.0 / (g - 1.0));
    o.inv_g_gm1 = (R)(1.0 / (g * (g - 1.0)));
    return o;
}

// ----------------------------------------------------------------- physics

// eq. minmod: the slope of smaller magnitude when both have the same strict
// sign, else zero -- which is the median of (a, b, 0).
template <typename R>
__device__ __forceinline__ R minmod(R a, R b) {
    return Ops<R>::minmod(a, b);
}

// Conserved -> primitive in FP64 (Sec. 3.1): r = 1/rho, v_d = m_d r,
// p = (gamma - 1)(E - (1/2) r sum_d m_d^2); returns admissibility.  The
// squares are rounded separately and summed in axis order, so interchanging
// x and y leaves the result bitwise unchanged.  LOWP: the values are rounded
// to FP32 afterwards, so 1/rho takes one Newton step instead of two.
// Admissibility is rho and p positive and finite: a non-finite momentum or
// energy makes p NaN or infinite, so it needs no test of its own.
template <int NDIM, bool LOWP = false>
__device__ __forceinline__ bool cons_to_prim(double gm1, const double (&u)[NDIM + 2],
                                             double (&w)[NDIM + 2]) {
    const double rho = u[0];
    const double r = LOWP ? Ops<double>::rcp1(rho) : Ops<double>::rcp(rho);
    double msq = 0.0;
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        w[1 + d] = u[1 + d] * r;
        msq = msq + u[1 + d] * u[1 + d];
    }
    const double p = gm1 * __builtin_fma(-0.5 * r, msq, u[NDIM + 1]);
    w[0] = rho;
    w[NDIM + 1] = p;
    return rho > 0.0 && rho < __builtin_inf() && p > 0.0 && p < __builtin_inf();
}

// HLLC flux in the face-normal frame, W = (rho, u, t_1..t_NT, p).
//   c_K = sqrt(g p_K / rho_K), evaluated as (g p_K) / sqrt(g p_K rho_K);
//   p* = max(0, primitive-variable guess);
//   ds_L = -c_L q_L, ds_R = c_R q_R with q_K = sqrt(1 + z (max(p*/p_K, 1) - 1))
//   (eq. hllc-mixed-dvel), evaluated as c_K q_K = a_K / sqrt(a_K rho_K) with
//   a_K = g (p_K + z max(p* - p_K, 0)), so ds_K = c_K exactly when p* <= p_K;
//   s_* from the bracketed form of eq. hllc-contact-spd.  Only the selected
//   side's star state and flux are evaluated; E_K/rho_K = c_K^2/(g (g-1)) +
//   |v_K|^2 / 2 and one reciprocal of (s_K - s_*) rho_K ds_K serve the star
//   state, so a face costs six reciprocal(-square-root) evaluations; the
//   tangential fluxes are the mass flux times the upwind side's tangential
//   velocities (the star state carries them unchanged).
template <typename R, int NT>
__device__ __forceinline__ void hllc(const Gas<R>& gas, const R (&WL)[NT + 3], const R (&WR)[NT + 3],
                                     R (&F)[NT + 3]) {
    using O = Ops<R>;
    constexpr int NC = NT + 3;
    const R g = gas.g;
    const R rl = WL[0], ul = WL[1], pl = WL[NC - 1];
    const R rr = WR[0], ur = WR[1], pr = WR[NC - 1];
    const R gpl = g * pl, gpr = g * pr;
    const R cl = gpl * O::rsq1(gpl * rl);
    const R cr = gpr * O::rsq1(gpr * rr);
    const R ppv = R(0.5) * (pl + pr) - R(0.125) * (ur - ul) * (rl + rr) * (cl + cr);
    const R ps = O::max0(ppv);
    const R al = g * O::fma(gas.z, O::max0(ps - pl), pl);
    const R ar = g * O::fma(gas.z, O::max0(ps - pr), pr);
    const R dsl = -(al * O::rsq1(al * rl));
    const R dsr = ar * O::rsq1(ar * rr);
    const R sl = ul + dsl;
    const R sr = ur + dsr;
    const R ml = rl * dsl, mr = rr * dsr;  // rho_K ds_K
    const R ss = (O::fma(-mr, ur, pr) - O::fma(-ml, ul, pl)) * O::rcp1(ml - mr);

    // s_L >= 0: F_L ; s_* >= 0: F*_L ; s_R > 0: F*_R ; else F_R
    const bool left = (sl >= R(0)) || (ss >= R(0));
    const bool star = left ? !(sl >= R(0)) : (sr > R(0));
    const R sK = left ? sl : sr;
    const R mK = left ? ml : mr;
    const R cK = left ? cl : cr;
    R W[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) W[c] = left ? WL[c] : WR[c];

    const R rho = W[0], u = W[1], p = W[NC - 1];
    const R mu = rho * u;
    // tangential |t|^2 as a sum of rounded squares: symmetric in the
    // tangential components, so interchanging two axes is bitwise
    R tsq = R(0);
#pragma unroll
    for (int k = 0; k < NT; ++k) tsq = tsq + W[2 + k] * W[2 + k];
    const R vsq = O::fma(u, u, tsq);
    const R E = O::fma(p, gas.inv_gm1, R(0.5) * rho * vsq);

    // star state chi (1, s_*, t, E/rho + (s_* - u)(s_* + p/(rho ds))),
    // chi = rho ds / (s - s_*), with 1/(s - s_*) and 1/(rho ds) from one
    // reciprocal; F*_K = F_K + s_K (U*_K - U_K) for mass, normal momentum and
    // energy (the upwind flux where no star state applies: there the star
    // quantities may not be finite, so the choice is a select)
    const R t1 = sK - ss;
    const R q = O::rcp1(t1 * mK);
    const R chi = mK * (mK * q);
    const R p_m = p * (t1 * q);
    const R e_rho = O::fma(cK * cK, gas.inv_g_gm1, R(0.5) * vsq);
    const R f0 = O::fma(sK, chi - rho, mu);
    const R f1 = O::fma(sK, chi * ss - mu, O::fma(mu, u, p));
    const R f4 = O::fma(sK, chi * O::fma(ss - u, ss + p_m, e_rho) - E, (E + p) * u);
    F[0] = star ? f0 : mu;
    F[1] = star ? f1 : O::fma(mu, u, p);
    F[NC - 1] = star ? f4 : (E + p) * u;
    // the tangential velocities are carried by the mass flux: in the star
    // regions U*_t = chi t and U_t = rho t give F_t = t (rho u + s_K (chi -
    // rho)) = t F_0, and outside them F_t = rho u t = t F_0 as well
#pragma unroll
    for (int k = 0; k < NT; ++k) F[2 + k] = W[2 + k] * F[0];
}

// Flux through the face between cells w1 and w2 along kernel axis AX from the
// global-frame primitive states of the four cells around it: PLM per
// component, rotate the face normal to the first velocity slot, HLLC, rotate
// back.  Tangential velocities keep increasing component order.
// FIRST: piecewise-constant states (the face states are w1 and w2).
template <int NDIM, int AX, typename R, bool FIRST = false>
__device__ __forceinline__ void face_flux(const Gas<R>& g, const R (&w0)[NDIM + 2], const R (&w1)[NDIM + 2],
                                          const R (&w2)[NDIM + 2], const R (&w3)[NDIM + 2],
                                          R (&F)[NDIM + 2]) {
    constexpr int NC = NDIM + 2;
    constexpr int NT = NDIM - 1;
    constexpr int VN = vcomp<NDIM>(AX);
    R wl[NC], wr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if constexpr (FIRST) {
            wl[c] = w1[c];
            wr[c] = w2[c];
        } else {
            R dj, dj1;
            Ops<R>::minmod2(w1[c] - w0[c], w2[c] - w1[c], w3[c] - w2[c], dj, dj1);
            wl[c] = Ops<R>::fma(R(0.5), dj, w1[c]);
            wr[c] = Ops<R>::fma(R(-0.5), dj1, w2[c]);
        }
    }
    R L[NT + 3], Rs[NT + 3], Fn[NT + 3];
    L[0] = wl[0];
    Rs[0] = wr[0];
    L[1] = wl[VN];
    Rs[1] = wr[VN];
    {
        int k = 2;
#pragma unroll
        for (int e = 1; e <= NDIM; ++e) {
            if (e == VN) continue;
            L[k] = wl[e];
            Rs[k] = wr[e];
            ++k;
        }
    }
    L[NT + 2] = wl[NC - 1];
    Rs[NT + 2] = wr[NC - 1];
    hllc<R, NT>(g, L, Rs, Fn);
    F[0] = Fn[0];
    F[VN] = Fn[1];
    {
        int k = 2;
#pragma unroll
        for (int e = 1; e <= NDIM; ++e) {
            if (e == VN) continue;
            F[e] = Fn[k++];
        }
    }
    F[NC - 1] = Fn[NT + 2];
}

// Flux through an in-plane face of a 3-D tile whose axis (0: x, 1: y) is a
// run-time value: the same arithmetic as face_flux<3, 0 or 1>, with the
// rotation done by selects so faces of both axes share one code path.
template <typename R, bool FIRST = false>
__device__ __forceinline__ void face_flux_xy(const Gas<R>& g, bool yaxis, const R (&w0)[5], const R (&w1)[5],
                                             const R (&w2)[5], const R (&w3)[5], R (&F)[5]) {
    R wl[5], wr[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        if constexpr (FIRST) {
            wl[c] = w1[c];
            wr[c] = w2[c];
        } else {
            R dj, dj1;
            Ops<R>::minmod2(w1[c] - w0[c], w2[c] - w1[c], w3[c] - w2[c], dj, dj1);
            wl[c] = Ops<R>::fma(R(0.5), dj, w1[c]);
            wr[c] = Ops<R>::fma(R(-0.5), dj1, w2[c]);
        }
    }
    // normal velocity first, then the other in-plane one, then z
    R L[5] = {wl[0], yaxis ? wl[2] : wl[1], yaxis ? wl[1] : wl[2], wl[3], wl[4]};
    R Rr[5] = {wr[0], yaxis ? wr[2] : wr[1], yaxis ? wr[1] : wr[2], wr[3], wr[4]};
    R Fn[5];
    hllc<R, 2>(g, L, Rr, Fn);
    F[0] = Fn[0];
    F[1] = yaxis ? Fn[2] : Fn[1];
    F[2] = yaxis ? Fn[1] : Fn[2];
    F[3] = Fn[3];
    F[4] = Fn[4];
}

// Flux from already reconstructed face states (global frame) along kernel
// axis AX: the rotation and HLLC of face_flux without the PLM step.
template <int NDIM, int AX, typename R>
__device__ __forceinline__ void face_flux_states(const Gas<R>& g, const R (&wl)[NDIM + 2],
                                                 const R (&wr)[NDIM + 2], R (&F)[NDIM + 2]) {
    constexpr int NC = NDIM + 2;
    constexpr int NT = NDIM - 1;
    constexpr int VN = vcomp<NDIM>(AX);
    R L[NT + 3], Rs[NT + 3], Fn[NT + 3];
    L[0] = wl[0];
    Rs[0] = wr[0];
    L[1] = wl[VN];
    Rs[1] = wr[VN];
    {
        int k = 2;
#pragma unroll
        for (int e = 1; e <= NDIM; ++e) {
            if (e == VN) continue;
            L[k] = wl[e];
            Rs[k] = wr[e];
            ++k;
        }
    }
    L[NT + 2] = wl[NC - 1];
    Rs[NT + 2] = wr[NC - 1];
    hllc<R, NT>(g, L, Rs, Fn);
    F[0] = Fn[0];
    F[VN] = Fn[1];
    {
        int k = 2;
#pragma unroll
        for (int e = 1; e <= NDIM; ++e) {
            if (e == VN) continue;
            F[e] = Fn[k++];
        }
    }
    F[NC - 1] = Fn[NT + 2];
}

// ---------------------------------------------------------------- boundaries

// Interior index for coordinate q on kernel axis ax of the whole mesh
// (extent n * blocks) and the treatment of the normal velocity (Sec. 3.1.1;
// each side read as the left-x case).
__device__ __forceinline__ int resolve_mesh(const Geo& g, int ax, int q, int& vmode) {
    const int N = g.n[ax] * g.blocks[ax];
    vmode = VM_NONE;
    if (q >= 0 && q < N) return q;
    if (q < 0) {
        switch (g.bc[ax][0]) {
            case BC_PERIODIC: return q + N;
            case BC_FREE: return 0;
            case BC_OUTFLOW: vmode = VM_CLIP_LO; return 0;
            default: vmode = VM_NEG; return -1 - q;
        }
    }
    switch (g.bc[ax][1]) {
        case BC_PERIODIC: return q - N;
        case BC_FREE: return N - 1;
        case BC_OUTFLOW: vmode = VM_CLIP_HI; return N - 1;
        default: vmode = VM_NEG; return 2 * N - 1 - q;
    }
}

// The sides of one block: the block-index offset of the neighbour a side
// reads its ghosts from (a c-boundary: inside the mesh, or across a periodic
// axis), or kNoLink at a face of the mesh with a p-boundary rule.
// On a refined mesh a side may instead read a ghost slot (slo/shi: the slot
// index, else -1).
constexpr int kNoLink = 0x7fffffff;
struct Links {
    int lo[3], hi[3];
    int slo[3], shi[3];
};

__device__ __forceinline__ Links block_links(const Geo& g, int blk) {
    Links L;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) L.slo[ax] = L.shi[ax] = -1;
    const int c[3] = {blk % g.blocks[0], (blk / g.blocks[0]) % g.blocks[1], blk / (g.blocks[0] * g.blocks[1])};
    const int stride[3] = {1, g.blocks[0], g.blocks[0] * g.blocks[1]};
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int B = g.blocks[ax];
        const int wrap = (B - 1) * stride[ax];
        L.lo[ax] = c[ax] > 0 ? -stride[ax] : (g.bc[ax][0] == BC_PERIODIC ? wrap : kNoLink);
        L.hi[ax] = c[ax] < B - 1 ? stride[ax] : (g.bc[ax][1] == BC_PERIODIC ? -wrap : kNoLink);
    }
    return L;
}

// The sides of a block of a refined mesh, from its side codes.
__device__ __forceinline__ Links table_links(const int* __restrict__ side, int blk) {
    Links L;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int lo = side[6 * blk + 2 * ax], hi = side[6 * blk + 2 * ax + 1];
        L.lo[ax] = lo >= 0 ? lo - blk : kNoLink;
        L.hi[ax] = hi >= 0 ? hi - blk : kNoLink;
        L.slo[ax] = lo <= kSideSlot0 ? kSideSlot0 - lo : -1;
        L.shi[ax] = hi <= kSideSlot0 ? kSideSlot0 - hi : -1;
    }
    return L;
}

// The refinement level of a block.
__device__ __forceinline__ int block_level(const LevelStarts& starts, int blk) {
    int lev = 0;
#pragma unroll
    for (int L = 1; L < kMaxLevels; ++L) lev += blk >= starts.s[L - 1] ? 1 : 0;
    return lev;
}

// The restriction slot (a level jump onto finer blocks) of the side of block
// blk that the cells at coordinate `at` of axis ax lie next to, or -1.
__device__ __forceinline__ int jump_slot(const Geo& g, const int* __restrict__ side, int nres, int blk, int ax,
                                         int at) {
    const int code = at == 0 ? side[6 * blk + 2 * ax] : (at == g.n[ax] - 1 ? side[6 * blk + 2 * ax + 1] : 0);
    const int slot = kSideSlot0 - code;
    return slot >= 0 && slot < nres ? slot : -1;
}

// The sides of a launch's block: from the side codes of a refined mesh, else
// from the uniform block grid (selected field by field, so the structure
// stays in registers).
__device__ __forceinline__ Links stage_links(const StageArgs& a, int blk) {
    const Geo& g = a.geo;
    const bool tab = a.side != nullptr;
    const Links G = block_links(g, blk);
    Links L;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int lo = tab ? a.side[6 * blk + 2 * ax] : 0, hi = tab ? a.side[6 * blk + 2 * ax + 1] : 0;
        L.lo[ax] = tab ? (lo >= 0 ? lo - blk : kNoLink) : G.lo[ax];
        L.hi[ax] = tab ? (hi >= 0 ? hi - blk : kNoLink) : G.hi[ax];
        L.slo[ax] = tab && lo <= kSideSlot0 ? kSideSlot0 - lo : -1;
        L.shi[ax] = tab && hi <= kSideSlot0 ? kSideSlot0 - hi : -1;
    }
    return L;
}

// Ghost coordinate q (one block's extent N on kernel axis ax) -> the cell it
// copies: in the linked block dblk (offset in blocks, 0 for the block
// itself) at q -/+ N, or by the p-boundary rule of a mesh face, with the
// treatment of the normal velocity (Sec. 3.1.1); or, at a level jump, the
// ghost slot `slot` (else -1) and the layer returned (0 next to the face).
__device__ __forceinline__ int resolve(const Geo& g, const Links& L, int ax, int q, int& vmode, int& dblk,
                                       int& slot) {
    const int N = g.n[ax];
    vmode = VM_NONE;
    dblk = 0;
    slot = -1;
    if (q >= 0 && q < N) return q;
    if (q < 0) {
        if (L.slo[ax] >= 0) {
            slot = L.slo[ax];
            return -1 - q;
        }
        if (L.lo[ax] != kNoLink) {
            dblk = L.lo[ax];
            return q + N;
        }
        switch (g.bc[ax][0]) {
            case BC_FREE: return 0;
            case BC_OUTFLOW: vmode = VM_CLIP_LO; return 0;
            default: vmode = VM_NEG; return -1 - q;
        }
    }
    if (L.shi[ax] >= 0) {
        slot = L.shi[ax];
        return q - N;
    }
    if (L.hi[ax] != kNoLink) {
        dblk = L.hi[ax];
        return q - N;
    }
    switch (g.bc[ax][1]) {
        case BC_FREE: return N - 1;
        case BC_OUTFLOW: vmode = VM_CLIP_HI; return N - 1;
        default: vmode = VM_NEG; return 2 * N - 1 - q;
    }
}

__device__ __forceinline__ double apply_vmode(double v, int vmode) {
    switch (vmode) {
        case VM_NEG: return -v;
        case VM_CLIP_LO: return v > 0.0 ? 0.0 : v;
        case VM_CLIP_HI: return v < 0.0 ? 0.0 : v;
        default: return v;
    }
}

// Primitive state at kernel coordinates (x, y, z) of the whole mesh, at most
// one of which lies outside it (the axis-aligned stencil never needs corner
// ghosts); U in the block layout.
template <int NDIM, typename R>
__device__ __forceinline__ void load_w(const Geo& g, const double* __restrict__ U, int x, int y, int z,
                                       R (&W)[NDIM + 2], bool& bad) {
    constexpr int NC = NDIM + 2;
    int vm = VM_NONE, ax = -1;
    if (x < 0 || x >= g.n[0] * g.blocks[0]) {
        x = resolve_mesh(g, 0, x, vm);
        ax = 0;
    } else if (y < 0 || y >= g.n[1] * g.blocks[1]) {
        y = resolve_mesh(g, 1, y, vm);
        ax = 1;
    } else if (z < 0 || z >= g.n[2] * g.blocks[2]) {
        z = resolve_mesh(g, 2, z, vm);
        ax = 2;
    }
    const int blk = x / g.n[0] + g.blocks[0] * (y / g.n[1] + g.blocks[1] * (z / g.n[2]));
    const long long cell = ((long long)(z % g.n[2]) * g.n[1] + y % g.n[1]) * g.n[0] + x % g.n[0];
    const double* Ub = U + (long long)blk * NC * g.ncells;
    double u[NC], w[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) u[c] = Ub[c * g.ncells + cell];
    bad |= !cons_to_prim<NDIM>(g.gamma - 1.0, u, w);
    if (ax >= 0) {
        const int vc = ax == 0 ? 1 : (ax == 1 ? 2 : NDIM);
#pragma unroll
        for (int c = 1; c <= NDIM; ++c)
            if (c == vc) w[c] = apply_vmode(w[c], vm);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) W[c] = (R)w[c];
}

// CFL rate of one cell, max over active kernel axes of (|v| + c)/dx; the
// time step is cfl / (max over cells of the rate), the same quantity as
// cfl * min over cells and axes of dx / (|v| + c) (Sec. 3.1).
template <int NDIM>
__device__ __forceinline__ double cfl_rate(const Geo& g, const double (&w)[NDIM + 2]) {
    const double gp = g.gamma * w[NDIM + 1];
    const double cs = gp * Ops<double>::rsq(gp * w[0]);  // sqrt(gamma p / rho)
    double best = (dabs(w[1]) + cs) * g.inv_dx[0];
    if (NDIM == 3) {
        const double c1 = (dabs(w[2]) + cs) * g.inv_dx[1];
        best = c1 > best ? c1 : best;
    }
    if (NDIM >= 2) {
        const double c2 = (dabs(w[NDIM]) + cs) * g.inv_dx[2];
        best = c2 > best ? c2 : best;
    }
    return best;
}

// dt of the next step from the control block: the CFL step, shortened to
// land on t_end when one is set.
__device__ __forceinline__ double device_dt(const Ctrl* c) {
    double dt = c->dt_raw;
    if (c->t_end > 0.0) {
        const double rem = c->t_end - c->t;
        if (dt >= rem) dt = rem;
    }
    return dt > 0.0 ? dt : 0.0;
}

__device__ __forceinline__ void update_done(Ctrl* c) {
    c->done = (c->t_end > 0.0 && !(c->t < c->t_end)) || (c->max_steps > 0 && c->steps >= c->max_steps);
}

// Advance time by the step just taken and take the next dt from the rate.
__device__ __forceinline__ void finalize_step(Ctrl* c, double cfl, double rate) {
    if (c->done) return;
    const double dt = device_dt(c);
    const bool last = c->t_end > 0.0 && c->dt_raw >= c->t_end - c->t;
    if (dt > 0.0) {
        c->t = last ? c->t_end : c->t + dt;
        c->steps += 1;
    }
    c->dt_raw = cfl / rate;
    c->dt_valid = 1;
    update_done(c);
}

// Work-groups are dispatched round-robin over the 8 XCDs; hand each XCD a
// contiguous range of tiles so neighbouring tiles share one L2.
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    constexpr int X = 8;
    const int q = nb / X, r = nb % X;
    const int x = bid % X, i = bid / X;
    return x * q + (x < r ? x : r) + i;
}

// A value that every lane holds, in scalar registers.
__device__ __forceinline__ double uniform(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | lo);
}

// max(v, v of the lane that the DPP control names, 0 where there is none)
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
    const double o = __longlong_as_double(((long long)hi << 32) | lo);
    return o > v ? o : v;
}

// Largest of the wave's non-negative values, in every lane; the whole wave
// takes part.  Six lane moves in the VALU (rows of 16 by shifts, then their
// last lanes broadcast on) instead of six exchanges through LDS: a 1-D step of
// 256 cells 2.87 -> 2.71 us, with its books beside the fluxes.
__device__ __forceinline__ double wave_max(double v) {
    v = dpp_max<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8
    v = dpp_max<0x112, 0xf>(v);
    v = dpp_max<0x114, 0xf>(v);
    v = dpp_max<0x118, 0xf>(v);
    v = dpp_max<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_max<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | lo);
}

__device__ __forceinline__ double load_slot(Ctrl* c, unsigned int par) {
    return __longlong_as_double((long long)*rate_slot(c, par, threadIdx.x % kRateSlots));
}

__device__ __forceinline__ void add_rate(Ctrl* c, unsigned int par, double rate) {
    atomicMax(rate_slot(c, par, blockIdx.x % kRateSlots), (unsigned long long)__double_as_longlong(rate));
}

// The control of the step that begins, from the pending rate (of set par,
// loaded by the caller): what CTRL_FINALIZE would make of the block, without
// writing it.  The step's own rate goes to the other set when one is pending.
__device__ __forceinline__ StepCtl begin_step(const Ctrl* c, double cfl, double rate) {
    Ctrl k;
    k.dt_raw = c->dt_raw;
    k.t = c->t;
    k.steps = c->steps;
    k.t_end = c->t_end;
    k.max_steps = c->max_steps;
    k.done = c->done;
    const unsigned int pend = c->pend;
    if (pend == kPendStep) finalize_step(&k, cfl, rate);
    if (pend == kPendRate) k.dt_raw = cfl / rate;
    StepCtl n;
    n.dt_raw = k.dt_raw;
    n.t = k.t;
    n.steps = k.steps;
    n.done = k.done;
    n.par = pend != kPendNone ? c->par ^ 1u : c->par;
    n.dt = device_dt(&k);
    return n;
}

// ------------------------------------------------------------- stage kernel

// Raw conserved values of one cell; cell = plane offset + column offset.
template <int NC>
__device__ __forceinline__ void load_u(const double* __restrict__ U, long long N, long long cell,
                                       double (&u)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) u[c] = U[c * N + cell];
}

// Primitive state of raw values u; the velocity along kernel axis vax (if
// any) takes the boundary treatment vm of the ghost it fills.
template <int NDIM, typename R, bool CHECK = true>
__device__ __forceinline__ void to_prim(double gm1, const double (&u)[NDIM + 2], int vax, int vm,
                                        R (&W)[NDIM + 2], bool& bad) {
    constexpr int NC = NDIM + 2;
    double w[NC];
    const bool ok = cons_to_prim<NDIM, sizeof(R) == 4>(gm1, u, w);
    if (CHECK) bad |= !ok;
    if (vax >= 0) {
        const int vc = vax == 0 ? 1 : (vax == 1 ? 2 : NDIM);
#pragma unroll
        for (int c = 1; c <= NDIM; ++c)
            if (c == vc) w[c] = apply_vmode(w[c], vm);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) W[c] = (R)w[c];
}

// The stencil input of a cell as primitive variables in R: conserved FP64
// values converted (to_prim), or, with PRIM, stored primitive values of type
// R (the van Leer predictor state) held as doubles, with the boundary
// treatment of the normal velocity applied.
template <int NDIM, typename R, bool PRIM, bool CHECK = true>
__device__ __forceinline__ void in_to_w(double gm1, const double (&u)[NDIM + 2], int vax, int vm,
                                        R (&W)[NDIM + 2], bool& bad) {
    constexpr int NC = NDIM + 2;
    if constexpr (PRIM) {
        const int vc = vax == 0 ? 1 : (vax == 1 ? 2 : NDIM);
#pragma unroll
        for (int c = 0; c < NC; ++c) W[c] = (R)((vax >= 0 && c == vc) ? apply_vmode(u[c], vm) : u[c]);
    } else {
        to_prim<NDIM, R, CHECK>(gm1, u, vax, vm, W, bad);
    }
}

// Access to one plane of a [comp][cell] field through a buffer resource:
// the plane base (component base + plane offset, the same for the whole
// work-group) lives in scalar registers and the thread supplies a 32-bit
// byte offset, so no per-thread 64-bit address arithmetic is needed.  The
// resource covers exactly the plane (extent bytes): an offset outside it
// reads 0 and writes nothing.
constexpr int kBufferWord3 = 0x00020000;  // raw buffer, 32-bit data format (gfx9)
typedef unsigned int u32x2 __attribute__((__vector_size__(2 * sizeof(unsigned int))));

template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const T* F, long long uniform_off,
                                                             uint32_t extent_bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(F + uniform_off), (short)0, (int)extent_bytes,
                                             kBufferWord3);
}

// Cache policy of the accesses that touch a value for the last time in a
// step (the final update's read of U^n and its write of U^{n+1}): the
// non-temporal hint (slc), so that streaming data does not displace the
// stencil's planes in L2.  Measured 1.5-2.5 % faster for those stages; the
// first stages keep the default policy (their output is read right after,
// and the hint measured neutral to 1.5 % slower there).
constexpr int kNonTemporal = 2;

template <typename T, int CPOL = 0>
__device__ __forceinline__ T plane_load(const T* F, long long uniform_off, uint32_t extent_bytes,
                                        uint32_t thread_bytes) {
    const __amdgpu_buffer_rsrc_t r = plane_rsrc(F, uniform_off, extent_bytes);
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, thread_bytes, 0, CPOL));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, thread_bytes, 0, CPOL));
}

template <typename T, int CPOL = 0>
__device__ __forceinline__ void plane_store(T* F, long long uniform_off, uint32_t extent_bytes,
                                            uint32_t thread_bytes, T v) {
    const __amdgpu_buffer_rsrc_t r = plane_rsrc(F, uniform_off, extent_bytes);
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, thread_bytes, 0, CPOL);
    else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, thread_bytes, 0, CPOL);
}

// NC values of one cell from a field of type T (layout [comp][cell]) as doubles.
template <int NC, typename T>
__device__ __forceinline__ void load_as_double(const T* __restrict__ F, long long N, long long cell,
                                               double (&u)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) u[c] = (double)F[c * N + cell];
}

// One stage over a TX x TY tile column and a chunk of kz planes.
//
// Software pipeline per plane k (kernel z): raw U of the interior plane k+3 is
// loaded one iteration before it is converted, so global loads stay in flight
// across the two LDS barriers; where StageOccupancy says so the halo cells of
// plane k+1 are too, and the input at plane k for the update comes from a ring
// in LDS.  Each thread owns at most one halo cell of the plane (4 TX + 4 TY <=
// TX TY).
// Work-groups per CU the compiler is asked to fit: the FP32 path keeps four
// 256-thread groups per CU (16 waves); FP64 needs more registers per thread.
// FEW: the form of the FP64 3-D Heun stage 2 for at most two waves on a SIMD,
// where a march is bound by the latency of its plane's loads and not by the
// waves that fit: everything is loaded a plane ahead.
constexpr bool has_few(int ndim, bool fp64, int mode) { return ndim == 3 && fp64 && mode == MODE_STAGE2; }

template <int NDIM, typename R, int MODE, bool FEW = false>
struct StageOccupancy {
    // Input ring: the raw input values of a cell, read for its conversion
    // when its plane enters the z stencil, are kept in LDS until the update
    // of that plane instead of being read again.  Two planes suffice: the
    // value of the plane that is updated is taken out at the top of the
    // iteration, before that of the plane two ahead goes into its place.
    // With three planes (and one prefetch more in stage 2) the mixed stages
    // held twelve waves on a CU; with two they hold sixteen in work-groups of
    // 32 x 16, whose halo and extra faces are a quarter less than those of
    // 32 x 8: at 256^3 stage 1 357 -> 333 us, stage 2 463 -> 450 us.  In 2-D
    // two rows leave the mixed stages their waves (4096 x 1024: a step 164 ->
    // 141 us with the halo prefetch below).  The FP64 stages lose a wave per
    // SIMD to it in 3-D and spill in 2-D (191 -> 198 us) and do without.  The
    // van Leer predictor looks one plane ahead only, so it needs one.
    static constexpr bool kPred = MODE == MODE_VL2_PRED || MODE == MODE_VL2_PRED_C;
    static constexpr bool kHeun = MODE == MODE_STAGE1 || MODE == MODE_STAGE2 || MODE == MODE_STAGE2_R;
    static constexpr bool kRing =
        FEW || kPred || (sizeof(R) == 4 && kHeun);
    // occupancy range (waves per SIMD) the compiler aims for: at least
    // kWaves (its register budget), at most kWavesMax (8: no bound)
    // The FP64 stage 2 holds three (twelve waves on a CU) without the double
    // buffers of W and the fluxes that one barrier per plane takes: 653 us at
    // 256^3 against 689 us in eight waves with one barrier.  (Launches of no
    // more than eight waves: FEW.)
    // In 2-D the FP64 stages hold four with a few spilled registers (4096 x
    // 1024: a step 200 -> 187 us, 1024^2 72 -> 66 us against three waves).
    static constexpr int kWaves = FEW ? 2 : (sizeof(R) == 4 || NDIM == 2 ? 4 : (NDIM == 3 ? 3 : 2));
    static constexpr int kWavesMax = 8;
    // The raw halo cell of the next plane loaded one iteration ahead, so the
    // barrier after the plane's W does not wait for it: ten more registers.
    // Measured at 256^3: the mixed Heun stage 2 holds them (462 -> 452 us at
    // four waves per SIMD), the mixed stage 1, the mixed 2-D stages and the
    // mixed van Leer predictor gain about 2 % (192^3 in blocks 128 -> 124 us);
    // the FP64 stages lose 5-6 % (a wave per SIMD; FEW has none to lose), the
    // mixed van Leer corrector 17 % in 3-D (383 -> 447 us), and do without.
    static constexpr bool kHaloPrefetch = FEW || (NDIM >= 2 && sizeof(R) == 4 && (kHeun || kPred));
    // U^n of the next updated plane loaded during this plane's update, before
    // its stores.  With the input ring and the halo prefetch it is what FEW is:
    // 96^3 in chunks of 64 planes (four waves on a CU) a step 512 -> 467 us, of
    // 16 planes 148 -> 138 us, 192^3 in chunks of 64 (eight waves) 698 -> 661 us.
    static constexpr bool kBaseAhead = FEW;
    // U^n for the update loaded before the faces instead of after them, so it
    // arrives beside them.  Measured: the mixed 2-D van Leer corrector 68 -> 63
    // us at 4096 x 1024; the mixed 2-D Heun stage 2 is even there and loses 2 %
    // in batches; in 3-D it costs registers (the van Leer step 663 -> 696 us,
    // the mixed Heun one +2 %, FP64 +5 %, spilled).
    static constexpr bool kBaseEarly =
        NDIM == 2 && sizeof(R) == 4 && (MODE == MODE_VL2_CORR || MODE == MODE_VL2_CORR_C);
    // The waves that convert the halo cells and compute the faces past the
    // tile's last row and column (the first waves of the work-group) run at
    // raised priority through that work, up to the barrier after the faces:
    // they are the ones the other waves wait for there.  Measured at 256^3:
    // mixed stage 2 -4.5 %, FP64 stage 1 -6.5 %.
    static constexpr bool kPrio = NDIM == 3;
};

template <int NDIM, typename R, int MODE, int TX, int TY, bool FEW>
__device__ __forceinline__ void stage_body(const StageArgs& a, int b, int blk, bool leader) {
    constexpr int NC = NDIM + 2;
    constexpr bool HY = (NDIM == 3);
    constexpr bool HZ = (NDIM >= 2);
    constexpr int NT = TX * TY;
    // van Leer modes: the predictor (piecewise-constant states, half step,
    // writes the predicted primitive state of type R into a.out; _C: the
    // predicted conserved state in FP64) and the corrector (reads that state
    // as its stencil input, PLM, full step from U^n in a.base, writes
    // U^{n+1} to a.out)
    constexpr bool PRED = MODE == MODE_VL2_PRED || MODE == MODE_VL2_PRED_C;
    constexpr bool CORR = MODE == MODE_VL2_CORR || MODE == MODE_VL2_CORR_C;
    constexpr bool PRIM_OUT = MODE == MODE_VL2_PRED;
    constexpr bool FIRST = PRED;
    // the stencil's reach on every axis: one cell for piecewise-constant states
    constexpr int HW = FIRST ? 1 : 2;
    constexpr bool PRIM_IN = MODE == MODE_VL2_CORR;
    constexpr bool STAGE2 = MODE == MODE_STAGE2 || MODE == MODE_STAGE2_R;
    constexpr bool NEED_UIN = MODE == MODE_STAGE1 || STAGE2 || PRED;
    constexpr bool NEED_BASE = STAGE2 || CORR;
    constexpr bool EPILOGUE = STAGE2 || CORR;
    // the second stage of a refined mesh leaves the rate of the cells that are
    // corrected after it to the correction (a mode of its own: the test took
    // the unrefined mixed stage 2 over its 128 registers, 48^3 +6 %)
    constexpr bool LEVELS = MODE == MODE_STAGE2_R || MODE == MODE_VL2_CORR_C;
    static_assert(HY || TY == 1, "tile rows need a second in-plane axis");
    static_assert(4 * TX + (HY ? 4 * TY : 0) <= NT || !HY, "one halo cell per thread");
    static_assert(HY || TX >= 4, "one halo cell per thread");

    const Geo& g = a.geo;
    const int n0 = g.n[0], n1 = g.n[1], n2 = g.n[2];
    const long long N = g.ncells;
    const long long P = (long long)n0 * n1;  // plane stride
    const long long BS = (long long)NC * N;  // elements of one block of a field
    const long long boff = (long long)blk * BS;
    const Links lk = stage_links(a, blk);
    const double gm1 = g.gamma - 1.0;

    const int tix = b % a.tiles_x;
    b /= a.tiles_x;
    const int tiy = b % a.tiles_y;
    b /= a.tiles_y;
    const int x0 = tix * TX, y0 = tiy * TY, z0 = b * a.kz;
    const int z1 = min(z0 + a.kz, n2);
    const int ax = min(TX, n0 - x0);
    const int ay = min(TY, n1 - y0);
    const int tid = threadIdx.x;
    const int lx = tid % TX, ly = tid / TX;
    const bool act = lx < ax && ly < ay;
    const long long col = (long long)(y0 + ly) * n0 + (x0 + lx);

    // this thread's halo cell (tile coordinates hx, hy), resolved once to an
    // element offset hcol in the field (its block's offset + the in-plane
    // index) or in the ghost buffer (hslot), with its plane and component
    // strides
    bool hact = false, hslot = false;
    int hx = 0, hy = 0, hvax = -1, hvm = VM_NONE, hk = 0;
    long long hcol = 0, hc = 0;
    {
        const int nhx = 2 * HW * ay;
        const int nhy = HY ? 2 * HW * ax : 0;
        if (tid < nhx) {
            const int q = tid % (2 * HW);
            hy = tid / (2 * HW);
            hx = q < HW ? q - HW : ax + (q - HW);
            hact = true;
        } else if (tid < nhx + nhy) {
            const int h2 = tid - nhx, q = h2 % (2 * HW);
            hx = h2 / (2 * HW);
            hy = q < HW ? q - HW : ay + (q - HW);
            hact = true;
        }
        if (hact) {
            int X = x0 + hx, Y = y0 + hy, db = 0, sl = -1;
            if (X < 0 || X >= n0) {
                X = resolve(g, lk, 0, X, hvm, db, sl);
                hvax = 0;
            } else if (Y < 0 || Y >= n1) {
                Y = resolve(g, lk, 1, Y, hvm, db, sl);
                hvax = 1;
            }
            if (sl >= 0) {
                // a ghost slot: [comp][layer][z][y] of an x side, [comp][layer][z][x] of a y side
                hslot = true;
                const long long sb = (long long)sl * NC * a.gcs;
                hcol = hvax == 0 ? sb + ((long long)X * n2) * n1 + Y : sb + ((long long)Y * n2) * n0 + X;
                hk = hvax == 0 ? n1 : n0;
                hc = a.gcs;
            } else {
                hcol = (long long)(blk + db) * BS + (long long)Y * n0 + X;
                hk = (int)P;
                hc = N;
            }
        }
    }

    // whether an in-plane side treats the normal velocity of its ghosts
    // (outflow, reflecting); uniform over the grid
    const bool halo_vm = g.bc[0][0] >= BC_OUTFLOW || g.bc[0][1] >= BC_OUTFLOW ||
                         (HY && (g.bc[1][0] >= BC_OUTFLOW || g.bc[1][1] >= BC_OUTFLOW));
    // both sets of rate slots, loaded ahead of the state (a chained first stage)
    double slot0 = 0.0, slot1 = 0.0;
    if (!EPILOGUE && a.chain) {
        slot0 = load_slot(a.ctrl, 0);
        slot1 = load_slot(a.ctrl, 1);
    }
    // the step's length, and whether the mesh still runs (uniform over the
    // launch; the leader is one work-group of the mesh's launch): taken before
    // the first planes in 3-D, and while they are on their way in 1-D and 2-D,
    // whose chunks are short (a batch of 48 meshes 5.78 -> 5.61 ms; the FP64
    // 3-D stage 1 would lose 3 % to it)
    constexpr bool CTRL_FIRST = NDIM == 3;
    // a refined mesh's block: level 0's cell widths times 2^-lev (exact)
    const int lev = a.side ? block_level(a.starts, blk) : 0;
    double lam0 = 0.0, lam1 = 0.0, lam2 = 0.0;
    unsigned int par = 0;
    auto take_step = [&]() __attribute__((always_inline)) -> bool {
        double dt_step = a.dt_host;
        if (a.chain && !EPILOGUE) {
            const StepCtl n = begin_step(a.ctrl, g.cfl, wave_max(a.ctrl->par ? slot1 : slot0));
            if (leader) {
                if (tid == 0) {
                    *ctrl_next(a.ctrl) = n;
                    if (a.use_device_dt && a.ctrl->pend == kPendRate && a.ctrl->pend_flags)
                        atomicOr(&a.ctrl->flags, a.ctrl->pend_flags);
                    a.ctrl->pend_flags = 0;
                }
                if (tid < kRateSlots) *rate_slot(a.ctrl, n.par, tid) = 0ull;
            }
            if (a.use_device_dt) {
                if (n.done) return false;
                dt_step = n.dt;
            }
        } else if (a.chain) {
            const StepCtl n = *ctrl_next(a.ctrl);
            par = __builtin_amdgcn_readfirstlane(n.par);
            if (leader && tid == 0) {
                a.ctrl->par = n.par;
                a.ctrl->pend = a.use_device_dt ? (n.done ? kPendNone : kPendStep)
                                              : (a.want_dt ? kPendRate : kPendNone);
                a.ctrl->dt_raw = n.dt_raw;
                a.ctrl->t = a.use_device_dt ? n.t : n.t + a.dt_host;
                a.ctrl->steps = a.use_device_dt ? n.steps : n.steps + 1;
                a.ctrl->done = n.done;
                a.ctrl->dt_valid = a.use_device_dt ? 1 : 0;
            }
            if (a.use_device_dt) {
                if (n.done) return false;
                dt_step = n.dt;
            }
        } else {
            if (a.use_device_dt) dt_step = device_dt(a.ctrl);
            if (EPILOGUE) par = a.ctrl->par;
        }
        dt_step = uniform(dt_step);
        const double dt = PRED ? 0.5 * dt_step : dt_step;  // the predictor advances half a step
        lam0 = uniform(dt / __builtin_ldexp(g.dx[0], -lev));
        lam1 = uniform(dt / __builtin_ldexp(g.dx[1], -lev));
        lam2 = uniform(dt / __builtin_ldexp(g.dx[2], -lev));
        return true;
    };
    if (CTRL_FIRST && !take_step()) return;
    const Gas<R> gr = make_gas<R>(g.gamma);

    constexpr bool RING = StageOccupancy<NDIM, R, MODE, FEW>::kRing && HZ;
    constexpr int RS = HW;  // ring slots: planes k .. k + HW - 1 between iterations
    __shared__ double sRaw[RING ? RS : 1][RING ? NC : 1][RING ? NT : 1];
    // rows of the W tile: in 1-D and 2-D a tile is one row (row offset RO)
    constexpr int RO = HY ? 0 : -2;
    __shared__ R sW[NC][HY ? TY + 4 : 1][TX + 4];
    using FT = R;
    __shared__ FT sFx[NC][TY][TX + 1];
    __shared__ FT sFy[HY ? NC : 1][HY ? TY + 1 : 1][TX];

    bool bad = false, bad_new = false;  // of the stage's input, and of the new state
    double rate = 0.0;
    // z pipeline entering iteration k: W_k and, with PLM, W_{k+1}, d = W_{k+1} -
    // W_k, the left state of face k+1/2 (W_k + delta_k / 2); fzb: the flux of
    // face k-1/2
    R wk[NC], wk1[NC], dk[NC], lz[NC];
    FT fzb[NC];
    // raw interior plane k+HW in flight (HZ)
    double ui[NC];
    int vmi = VM_NONE;
    // the raw halo cell of this thread (HALO_PF: the next plane's, in flight)
    constexpr bool HALO_PF = StageOccupancy<NDIM, R, MODE, FEW>::kHaloPrefetch;
    constexpr bool PRIO = StageOccupancy<NDIM, R, MODE, FEW>::kPrio;
    constexpr bool BASE_EARLY = StageOccupancy<NDIM, R, MODE, FEW>::kBaseEarly;
    constexpr bool BASE_AHEAD = StageOccupancy<NDIM, R, MODE, FEW>::kBaseAhead && NEED_BASE;
    double uhalo[NC];

    // interior plane z (any z: outside the mesh it is a ghost plane)
    // cell (plane offset poff, the same for the work-group) + (in-plane index tc)
    const uint32_t ext8 = (uint32_t)P * 8u, extR = (uint32_t)P * (uint32_t)sizeof(R);
    auto load_in = [&](long long poff, uint32_t tc, double (&u)[NC]) {
        if constexpr (PRIM_IN) {
            const R* F = reinterpret_cast<const R*>(a.in);
#pragma unroll
            for (int c = 0; c < NC; ++c) u[c] = (double)plane_load(F, c * N + poff, extR, tc * (uint32_t)sizeof(R));
        } else {
#pragma unroll
            for (int c = 0; c < NC; ++c) u[c] = plane_load(a.in, c * N + poff, ext8, tc * 8u);
        }
    };
    // the halo cell of plane k: it may lie in another block or in a ghost
    // slot, so it is addressed from the base with a per-thread offset
    auto load_halo = [&](int k, double (&u)[NC]) {
        const long long o = hcol + (long long)k * hk;
        if constexpr (PRIM_IN) {
            // (a refined mesh's ghost slots hold conserved values: its van
            // Leer corrector reads the conserved predictor, not this form)
            const R* F = reinterpret_cast<const R*>(a.in) + o;
#pragma unroll
            for (int c = 0; c < NC; ++c) u[c] = (double)F[c * hc];
        } else {
            // (the base is selected as an integer: selecting between the two
            // argument fields themselves makes the compiler copy the
            // arguments to private memory)
            const uintptr_t bi = reinterpret_cast<uintptr_t>(a.in), bg = reinterpret_cast<uintptr_t>(a.gbuf);
            const double* F = reinterpret_cast<const double*>(hslot ? bg : bi) + o;
#pragma unroll
            for (int c = 0; c < NC; ++c) u[c] = F[c * hc];
        }
    };
    const uint32_t col32 = (uint32_t)col;
    auto load_interior = [&](int z, double (&u)[NC], int& vm) {
        vm = VM_NONE;
        int zr = z, db = 0, sl = -1;
        if (z < 0 || z >= n2) zr = resolve(g, lk, 2, z, vm, db, sl);
        if (!PRIM_IN && sl >= 0) {
            // a ghost slot of a z side: [comp][layer][y][x], one plane per layer
#pragma unroll
            for (int c = 0; c < NC; ++c)
                u[c] = plane_load(a.gbuf, ((long long)sl * NC + c) * a.gcs + (long long)zr * P, ext8, col32 * 8u);
        } else {
            load_in((long long)(blk + db) * BS + (long long)zr * P, col32, u);
        }
    };

    if (HZ && act) {
        // planes z0-HW .. z0+HW-1: face z0-1/2 and, with PLM, the left state of
        // face z0+1/2, in the operations face_flux uses
        R w[2 * HW][NC];
#pragma unroll
        for (int q = 0; q < 2 * HW; ++q) {
            int vm;
            double u[NC];
            load_interior(z0 - HW + q, u, vm);
            in_to_w<NDIM, R, PRIM_IN>(gm1, u, vm == VM_NONE ? -1 : 2, vm, w[q], bad);
            if (RING && q >= HW) {
#pragma unroll
                for (int c = 0; c < NC; ++c) sRaw[RING ? (z0 - HW + q) % RS : 0][RING ? c : 0][RING ? tid : 0] = u[c];
            }
        }
        R wl[NC], wr[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            wk[c] = w[HW][c];
            if constexpr (FIRST) {
                wl[c] = w[0][c];
                wr[c] = w[1][c];
            } else {
                const R d0 = w[1][c] - w[0][c], d1 = w[2][c] - w[1][c], d2 = w[3][c] - w[2][c];
                R s1, s2;
                Ops<R>::minmod2(d0, d1, d2, s1, s2);
                wl[c] = Ops<R>::fma(R(0.5), s1, w[1][c]);
                wr[c] = Ops<R>::fma(R(-0.5), s2, w[2][c]);
                lz[c] = Ops<R>::fma(R(0.5), s2, w[2][c]);
                wk1[c] = w[3][c];
                dk[c] = d2;
            }
        }
        {
            R f[NC];
            face_flux_states<NDIM, 2, R>(gr, wl, wr, f);
#pragma unroll
            for (int c = 0; c < NC; ++c) fzb[c] = (FT)f[c];
        }
        load_interior(z0 + HW, ui, vmi);
    }
    if (!CTRL_FIRST && !take_step()) return;
    if (HALO_PF && hact && z0 < z1) load_halo(z0, uhalo);
    double uahead[NC];  // (BASE_AHEAD) U^n of the next updated plane
    auto load_ahead = [&](int k) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            uahead[c] = plane_load<double, kNonTemporal>(a.base, c * N + boff + (long long)k * P, ext8, col32 * 8u);
    };
    if (BASE_AHEAD && act && z0 < z1) load_ahead(z0);

    // One iteration: plane k + HW enters the stencil (its raw data ui, the
    // ghost treatment vmi), the plane after it is loaded into ui in its place,
    // and one plane is updated.
    auto plane = [&](const int k) __attribute__((always_inline)) {
        FT fzc[NC];                              // flux of face k+1/2
        double uin[NC], ubase[NC];
        if (RING && act) {
#pragma unroll
            for (int c = 0; c < NC; ++c) uin[c] = sRaw[RING ? k % RS : 0][RING ? c : 0][RING ? tid : 0];
        }
        if (act) {
            R wc[NC];
            if (HZ) {
                // W_{k+HW} arrived: z face k+1/2
                R w2[NC], wr[NC];
                // the ghost treatment of a plane is the same for the whole
                // work-group: held in a scalar register, it costs no divergence
                const int vz = __builtin_amdgcn_readfirstlane(vmi);
                in_to_w<NDIM, R, PRIM_IN>(gm1, ui, vz == VM_NONE ? -1 : 2, vz, w2, bad);
                // plane k+HW is an interior plane whenever its update comes
                if (RING) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) sRaw[RING ? (k + HW) % RS : 0][RING ? c : 0][RING ? tid : 0] = ui[c];
                }
                // the next iteration's; it lies at most HW planes outside the
                // mesh only while that iteration exists
                if (k + 1 < z1) load_interior(k + 1 + HW, ui, vmi);
                if constexpr (FIRST) {
                    // from the cells' values W_k and W_{k+1}
                    R f[NC];
                    face_flux_states<NDIM, 2, R>(gr, wk, w2, f);
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        fzc[c] = (FT)f[c];
                        wc[c] = wk[c];
                        wk[c] = w2[c];
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const R d2 = w2[c] - wk1[c];
                        const R s1 = minmod(dk[c], d2);
                        wr[c] = Ops<R>::fma(R(-0.5), s1, wk1[c]);
                        const R lnext = Ops<R>::fma(R(0.5), s1, wk1[c]);
                        wc[c] = wk[c];
                        dk[c] = d2;
                        wk[c] = wk1[c];
                        wk1[c] = w2[c];
                        w2[c] = lnext;  // reuse: left state of face k+3/2
                    }
                    {
                        R f[NC];
                        face_flux_states<NDIM, 2, R>(gr, lz, wr, f);
#pragma unroll
                        for (int c = 0; c < NC; ++c) fzc[c] = (FT)f[c];
                    }
#pragma unroll
                    for (int c = 0; c < NC; ++c) lz[c] = w2[c];
                }
            } else {
                double u[NC];
                load_in(boff + (long long)k * P, col32, u);
                in_to_w<NDIM, R, PRIM_IN>(gm1, u, -1, VM_NONE, wc, bad);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) sW[c][ly + 2 + RO][lx + 2] = wc[c];
        }
        if (hact) {
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(2);
            R wh[NC];
            // the halo cell of plane k: loaded one iteration ahead (HALO_PF),
            // else now
            if (!HALO_PF) load_halo(k, uhalo);
            // not checked here: every cell is checked by the tile that owns it
            in_to_w<NDIM, R, PRIM_IN, false>(gm1, uhalo, halo_vm ? hvax : -1, hvm, wh, bad);
#pragma unroll
            for (int c = 0; c < NC; ++c) sW[c][hy + 2 + RO][hx + 2] = wh[c];
            if (HALO_PF && k + 1 < z1) load_halo(k + 1, uhalo);
        }
        __syncthreads();

        if (NEED_BASE && BASE_EARLY && act) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                ubase[c] = plane_load<double, kNonTemporal>(a.base, c * N + boff + (long long)k * P, ext8, col32 * 8u);
        }
        // x faces: face i separates tile columns i-1 and i; LDS columns i..i+3
        if (ly < ay && lx <= ax) {
            R w0[NC], w1[NC], w2[NC], w3[NC], F[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                w0[c] = sW[c][ly + 2 + RO][lx];
                w1[c] = sW[c][ly + 2 + RO][lx + 1];
                w2[c] = sW[c][ly + 2 + RO][lx + 2];
                w3[c] = sW[c][ly + 2 + RO][lx + 3];
            }
            face_flux<NDIM, 0, R, FIRST>(gr, w0, w1, w2, w3, F);
#pragma unroll
            for (int c = 0; c < NC; ++c) sFx[c][ly][lx] = (FT)F[c];
        }
        if (HY && lx < ax && ly <= ay) {
            R w0[NC], w1[NC], w2[NC], w3[NC], F[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                w0[c] = sW[c][HY ? ly : 0][lx + 2];
                w1[c] = sW[c][HY ? ly + 1 : 0][lx + 2];
                w2[c] = sW[c][ly + 2 + RO][lx + 2];
                w3[c] = sW[c][HY ? ly + 3 : 0][lx + 2];
            }
            face_flux<NDIM, 1, R, FIRST>(gr, w0, w1, w2, w3, F);
#pragma unroll
            for (int c = 0; c < NC; ++c) sFy[HY ? c : 0][HY ? ly : 0][lx] = (FT)F[c];
        }
        // faces past the last thread column / row of a full tile; in 3-D the
        // x and y ones share one code path (axis chosen per lane)
        const int ex = (ax == TX) ? ay : 0;
        const int ey = (HY && ay == TY) ? ax : 0;
        for (int e = tid; e < ex + ey; e += NT) {
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(2);
            R w0[NC], w1[NC], w2[NC], w3[NC], F[NC];
            if constexpr (HY) {
                const bool yaxis = e >= ex;
                // x face (row e, column TX) or y face (row TY, column e - ex)
                const int r0 = yaxis ? TY : e + 2, c0 = yaxis ? e - ex + 2 : TX;
                const int dr = yaxis ? 1 : 0, dc = yaxis ? 0 : 1;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    w0[c] = sW[c][HY ? r0 : 0][c0];
                    w1[c] = sW[c][HY ? r0 + dr : 0][c0 + dc];
                    w2[c] = sW[c][HY ? r0 + 2 * dr : 0][c0 + 2 * dc];
                    w3[c] = sW[c][HY ? r0 + 3 * dr : 0][c0 + 3 * dc];
                }
                face_flux_xy<R, FIRST>(gr, yaxis, w0, w1, w2, w3, F);
                if (yaxis) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) sFy[c][TY][e - ex] = (FT)F[c];
                } else {
#pragma unroll
                    for (int c = 0; c < NC; ++c) sFx[c][e][TX] = (FT)F[c];
                }
            } else {
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    w0[c] = sW[c][e + 2 + RO][TX];
                    w1[c] = sW[c][e + 2 + RO][TX + 1];
                    w2[c] = sW[c][e + 2 + RO][TX + 2];
                    w3[c] = sW[c][e + 2 + RO][TX + 3];
                }
                face_flux<NDIM, 0, R, FIRST>(gr, w0, w1, w2, w3, F);
#pragma unroll
                for (int c = 0; c < NC; ++c) sFx[c][e][TX] = (FT)F[c];
            }
        }
        if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
        __syncthreads();

        if (act) {
            const long long kP = boff + (long long)k * P;  // plane offset of the cell
            const uint32_t colb = col32 * (uint32_t)sizeof(double);
            if (NEED_UIN && !RING) {
#pragma unroll
                for (int c = 0; c < NC; ++c) uin[c] = plane_load(a.in, c * N + kP, ext8, colb);
            }
            if (BASE_AHEAD) {
#pragma unroll
                for (int c = 0; c < NC; ++c) ubase[c] = uahead[c];
            } else if (NEED_BASE && !BASE_EARLY) {
#pragma unroll
                for (int c = 0; c < NC; ++c) ubase[c] = plane_load<double, kNonTemporal>(a.base, c * N + kP, ext8, colb);
            }
            double unew[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                // the axis terms summed in x, y, z order from the first one
                // (a sum of two rounded products is the same either way round,
                // so interchanging two axes leaves the update bitwise unchanged)
                double acc = lam0 * ((double)sFx[c][ly][lx] - (double)sFx[c][ly][lx + 1]);
                if (HY)
                    acc = acc + lam1 * ((double)sFy[HY ? c : 0][HY ? ly : 0][lx] -
                                        (double)sFy[HY ? c : 0][HY ? ly + 1 : 0][lx]);
                if (HZ) acc = acc + lam2 * ((double)fzb[c] - (double)fzc[c]);
                double r;
                if (MODE == MODE_RHS)
                    r = acc;
                else if (MODE == MODE_STAGE1 || PRED)
                    r = uin[c] + acc;
                else if (CORR)
                    r = ubase[c] + acc;
                else
                    r = 0.5 * ubase[c] + 0.5 * (uin[c] + acc);
                if (!PRIM_OUT && !BASE_AHEAD)
                    plane_store<double, EPILOGUE ? kNonTemporal : 0>(a.out, c * N + kP, ext8, colb, r);
                unew[c] = r;
            }
            if (BASE_AHEAD) {
                if (k + 1 < z1) load_ahead(k + 1);
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    plane_store<double, EPILOGUE ? kNonTemporal : 0>(a.out, c * N + kP, ext8, colb, unew[c]);
            }
            if (PRIM_OUT) {
                // the predicted state is kept only as primitive variables of type R
                double w[NC];
                bad |= !cons_to_prim<NDIM>(gm1, unew, w);
                R* wout = reinterpret_cast<R*>(a.out);
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    plane_store(wout, c * N + kP, extR, col32 * (uint32_t)sizeof(R), (R)w[c]);
            }
            bool final_value = true;
            if (LEVELS) {
                const int at[3] = {x0 + lx, y0 + ly, k};
#pragma unroll
                for (int ax = 0; ax < 3; ++ax)
                    if (ax == 0 || (ax == 1 && HY) || (ax == 2 && HZ))
                        final_value = final_value && jump_slot(g, a.side, a.nres, blk, ax, at[ax]) < 0;
            }
            if (EPILOGUE && a.want_dt && final_value) {
                double w[NC];
                bad_new |= !cons_to_prim<NDIM>(gm1, unew, w);
                const double cr = cfl_rate<NDIM>(g, w);
                rate = cr > rate ? cr : rate;
            }
        }
        if (HZ && act) {
#pragma unroll
            for (int c = 0; c < NC; ++c) fzb[c] = fzc[c];
        }
    };

    for (int k = z0; k < z1; ++k) plane(k);

    if (bad || (bad_new && a.use_device_dt)) atomicOr(&a.ctrl->flags, FLAG_NONPHYSICAL);
    if (EPILOGUE && a.want_dt) {
        // a host-dt step's new state is not looked at until its dt is asked for
        if (bad_new && !a.use_device_dt) atomicOr(&a.ctrl->pend_flags, FLAG_NONPHYSICAL);
        __shared__ double red[NT / 64 > 0 ? NT / 64 : 1];
        rate = wave_max(rate);
        if ((tid & 63) == 0) red[tid >> 6] = rate;
        __syncthreads();
        if (tid == 0) {
            double m = red[0];
            for (int i = 1; i < NT / 64; ++i) m = red[i] > m ? red[i] : m;
            add_rate(a.ctrl, par, LEVELS ? __builtin_ldexp(m, lev) : m);
        }
    }
}

template <int NDIM, typename R, int MODE, int TX, int TY, bool FEW>
__global__ __launch_bounds__(TX * TY)
__attribute__((amdgpu_waves_per_eu(StageOccupancy<NDIM, R, MODE, FEW>::kWaves, StageOccupancy<NDIM, R, MODE, FEW>::kWavesMax)))
void stage_kernel(StageArgs a) {
    if (!a.chain && a.use_device_dt && a.ctrl->done) return;  // uniform over the grid
    // work-group -> (block, work-group within the block), block after block:
    // each XCD's contiguous range of work-groups covers whole blocks (measured
    // faster than taking them in the order of the whole mesh's tile grid)
    int wg = xcd_remap(blockIdx.x, gridDim.x);
    int blk = a.blk0;
    if (a.nblk > 1) {
        const int per = a.tiles_x * a.tiles_y * a.chunks_z;
        const int q = wg / per;
        blk += q;
        wg -= q * per;
    }
    stage_body<NDIM, R, MODE, TX, TY, FEW>(a, wg, blk, blockIdx.x == 0);
}

// Batched stage: work-group -> (member, work-group of the member) from a
// table; members that reached their run limit are skipped.
template <int NDIM, typename R, int MODE, int TX, int TY, bool FEW>
__global__ __launch_bounds__(TX * TY)
__attribute__((amdgpu_waves_per_eu(StageOccupancy<NDIM, R, MODE, FEW>::kWaves, StageOccupancy<NDIM, R, MODE, FEW>::kWavesMax)))
void stage_kernel_batch(
    const MeshDesc* __restrict__ descs, const int2* __restrict__ blk) {
    const int2 e = blk[xcd_remap(blockIdx.x, gridDim.x)];
    const MeshDesc& d = descs[e.x];
    StageArgs a{};  // every field set: a batch member is one unrefined block
    a.ctrl = d.ctrl;
    a.geo = d.geo;
    a.dt_host = 0.0;
    a.use_device_dt = 1;
    a.chain = 1;
    a.tiles_x = d.tiles_x;
    a.tiles_y = d.tiles_y;
    a.chunks_z = d.chunks_z;
    a.kz = d.kz;
    a.blk0 = 0;
    a.nblk = 1;
    a.conc = 1;
    a.side = nullptr;
    a.gbuf = nullptr;
    a.gcs = 0;
    if (MODE == MODE_STAGE1 || MODE == MODE_VL2_PRED) {
        a.in = d.U;
        a.base = d.U;
        a.out = d.U1;  // van Leer: the predicted primitive state, type R
        a.want_dt = 0;
    } else {
        a.in = d.U1;
        a.base = d.U;
        a.out = d.U;
        a.want_dt = 1;
    }
    stage_body<NDIM, R, MODE, TX, TY, FEW>(a, e.y, 0, e.y == 0);
}

// ------------------------------------------------- 1-D meshes of one work-group

// nsteps device-dt steps of a 1-D mesh in one work-group, one cell a thread.
// What bounds such a mesh is not work but launches (a step of two stage
// launches takes 9.7 us from 64 to 10^5 cells) and then latency: here the state
// stays in registers and the primitive variables of both stages in LDS, a
// thread computes both faces of its cell (the two Riemann solves overlap, and
// no flux has to be exchanged), and the rate's reduction shares the barrier of
// the next step's first stage, so a step has two barriers.  A step takes
// 2.7 us at 256 cells and 7.4 us at 1024 in FP64 (2.3 and 5.3 us mixed).
// Every face and update is the arithmetic of the stage kernels: the states are
// theirs bit for bit.
template <typename R, bool VL2>
__global__ __launch_bounds__(kRun1dMost) void run_1d_kernel(Geo g, double* __restrict__ U, Ctrl* ctrl, int nsteps) {
    constexpr int NC = 3, NW = kRun1dMost / 64;
    // two stages' primitive variables; cell i at i + 2
    __shared__ R sW[2][NC][kRun1dMost + 4];
    __shared__ double sRate[NW];
    const int n = g.n[0], i = threadIdx.x, waves = blockDim.x / 64;
    const bool act = i < n;
    const double gm1 = g.gamma - 1.0;
    const Gas<R> gr = make_gas<R>(g.gamma);
    const Links none = block_links(g, 0);  // one block: a periodic side links to itself
    // ghosts -2, -1, n, n + 1: the cell each copies and its velocity's treatment
    int src[4], vmode[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int db, sl;
        src[q] = resolve(g, none, 0, q < 2 ? q - 2 : n + q - 2, vmode[q], db, sl);
    }
    double u[NC], u1[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) u[c] = act ? U[c * g.ncells + i] : 0.0;
    bool bad = false;
    auto publish = [&](int b, const R (&w)[NC]) {
#pragma unroll
        for (int c = 0; c < NC; ++c) sW[b][c][i + 2] = w[c];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (src[q] == i) {
                const int at = q < 2 ? q : n + q;
#pragma unroll
                for (int c = 0; c < NC; ++c) sW[b][c][at] = c == 1 ? (R)apply_vmode((double)w[c], vmode[q]) : w[c];
            }
    };
    // the cell's flux difference from the states in buffer b
    auto difference = [&](auto first, int b, double (&d)[NC]) {
        constexpr bool FIRST = decltype(first)::value;
        R w[5][NC], fl[NC], fr[NC];
#pragma unroll
        for (int q = 0; q < 5; ++q)
#pragma unroll
            for (int c = 0; c < NC; ++c) w[q][c] = sW[b][c][i + q];
        face_flux<1, 0, R, FIRST>(gr, w[0], w[1], w[2], w[3], fl);
        face_flux<1, 0, R, FIRST>(gr, w[1], w[2], w[3], w[4], fr);
#pragma unroll
        for (int c = 0; c < NC; ++c) d[c] = (double)fl[c] - (double)fr[c];
    };
    Ctrl k = *ctrl;
    double rate = wave_max(load_slot(ctrl, k.par));
    for (int s = 0;; ++s) {
        if (act) {
            R w[NC];
            to_prim<1, R>(gm1, u, -1, VM_NONE, w, bad);
            publish(0, w);
        }
        __syncthreads();
        // the fluxes need no time step: ahead of the books of the last one, they
        // overlap its divisions (after the last step they go unused)
        double d[NC];
        if (act) difference(std::integral_constant<bool, VL2>{}, 0, d);
        if (s > 0) {
            rate = sRate[0];
            for (int q = 1; q < waves; ++q) rate = sRate[q] > rate ? sRate[q] : rate;
        }
        if (k.pend == kPendStep) finalize_step(&k, g.cfl, rate);
        if (k.pend == kPendRate) {
            k.dt_raw = g.cfl / rate;
            k.flags |= k.pend_flags;
        }
        k.pend = kPendStep;
        if (s == nsteps || k.done) break;
        const double dt = device_dt(&k);
        const double lam = (VL2 ? 0.5 * dt : dt) / g.dx[0], lam2 = dt / g.dx[0];
        if (act) {
            R w[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) u1[c] = u[c] + lam * d[c];
            if (VL2) {
                double wd[NC];
                bad |= !cons_to_prim<1>(gm1, u1, wd);
#pragma unroll
                for (int c = 0; c < NC; ++c) w[c] = (R)wd[c];
            } else {
                to_prim<1, R>(gm1, u1, -1, VM_NONE, w, bad);
            }
            publish(1, w);
        }
        __syncthreads();
        double best = 0.0;
        if (act) {
            double w[NC];
            difference(std::false_type{}, 1, d);
#pragma unroll
            for (int c = 0; c < NC; ++c) u[c] = VL2 ? u[c] + lam2 * d[c] : 0.5 * u[c] + 0.5 * (u1[c] + lam2 * d[c]);
            bad |= !cons_to_prim<1>(gm1, u, w);
            const double cr = cfl_rate<1>(g, w);
            best = cr > best ? cr : best;
        }
        best = wave_max(best);
        if ((i & 63) == 0) sRate[i >> 6] = best;
    }
    if (act)
#pragma unroll
        for (int c = 0; c < NC; ++c) U[c * g.ncells + i] = u[c];
    if (bad) atomicOr(&ctrl->flags, FLAG_NONPHYSICAL);
    // every wave has read the control block and the slots (the barriers above)
    if (i < 64) *rate_slot(ctrl, i / kRateSlots, i % kRateSlots) = 0ull;
    if (i == 0) {
        ctrl->dt_raw = k.dt_raw;
        ctrl->dt_valid = 1;
        ctrl->t = k.t;
        ctrl->steps = k.steps;
        ctrl->done = k.done;
        if (k.flags) atomicOr(&ctrl->flags, k.flags);
        ctrl->pend = kPendNone;
        ctrl->pend_flags = 0;
    }
}

// ------------------------------------------------------------- small kernels

// m_d = rho v_d, E = p/(gamma - 1) + (1/2) sum_d m_d v_d
template <int NDIM>
__device__ __forceinline__ void prim_to_cons_cell(double gamma, const double (&w)[NDIM + 2], double (&u)[NDIM + 2]) {
    double ke2 = 0.0;
    u[0] = w[0];
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        const double mom = w[0] * w[1 + d];
        u[1 + d] = mom;
        ke2 = ke2 + mom * w[1 + d];
    }
    u[NDIM + 1] = w[NDIM + 1] / (gamma - 1.0) + 0.5 * ke2;
}

// Geometry of block blk: a refined mesh's blocks of level L (from the level
// starts) have inverse cell widths of level 0's times 2^L (exact: 1 / (dx
// 2^-L) rounds to (1 / dx) 2^L).
__device__ __forceinline__ Geo block_geo(const Geo& g0, const LevelStarts& starts, int blk) {
    Geo g = g0;
    const int lev = block_level(starts, blk);
#pragma unroll
    for (int k = 0; k < 3; ++k) g.inv_dx[k] = __builtin_ldexp(g0.inv_dx[k], lev);
    return g;
}

// Largest rate of a work-group of four waves into the slots.
__device__ __forceinline__ void block_rate(Ctrl* ctrl, double best) {
    __shared__ double red[4];
    best = wave_max(best);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = red[0];
        for (int i = 1; i < 4; ++i) m = red[i] > m ? red[i] : m;
        add_rate(ctrl, ctrl->par, m);
    }
}

// blockIdx.y: the block of the mesh (block layout); a refined mesh's blocks
// of level L (from the level starts) take level 0's cell widths times 2^-L
template <int NDIM>
__global__ __launch_bounds__(256) void dt_kernel(Geo g0, LevelStarts starts, const double* __restrict__ U,
                                                 Ctrl* ctrl) {
    constexpr int NC = NDIM + 2;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) ctrl->pend = kPendRate;
    const Geo g = block_geo(g0, starts, blockIdx.y);
    U += (long long)blockIdx.y * NC * g.ncells;
    double best = 0.0;
    bool bad = false;
    for (long long cell = (long long)blockIdx.x * blockDim.x + threadIdx.x; cell < g.ncells;
         cell += (long long)gridDim.x * blockDim.x) {
        double u[NC], w[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) u[c] = U[c * g.ncells + cell];
        bad |= !cons_to_prim<NDIM>(g.gamma - 1.0, u, w);
        const double cr = cfl_rate<NDIM>(g, w);
        best = cr > best ? cr : best;
    }
    if (bad) atomicOr(&ctrl->flags, FLAG_NONPHYSICAL);
    block_rate(ctrl, best);
}

// Use the rate in the slots (pend: what for) and clear both sets; one wave.
// Latency bound (a chain of two loads at most): each lane takes one slot of
// both sets, and the block is read whole beside them.
__device__ __forceinline__ void finalize_ctrl(Ctrl* c, int op, double cfl) {
    const unsigned int set = threadIdx.x / kRateSlots;
    unsigned long long* slot = rate_slot(c, set, threadIdx.x % kRateSlots);
    const double mine = __longlong_as_double((long long)*slot);
    Ctrl k;
    k.dt_raw = c->dt_raw;
    k.t = c->t;
    k.pend = c->pend;
    k.par = c->par;
    k.flags = c->flags;
    k.dt_valid = c->dt_valid;
    k.steps = c->steps;
    k.t_end = c->t_end;
    k.max_steps = c->max_steps;
    k.done = c->done;
    k.pend_flags = c->pend_flags;
    const double rate = wave_max(set == k.par ? mine : 0.0);
    *slot = 0ull;
    if (op == CTRL_FINALIZE_STEP) k.pend = kPendStep;
    if (k.pend == kPendStep) finalize_step(&k, cfl, rate);
    if (k.pend == kPendRate) {
        k.dt_raw = cfl / rate;
        k.dt_valid = 1;
        k.flags |= k.pend_flags;
    }
    if (threadIdx.x != 0) return;
    c->dt_raw = k.dt_raw;
    c->t = k.t;
    c->flags = k.flags;
    c->dt_valid = k.dt_valid;
    c->steps = k.steps;
    c->done = k.done;
    c->pend = kPendNone;
    c->pend_flags = 0;
}

__global__ __launch_bounds__(64) void ctrl_kernel(Ctrl* c, int op, double a0, double a1, double cfl) {
    static_assert(2 * kRateSlots == 64, "one wave clears both sets of slots");
    if (op == CTRL_FINALIZE || op == CTRL_FINALIZE_STEP) {
        finalize_ctrl(c, op, cfl);
        return;
    }
    // these leave nothing pending (a replayed host-dt step may meet a state
    // whose rate is)
    if (op == CTRL_INIT || op == CTRL_ADVANCE_T || op == CTRL_DROP_RATE)
        *rate_slot(c, threadIdx.x / kRateSlots, threadIdx.x % kRateSlots) = 0ull;
    if (threadIdx.x != 0) return;
    switch (op) {
        case CTRL_INIT:
            c->t = a0;
            c->steps = 0;
            c->flags = 0;
            c->dt_valid = 0;
            c->dt_raw = 0.0;
            c->pend = kPendNone;
            c->par = 0;
            c->pend_flags = 0;
            c->t_end = 0.0;
            c->max_steps = 0ull;
            c->done = 0;
            break;
        case CTRL_ADVANCE_T:
            c->t = c->t + a0;
            c->steps += 1;
            c->dt_valid = 0;
            c->pend = kPendNone;
            c->pend_flags = 0;
            break;
        case CTRL_DROP_RATE:
            c->pend = kPendNone;
            c->pend_flags = 0;
            break;
        case CTRL_SET_LIMITS:
            c->t_end = a0;
            c->max_steps = a1 > 0.0 ? c->steps + (unsigned long long)a1 : 0ull;
            update_done(c);
            break;
        default:
            break;
    }
}

// Status of every batch member (done, flags, steps) into one table.
__global__ void status_gather_kernel(const MeshDesc* __restrict__ d, int n, unsigned long long* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const Ctrl* c = d[i].ctrl;
        out[3 * i] = c->done;
        out[3 * i + 1] = c->flags;
        out[3 * i + 2] = c->steps;
    }
}

// One wave per member.
__global__ __launch_bounds__(64) void ctrl_batch_kernel(const MeshDesc* __restrict__ d) {
    finalize_ctrl(d[blockIdx.x].ctrl, CTRL_FINALIZE, d[blockIdx.x].geo.cfl);
}

// Neumaier-compensated accumulator combined pairwise in a fixed tree.
struct Comp {
    double s, c;
};
__device__ __forceinline__ Comp comp_add(Comp a, double x) {
    const double t = a.s + x;
    if (dabs(a.s) >= dabs(x))
        a.c += (a.s - t) + x;
    else
        a.c += (x - t) + a.s;
    a.s = t;
    return a;
}
__device__ __forceinline__ Comp comp_merge(Comp a, Comp b) {
    Comp r = comp_add(a, b.s);
    r.c += b.c;
    return r;
}

// blockIdx.y: the block of the mesh (block layout); one partial per work-group
template <int NC>
__global__ __launch_bounds__(256) void totals_pass1(long long ncells, const double* __restrict__ U,
                                                    double* __restrict__ parts) {
    __shared__ double ss[NC][256], sc[NC][256];
    U += (long long)blockIdx.y * NC * ncells;
    parts += (long long)blockIdx.y * gridDim.x * NC * 2;
    const long long per = (ncells + gridDim.x - 1) / gridDim.x;
    const long long lo = (long long)blockIdx.x * per;
    const long long hi = lo + per < ncells ? lo + per : ncells;
    Comp acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = Comp{0.0, 0.0};
    for (long long i = lo + threadIdx.x; i < hi; i += 256)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = comp_add(acc[c], U[c * ncells + i]);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        ss[c][threadIdx.x] = acc[c].s;
        sc[c][threadIdx.x] = acc[c].c;
    }
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                Comp r = comp_merge(Comp{ss[c][threadIdx.x], sc[c][threadIdx.x]},
                                    Comp{ss[c][threadIdx.x + w], sc[c][threadIdx.x + w]});
                ss[c][threadIdx.x] = r.s;
                sc[c][threadIdx.x] = r.c;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            parts[(blockIdx.x * NC + c) * 2] = ss[c][0];
            parts[(blockIdx.x * NC + c) * 2 + 1] = sc[c][0];
        }
}

// The fixed tree over the partials.  out == null: the (sum, compensation)
// pairs go to sums[2 c], sums[2 c + 1]; else out[c] = dV (sum + compensation).
template <int NC>
__global__ __launch_bounds__(256) void totals_pass2(int nparts, const double* __restrict__ parts,
                                                    double* __restrict__ sums, double* __restrict__ out,
                                                    double dV) {
    __shared__ double ss[NC][256], sc[NC][256];
    Comp acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = Comp{0.0, 0.0};
    for (int p = threadIdx.x; p < nparts; p += 256)
#pragma unroll
        for (int c = 0; c < NC; ++c)
            acc[c] = comp_merge(acc[c], Comp{parts[(p * NC + c) * 2], parts[(p * NC + c) * 2 + 1]});
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        ss[c][threadIdx.x] = acc[c].s;
        sc[c][threadIdx.x] = acc[c].c;
    }
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                Comp r = comp_merge(Comp{ss[c][threadIdx.x], sc[c][threadIdx.x]},
                                    Comp{ss[c][threadIdx.x + w], sc[c][threadIdx.x + w]});
                ss[c][threadIdx.x] = r.s;
                sc[c][threadIdx.x] = r.c;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (out) {
                out[c] = dV * (ss[c][0] + sc[c][0]);
            } else {
                sums[2 * c] = ss[c][0];
                sums[2 * c + 1] = sc[c][0];
            }
        }
}

// m_d = rho v_d, E = p/(gamma - 1) + (1/2) sum_d m_d v_d, and the CFL rate of
// the conserved state, left pending for the first time step: one pass over
// the state instead of three.  1024 work-groups, each with the next cells'
// values on their way: the passes of a larger grid end in more work-groups'
// reductions and atomics than they hide.  A state set and its dt read back
// take 273 us at 256^3 and 38 us at 1024^2 (as passes of their own 398 and
// 66, with 4096 work-groups without the early loads 287 and 40); a state set
// alone 252 and 16 us (the conversion alone 244 and 15, with 4096 268 and 19).
// W and U may be the same array (each cell is read before it is written);
// blockIdx.y: the block of the mesh (block layout); MESH: W is in the mesh
// layout of a uniform block grid.
template <int NDIM, bool MESH>
__global__ __launch_bounds__(256) void prim_to_cons_kernel(Geo g0, LevelStarts starts, const double* W, double* U,
                                                           Ctrl* ctrl) {
    constexpr int NC = NDIM + 2;
    const Geo g = block_geo(g0, starts, blockIdx.y);
    const int blk = blockIdx.y;
    const long long N = g.ncells;
    // component stride and the block's first cell in W
    long long ws = N, w0 = (long long)blk * NC * N;
    long long row = g.n[0], plane = (long long)g.n[0] * g.n[1];
    if (MESH) {
        row = (long long)g.n[0] * g.blocks[0];
        plane = row * g.n[1] * g.blocks[1];
        ws = plane * g.n[2] * g.blocks[2];
        w0 = (long long)(blk % g.blocks[0]) * g.n[0] +
             (long long)((blk / g.blocks[0]) % g.blocks[1]) * g.n[1] * row +
             (long long)(blk / (g.blocks[0] * g.blocks[1])) * g.n[2] * plane;
    }
    W += w0;
    U += (long long)blk * NC * N;
    double best = 0.0;
    bool bad = false;
    // the primitive state of a cell
    auto load = [&](long long cell, double(&w)[NC]) {
        long long q = cell;
        if (MESH) {
            const long long r = cell / g.n[0];
            q = cell % g.n[0] + (r % g.n[1]) * row + (r / g.n[1]) * plane;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) w[c] = W[c * ws + q];
    };
    const long long step = (long long)gridDim.x * blockDim.x;
    long long cell = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    double next[NC];
    if (cell < N) load(cell, next);
    for (; cell < N; cell += step) {
        double w[NC], u[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) w[c] = next[c];
        if (cell + step < N) load(cell + step, next);
        prim_to_cons_cell<NDIM>(g.gamma, w, u);
#pragma unroll
        for (int c = 0; c < NC; ++c) U[c * N + cell] = u[c];
        bad |= !cons_to_prim<NDIM>(g.gamma - 1.0, u, w);
        const double cr = cfl_rate<NDIM>(g, w);
        best = cr > best ? cr : best;
    }
    // looked at once the dt is asked for
    if (bad) atomicOr(&ctrl->pend_flags, FLAG_NONPHYSICAL);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) ctrl->pend = kPendRate;
    block_rate(ctrl, best);
}

// Padded primitive export: physical padded layout [c][K][J][I] with two ghost
// layers on every active physical axis, corners zero.
template <int NDIM, typename R>
__global__ __launch_bounds__(256) void padded_prim_kernel(Geo g, const double* __restrict__ U,
                                                          double* __restrict__ Wp, Ctrl* ctrl) {
    constexpr int NC = NDIM + 2;
    // physical extents of the mesh: axis p of NDIM -> kernel axis (3-D
    // identity; 2-D y is kernel z)
    const int m0 = g.n[0] * g.blocks[0], m1 = g.n[1] * g.blocks[1], m2 = g.n[2] * g.blocks[2];
    int nph[3] = {m0, NDIM == 3 ? m1 : (NDIM == 2 ? m2 : 1), NDIM == 3 ? m2 : 1};
    int P[3];
    for (int d = 0; d < 3; ++d) P[d] = nph[d] + (d < NDIM ? 4 : 0);
    const long long total = (long long)P[0] * P[1] * P[2];
    bool bad = false;
    for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < total;
         q += (long long)gridDim.x * blockDim.x) {
        const int I = (int)(q % P[0]);
        const int J = (int)((q / P[0]) % P[1]);
        const int K = (int)(q / ((long long)P[0] * P[1]));
        int pc[3] = {I - (NDIM >= 1 ? 2 : 0), J - (NDIM >= 2 ? 2 : 0), K - (NDIM >= 3 ? 2 : 0)};
        int outside = 0;
        for (int d = 0; d < NDIM; ++d) outside += (pc[d] < 0 || pc[d] >= nph[d]);
        double out[NC];
        if (outside > 1) {
            for (int c = 0; c < NC; ++c) out[c] = 0.0;
        } else {
            R w[NC];
            int kx = pc[0], ky = NDIM == 3 ? pc[1] : 0, kzc = NDIM == 3 ? pc[2] : (NDIM == 2 ? pc[1] : 0);
            load_w<NDIM, R>(g, U, kx, ky, kzc, w, bad);
            for (int c = 0; c < NC; ++c) out[c] = (double)w[c];
        }
        for (int c = 0; c < NC; ++c) Wp[c * total + q] = out[c];
    }
    if (bad) atomicOr(&ctrl->flags, FLAG_NONPHYSICAL);
}

// ------------------------------------------------------- static refinement

// The two transverse kernel axes of a side of kernel axis ax (lower first).
__device__ __forceinline__ void transverse(int ax, int& lo, int& hi) {
    lo = ax == 0 ? 1 : 0;
    hi = ax == 2 ? 1 : 2;
}

// Element i (a run-time index) of an array, by selects: indexing the array
// itself would place it in private memory.
__device__ __forceinline__ int at3(const int (&a)[3], int i) { return i == 0 ? a[0] : (i == 1 ? a[1] : a[2]); }

// Where the conserved values of a refined mesh's cell lie (component c at
// p[c * cs]), and the boundary treatment of its velocity (vax, vm).
struct CellRef {
    const double* p;
    long long cs;
    int vax, vm;
};

// Cell (x, y, z) of block blk, at most one coordinate outside the block (by up
// to two cells): through the block's side codes, in a neighbouring block, by a
// mesh face's boundary rule, or in a ghost slot.  The address alone, so that a
// caller has the loads of all its cells in flight at once (read one after
// another behind these branches, the seven cells of a prolongation took 14 us,
// the eight of a flux correction 21 us).
__device__ __forceinline__ CellRef smr_cell(const Geo& g, const Links& L, const double* __restrict__ U,
                                            const double* __restrict__ gbuf, int nc, long long gcs, int blk, int x,
                                            int y, int z) {
    int c3[3] = {x, y, z};
    int b = blk, slot = -1, sax = 0, layer = 0;
    CellRef o;
    o.vax = -1;
    o.vm = VM_NONE;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        if (c3[ax] >= 0 && c3[ax] < g.n[ax]) continue;
        int db = 0, sl = -1, vm;
        const int q = resolve(g, L, ax, c3[ax], vm, db, sl);
        if (sl >= 0) {
            slot = sl;
            sax = ax;
            layer = q;
        } else {
            c3[ax] = q;
            b = blk + db;
            if (vm != VM_NONE) {
                o.vax = ax;
                o.vm = vm;
            }
        }
    }
    int lo, hi;
    transverse(sax, lo, hi);
    const long long in_slot =
        (long long)slot * nc * gcs + ((long long)layer * at3(g.n, hi) + at3(c3, hi)) * at3(g.n, lo) + at3(c3, lo);
    const long long in_block =
        (long long)b * nc * g.ncells + ((long long)c3[2] * g.n[1] + c3[1]) * g.n[0] + c3[0];
    o.p = slot >= 0 ? gbuf + in_slot : U + in_block;
    o.cs = slot >= 0 ? gcs : g.ncells;
    return o;
}

// Kernel axis of the k-th active axis (physical order: x, y, z).
template <int NDIM>
__device__ __forceinline__ constexpr int active_axis(int k) {
    return NDIM == 2 ? (k == 0 ? 0 : 2) : k;
}

// Restriction onto the two ghost layers of a coarse block's side that faces
// finer blocks: each ghost is the volume average of the 2^NDIM fine cells it
// covers (pairwise means along x, then y, then z), on primitive variables;
// stored as conserved values.  The fine cells lie inside their blocks, so they
// are read where they are.  blockIdx.x: the slot; one thread per ghost.
// Latency bound (a few hundred waves); reading through the side codes and a
// private copy of the task it took 16 us for 24 slots of 32 x 32 faces.
template <int NDIM>
__global__ __launch_bounds__(64) void smr_restrict_kernel(Geo g, const double* __restrict__ U,
                                                           double* __restrict__ gbuf, long long gcs,
                                                           const GhostTask* __restrict__ tasks, Ctrl* ctrl) {
    constexpr int NC = NDIM + 2;
    constexpr int K = 1 << NDIM;
    const GhostTask& t = tasks[blockIdx.x];
    const int tax = t.ax, ts = t.s;
    int lo, hi;
    transverse(tax, lo, hi);
    const int nlo = at3(g.n, lo), nhi = at3(g.n, hi), face = nlo * nhi;
    bool bad = false;
    const int q = blockIdx.y * blockDim.x + threadIdx.x;
    if (q < 2 * face) {
        const int layer = q / face, r = q - layer * face;
        const int tl = r % nlo, th = r / nlo;
        double u[K][NC], v[NC][K];
#pragma unroll
        for (int o = 0; o < K; ++o) {
            int x3[3] = {0, 0, 0};
            int cb[3] = {0, 0, 0};  // child offsets on the transverse axes
#pragma unroll
            for (int k = 0; k < NDIM; ++k) {
                const int ax = active_axis<NDIM>(k);
                const int off = (o >> k) & 1;
                if (ax == tax) {
                    // fine cells 2 layer, 2 layer + 1 in from the face (off 0: the lower)
                    x3[ax] = ts ? 2 * layer + off : g.n[ax] - 2 - 2 * layer + off;
                } else {
                    const int p = 2 * (ax == lo ? tl : th) + off;  // from the refined root's origin
                    cb[ax] = p >= g.n[ax] ? 1 : 0;
                    x3[ax] = p - cb[ax] * g.n[ax];
                }
            }
            const int fb = t.src[at3(cb, lo) + 2 * at3(cb, hi)];
            const double* F = U + (long long)fb * NC * g.ncells + ((long long)x3[2] * g.n[1] + x3[1]) * g.n[0] + x3[0];
#pragma unroll
            for (int c = 0; c < NC; ++c) u[o][c] = F[c * g.ncells];
        }
#pragma unroll
        for (int o = 0; o < K; ++o) {
            double w[NC];
            to_prim<NDIM, double>(g.gamma - 1.0, u[o], -1, VM_NONE, w, bad);
#pragma unroll
            for (int c = 0; c < NC; ++c) v[c][o] = w[c];
        }
        double w[NC], uc[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            // pairwise means: along x first (bit 0), then y, then z
#pragma unroll
            for (int k = 0; k < NDIM; ++k)
#pragma unroll
                for (int i = 0; i < (K >> (k + 1)); ++i) v[c][i] = 0.5 * (v[c][2 * i] + v[c][2 * i + 1]);
            w[c] = v[c][0];
        }
        prim_to_cons_cell<NDIM>(g.gamma, w, uc);
        const long long o = (long long)t.slot * NC * gcs + (long long)layer * face + r;
#pragma unroll
        for (int c = 0; c < NC; ++c) gbuf[o + c * gcs] = uc[c];
    }
    if (bad) atomicOr(&ctrl->flags, FLAG_NONPHYSICAL);
}

// Prolongation onto the two ghost layers of a fine block's side that faces a
// coarser block: the coarse cell's value plus, per axis, a quarter of its
// minmod-limited difference (eq. minmod), signed by the side of the coarse
// centre the ghost's centre lies on; the coarse block's own ghosts (same
// level, boundary rule, restricted slots) complete its stencil.  Primitive
// variables; stored as conserved values.  blockIdx.x: the slot; one thread
// per coarse cell, which holds both layers and 2^(NDIM-1) ghosts of each: they
// share its stencil of 2 NDIM + 1 cells (a thread per ghost loaded and
// converted it eight times over in 3-D, 36 us for 96 slots of 32 x 32 faces).
template <int NDIM>
__global__ __launch_bounds__(64) void smr_prolong_kernel(Geo g, const double* __restrict__ U,
                                                          const int* __restrict__ side, double* __restrict__ gbuf,
                                                          long long gcs, const GhostTask* __restrict__ tasks,
                                                          Ctrl* ctrl) {
    constexpr int NC = NDIM + 2;
    const GhostTask& t = tasks[blockIdx.x];
    const int tax = t.ax, ts = t.s;
    int lo, hi;
    transverse(tax, lo, hi);
    const int nlo = at3(g.n, lo), nhi = at3(g.n, hi), face = nlo * nhi;
    // coarse cells across the side (an axis of one cell is inactive)
    const int mlo = nlo > 1 ? nlo / 2 : 1, mhi = nhi > 1 ? nhi / 2 : 1;
    const int cblk = t.src[0];
    const Links L = table_links(side, cblk);
    bool bad = false;
    const int q = blockIdx.y * blockDim.x + threadIdx.x;
    if (q < mlo * mhi) {
        const int tl = q % mlo, th = q / mlo;
        int ci[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < NDIM; ++k) {
            const int ax = active_axis<NDIM>(k);
            // the coarse cell next to the face; across it, counted from the parent's origin
            if (ax == tax)
                ci[ax] = ts ? 0 : g.n[ax] - 1;
            else
                ci[ax] = t.child[ax] * (g.n[ax] / 2) + (ax == lo ? tl : th);
        }
        // the cell and its neighbours below and above on each axis
        CellRef at[2 * NDIM + 1];
        at[0] = smr_cell(g, L, U, gbuf, NC, gcs, cblk, ci[0], ci[1], ci[2]);
#pragma unroll
        for (int k = 0; k < NDIM; ++k) {
            const int ax = active_axis<NDIM>(k);
            int a3[3] = {ci[0], ci[1], ci[2]}, b3[3] = {ci[0], ci[1], ci[2]};
            a3[ax] -= 1;
            b3[ax] += 1;
            at[1 + 2 * k] = smr_cell(g, L, U, gbuf, NC, gcs, cblk, a3[0], a3[1], a3[2]);
            at[2 + 2 * k] = smr_cell(g, L, U, gbuf, NC, gcs, cblk, b3[0], b3[1], b3[2]);
        }
        double u7[2 * NDIM + 1][NC], w7[2 * NDIM + 1][NC], slope[NDIM][NC];
#pragma unroll
        for (int j = 0; j < 2 * NDIM + 1; ++j)
#pragma unroll
            for (int c = 0; c < NC; ++c) u7[j][c] = at[j].p[c * at[j].cs];
#pragma unroll
        for (int j = 0; j < 2 * NDIM + 1; ++j)
            to_prim<NDIM, double>(g.gamma - 1.0, u7[j], at[j].vax, at[j].vm, w7[j], bad);
        const double(&wc)[NC] = w7[0];
#pragma unroll
        for (int k = 0; k < NDIM; ++k)
#pragma unroll
            for (int c = 0; c < NC; ++c)
                slope[k][c] = minmod(wc[c] - w7[1 + 2 * k][c], w7[2 + 2 * k][c] - wc[c]);
#pragma unroll
        for (int o = 0; o < (1 << NDIM); ++o) {
            // bit k of o: the side of the coarse centre on the k-th active axis
            double acc[NC], u[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[c] = wc[c];
            int layer = 0, fl = 0, fh = 0;
#pragma unroll
            for (int k = 0; k < NDIM; ++k) {
                const int ax = active_axis<NDIM>(k), bit = (o >> k) & 1;
                if (ax == tax)
                    layer = ts ? bit : 1 - bit;
                else if (ax == lo)
                    fl = 2 * tl + bit;
                else
                    fh = 2 * th + bit;
                const double sg = bit ? 1.0 : -1.0;
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] = acc[c] + (0.25 * sg) * slope[k][c];
            }
            prim_to_cons_cell<NDIM>(g.gamma, acc, u);
            const long long to = (long long)t.slot * NC * gcs + (long long)layer * face + fh * nlo + fl;
#pragma unroll
            for (int c = 0; c < NC; ++c) gbuf[to + c * gcs] = u[c];
        }
    }
    if (bad) atomicOr(&ctrl->flags, FLAG_NONPHYSICAL);
}

// Flux correction at a level jump of kernel axis AX, for coarse cell x3 next
// to restriction slot t: the cell is to get factor * lam * (F_coarse - mean of
// the fine fluxes) (sign by side), so that its update uses the fine fluxes'
// mean in place of its own.  The fluxes are recomputed from the same stage
// input, ghosts and operations as in the stage kernel, so F_coarse cancels
// exactly; the correction is added to u.  A lane per fine face: 2^NT adjacent
// lanes share the coarse one (o: this lane's), so the fine fluxes run side by
// side and their mean is two exchanges.
template <int NDIM, typename R, bool FIRST, int AX>
__device__ __forceinline__ void reflux_cell(const Geo& g, const double* __restrict__ in, double factor, double dt,
                                            const int* __restrict__ side, const double* __restrict__ gbuf,
                                            long long gcs, const GhostTask& t, const int (&x3)[3], int o,
                                            double (&ucell)[NDIM + 2], bool& bad) {
    constexpr int NC = NDIM + 2;
    constexpr int NT = NDIM - 1;
    // the coarse block's cell width: level 0's times 2^-lev (exact)
    const double lam = dt / __builtin_ldexp(g.dx[AX], -t.lev);
    const Gas<R> gr = make_gas<R>(g.gamma);
    const double gm1 = g.gamma - 1.0;
    constexpr int lo = AX == 0 ? 1 : 0, hi = AX == 2 ? 1 : 2;
    const int n = g.n[AX], ts = t.s;
    // four cells across the coarse face, and across this lane's fine face (at
    // transverse child offsets o)
    CellRef at[2][4];
    {
        const Links Lc = table_links(side, t.leaf);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int c3[3] = {x3[0], x3[1], x3[2]};
            c3[AX] = ts ? n - 2 + j : -2 + j;
            at[0][j] = smr_cell(g, Lc, in, gbuf, NC, gcs, t.leaf, c3[0], c3[1], c3[2]);
        }
        int f3[3] = {0, 0, 0};
        int cb[3] = {0, 0, 0};
        int bit = 0;
#pragma unroll
        for (int k = 0; k < NDIM; ++k) {
            const int ax = active_axis<NDIM>(k);
            if (ax == AX) continue;
            const int p = 2 * x3[ax] + ((o >> bit) & 1);
            ++bit;
            cb[ax] = p >= g.n[ax] ? 1 : 0;
            f3[ax] = p - cb[ax] * g.n[ax];
        }
        const int fb = t.src[cb[lo] + 2 * cb[hi]];
        const Links Lf = table_links(side, fb);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int c3[3] = {f3[0], f3[1], f3[2]};
            c3[AX] = ts ? -2 + j : n - 2 + j;
            at[1][j] = smr_cell(g, Lf, in, gbuf, NC, gcs, fb, c3[0], c3[1], c3[2]);
        }
    }
    double u8[2][4][NC];
    R w[2][4][NC], Fc[NC], F[NC];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int c = 0; c < NC; ++c) u8[m][j][c] = at[m][j].p[c * at[m][j].cs];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            in_to_w<NDIM, R, false>(gm1, u8[m][j], at[m][j].vax, at[m][j].vm, w[m][j], bad);
    face_flux<NDIM, AX, R, FIRST>(gr, w[0][0], w[0][1], w[0][2], w[0][3], Fc);
    face_flux<NDIM, AX, R, FIRST>(gr, w[1][0], w[1][1], w[1][2], w[1][3], F);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        // pairwise means of the fine fluxes in the order of their offsets
        double mean = (double)F[c];
#pragma unroll
        for (int k = 0; k < NT; ++k) mean = 0.5 * (mean + __shfl_xor(mean, 1 << k, 64));
        const double d = ts ? ((double)Fc[c] - mean) : (mean - (double)Fc[c]);
        ucell[c] = ucell[c] + factor * (lam * d);
    }
}

// The flux corrections of a stage, after it, one launch for all axes.  A
// coarse cell next to jumps on several axes is taken by the slot of its first
// axis, which adds them in axis order.  want_dt: the CFL rate of the corrected
// cells (which the stage left out).  FIRST: the fluxes of piecewise-constant
// states (the van Leer predictor).  blockIdx.x: the slot; one thread per fine
// face.  Latency bound; recomputing and adding in one launch instead of one
// beside the stage and one per axis after it also leaves the stage alone (a
// recomputation running beside it took it from 91 to 115 us).
template <int NDIM, typename R, bool FIRST>
__global__ __launch_bounds__(64) void smr_correct_kernel(Geo g, const double* __restrict__ in,
                                                          double* __restrict__ out, double factor,
                                                          int use_device_dt, double dt_host,
                                                          const int* __restrict__ side,
                                                          const double* __restrict__ gbuf, long long gcs,
                                                          const GhostTask* __restrict__ tasks, int nres, int want_dt,
                                                          Ctrl* ctrl) {
    constexpr int NC = NDIM + 2;
    constexpr int NT = NDIM - 1;
    const StepCtl step = *ctrl_next(ctrl);  // the stage has left or used it
    if (use_device_dt && step.done) return;  // uniform over the grid
    const double dt = use_device_dt ? step.dt : dt_host;
    const GhostTask& t = tasks[blockIdx.x];
    const int tax = t.ax, leaf = t.leaf;
    int lo, hi;
    transverse(tax, lo, hi);
    const int nlo = at3(g.n, lo), face = nlo * at3(g.n, hi);
    const int q = blockIdx.y * blockDim.x + threadIdx.x, r = q >> NT, o = q & ((1 << NT) - 1);
    double rate = 0.0;
    bool bad = false, bad_new = false, mine = r < face;
    int c3[3] = {0, 0, 0}, slot[3] = {-1, -1, -1};
    if (mine) {
        const int tl = r % nlo, th = r / nlo, side_at = t.s ? at3(g.n, tax) - 1 : 0;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) c3[ax] = ax == tax ? side_at : (ax == lo ? tl : th);
#pragma unroll
        for (int k = 0; k < NDIM; ++k) {
            const int ax = active_axis<NDIM>(k);
            slot[ax] = ax == tax ? (int)blockIdx.x : jump_slot(g, side, nres, leaf, ax, c3[ax]);
            mine = mine && (slot[ax] < 0 || ax >= tax);
        }
    }
    if (mine) {
        double* cell = out + (long long)leaf * NC * g.ncells + ((long long)c3[2] * g.n[1] + c3[1]) * g.n[0] + c3[0];
        double u[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) u[c] = cell[c * g.ncells];
        if (slot[0] >= 0)
            reflux_cell<NDIM, R, FIRST, 0>(g, in, factor, dt, side, gbuf, gcs, tasks[slot[0]], c3, o, u, bad);
        if constexpr (NDIM == 3)
            if (slot[1] >= 0)
                reflux_cell<NDIM, R, FIRST, 1>(g, in, factor, dt, side, gbuf, gcs, tasks[slot[1]], c3, o, u, bad);
        if constexpr (NDIM >= 2)
            if (slot[2] >= 0)
                reflux_cell<NDIM, R, FIRST, 2>(g, in, factor, dt, side, gbuf, gcs, tasks[slot[2]], c3, o, u, bad);
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if ((c & ((1 << NT) - 1)) == o) cell[c * g.ncells] = u[c];
        if (want_dt) {
            double w[NC];
            bad_new = !cons_to_prim<NDIM>(g.gamma - 1.0, u, w);
            rate = __builtin_ldexp(cfl_rate<NDIM>(g, w), t.lev);
        }
    }
    if (bad || (bad_new && use_device_dt)) atomicOr(&ctrl->flags, FLAG_NONPHYSICAL);
    if (want_dt) {
        if (bad_new && !use_device_dt) atomicOr(&ctrl->pend_flags, FLAG_NONPHYSICAL);
        rate = wave_max(rate > 0.0 ? rate : 0.0);
        if (threadIdx.x == 0)
            atomicMax(rate_slot(ctrl, step.par, (blockIdx.x + blockIdx.y) % kRateSlots),
                      (unsigned long long)__double_as_longlong(rate));
    }
}

// Mesh layout [comp][k][j][i] <-> block layout; q runs over the mesh cells.
__global__ __launch_bounds__(256) void relayout_kernel(Geo g, int nc, double* __restrict__ mesh,
                                                       double* __restrict__ blk, int to_blocks) {
    const long long m0 = (long long)g.n[0] * g.blocks[0], m1 = (long long)g.n[1] * g.blocks[1];
    const long long total = m0 * m1 * ((long long)g.n[2] * g.blocks[2]);
    for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < total;
         q += (long long)gridDim.x * blockDim.x) {
        const int x = (int)(q % m0);
        const int y = (int)((q / m0) % m1);
        const int z = (int)(q / (m0 * m1));
        const int b = x / g.n[0] + g.blocks[0] * (y / g.n[1] + g.blocks[1] * (z / g.n[2]));
        const long long cell = ((long long)(z % g.n[2]) * g.n[1] + y % g.n[1]) * g.n[0] + x % g.n[0];
        const long long bo = (long long)b * nc * g.ncells + cell;
        for (int c = 0; c < nc; ++c) {
            if (to_blocks)
                blk[bo + c * g.ncells] = mesh[c * total + q];
            else
                mesh[c * total + q] = blk[bo + c * g.ncells];
        }
    }
}

template <typename R, int NT>
__global__ __launch_bounds__(256) void riemann_kernel(double gamma, long long n,
                                                      const double* __restrict__ WL,
                                                      const double* __restrict__ WR,
                                                      double* __restrict__ F) {
    constexpr int NC = NT + 3;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        R L[NC], Rr[NC], Fo[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            L[c] = (R)WL[c * n + i];
            Rr[c] = (R)WR[c * n + i];
        }
        hllc<R, NT>(make_gas<R>(gamma), L, Rr, Fo);
#pragma unroll
        for (int c = 0; c < NC; ++c) F[c * n + i] = (double)Fo[c];
    }
}

int grid_for(long long work, int block, int cap) {
    long long gb = (work + block - 1) / block;
    if (gb < 1) gb = 1;
    return (int)(gb < cap ? gb : cap);
}

// Work-groups of 512 threads: no more than one fits on a CU in either form.
template <int NDIM, typename R, int MODE, int TX, int TY>
constexpr bool always_few() {
    return has_few(NDIM, sizeof(R) == 8, MODE) && TX * TY > 256;
}

// What the device holds of this stage kernel at once (zero if the runtime
// cannot tell).
template <int NDIM, typename R, int MODE, int TX, int TY>
Slots stage_slots() {
    static const Slots slots = [] {
        Slots o{0, 0, (TX * TY + 63) / 64};
        int dev = 0, nb = 0;
        if (hipGetDevice(&dev) != hipSuccess) return Slots{0, 0, 0};
        if (hipDeviceGetAttribute(&o.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return Slots{0, 0, 0};
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &nb, reinterpret_cast<const void*>(&stage_kernel<NDIM, R, MODE, TX, TY, always_few<NDIM, R, MODE, TX, TY>()>),
                TX * TY, 0) !=
            hipSuccess)
            return Slots{0, 0, 0};
        o.per_cu = nb;
        return o;
    }();
    return slots;
}

// Whether a launch of the given work-groups takes the FEW form: where they put
// no more than two waves on a SIMD (eight on a CU).  With twelve the other form
// is faster (256^3 650 against 689 us for its predecessor in eight waves), but
// work-groups of 512 threads never get there: 192^3 in 32 x 16 a step 743 ->
// 708 us, in 64 x 8 771 -> 728 us.
template <int NDIM, typename R, int MODE, int TX, int TY>
bool few_waves(long long wgs) {
    if constexpr (!has_few(NDIM, sizeof(R) == 8, MODE)) return false;
    if (always_few<NDIM, R, MODE, TX, TY>()) return true;
    const Slots sl = stage_slots<NDIM, R, MODE, TX, TY>();
    return wgs * sl.waves <= 8ll * sl.cus;
}

template <int NDIM, typename R, int MODE, int TX, int TY>
hipError_t launch_stage_t(const LaunchCtx& L, hipStream_t s) {
    constexpr bool kRegular = !always_few<NDIM, R, MODE, TX, TY>();
    if (L.slots) {
        *L.slots = stage_slots<NDIM, R, MODE, TX, TY>();
    } else if (L.a) {
        StageArgs a = *L.a;
        const long long nb = (long long)a.tiles_x * a.tiles_y * a.chunks_z * a.nblk;
        if (a.nblk < 1 || nb > 0x7fffffffll) return hipErrorInvalidValue;
        auto launch = [&](auto* kernel) {
            if (L.rec) {
                L.rec->func = reinterpret_cast<const void*>(kernel);
                L.rec->grid = dim3((unsigned)nb);
                L.rec->block = dim3(TX * TY);
                L.rec->args = a;
                return hipSuccess;
            }
            hipLaunchKernelGGL(kernel, dim3((unsigned)nb), dim3(TX * TY), 0, s, a);
            return hipGetLastError();
        };
        if constexpr (has_few(NDIM, sizeof(R) == 8, MODE)) {
            // with the work-groups of the launches on the other streams
            if (few_waves<NDIM, R, MODE, TX, TY>(a.conc > a.nblk ? nb / a.nblk * a.conc : nb))
                return launch(&stage_kernel<NDIM, R, MODE, TX, TY, true>);
        }
        if constexpr (kRegular) return launch(&stage_kernel<NDIM, R, MODE, TX, TY, false>);
    } else if constexpr (MODE == MODE_RHS || MODE == MODE_STAGE2_R || MODE == MODE_VL2_PRED_C || MODE == MODE_VL2_CORR_C) {
        return hipErrorInvalidValue;  // not a batch member's stage
    } else {
        if (L.nblk <= 0) return hipSuccess;
        auto launch = [&](auto* kernel) {
            hipLaunchKernelGGL(kernel, dim3(L.nblk), dim3(TX * TY), 0, s, L.d, L.blk);
            return hipGetLastError();
        };
        if constexpr (has_few(NDIM, sizeof(R) == 8, MODE)) {
            if (few_waves<NDIM, R, MODE, TX, TY>(L.nblk))
                return launch(&stage_kernel_batch<NDIM, R, MODE, TX, TY, true>);
        }
        if constexpr (kRegular) return launch(&stage_kernel_batch<NDIM, R, MODE, TX, TY, false>);
    }
    return hipGetLastError();
}

// The van Leer stages of a refined mesh (conserved predictor) take one tile
// each: a refined handle is not autotuned.
template <int NDIM, typename R, int MODE>
hipError_t launch_stage_refined(const Tile& t, const LaunchCtx& L, hipStream_t s) {
    if (!L.a && !L.slots) return hipErrorInvalidValue;
    if constexpr (NDIM == 3) {
        if (t.tx == 32 && t.ty == 8) return launch_stage_t<NDIM, R, MODE, 32, 8>(L, s);
    } else {
        if (t.tx == 64 && t.ty == 1) return launch_stage_t<NDIM, R, MODE, 64, 1>(L, s);
    }
    return hipErrorInvalidValue;
}

template <int NDIM, typename R, int MODE>
hipError_t launch_stage_tile(const Tile& t, const LaunchCtx& L, hipStream_t s) {
    if constexpr (NDIM == 3) {
        if (t.tx == 32 && t.ty == 8) return launch_stage_t<NDIM, R, MODE, 32, 8>(L, s);
        if (t.tx == 64 && t.ty == 8) return launch_stage_t<NDIM, R, MODE, 64, 8>(L, s);
        if (t.tx == 16 && t.ty == 16) return launch_stage_t<NDIM, R, MODE, 16, 16>(L, s);
        if (t.tx == 32 && t.ty == 16) return launch_stage_t<NDIM, R, MODE, 32, 16>(L, s);
        return hipErrorInvalidValue;
    } else {
        if (t.ty != 1) return hipErrorInvalidValue;
        if (t.tx == 64) return launch_stage_t<NDIM, R, MODE, 64, 1>(L, s);
        if (t.tx == 128) return launch_stage_t<NDIM, R, MODE, 128, 1>(L, s);
        if (t.tx == 256) return launch_stage_t<NDIM, R, MODE, 256, 1>(L, s);
        return hipErrorInvalidValue;
    }
}

template <int NDIM, typename R>
hipError_t launch_stage_mode(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s) {
    switch (mode) {
        case MODE_RHS:
            if (!L.a && !L.slots) return hipErrorInvalidValue;
            return launch_stage_tile<NDIM, R, MODE_RHS>(t, L, s);
        case MODE_STAGE1: return launch_stage_tile<NDIM, R, MODE_STAGE1>(t, L, s);
        case MODE_STAGE2: return launch_stage_tile<NDIM, R, MODE_STAGE2>(t, L, s);
        case MODE_STAGE2_R:
            if (!L.a && !L.slots) return hipErrorInvalidValue;
            return launch_stage_tile<NDIM, R, MODE_STAGE2_R>(t, L, s);
        case MODE_VL2_PRED: return launch_stage_tile<NDIM, R, MODE_VL2_PRED>(t, L, s);
        case MODE_VL2_CORR: return launch_stage_tile<NDIM, R, MODE_VL2_CORR>(t, L, s);
        case MODE_VL2_PRED_C: return launch_stage_refined<NDIM, R, MODE_VL2_PRED_C>(t, L, s);
        case MODE_VL2_CORR_C: return launch_stage_refined<NDIM, R, MODE_VL2_CORR_C>(t, L, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// The stage kernels of one dimensionality and precision, each compiled as a
// translation unit of its own (HYDRO_PART 1 .. 6).
#if HYDRO_PART == 1 || HYDRO_PART == 2
namespace {
template <typename R>
hipError_t launch_run_1d(int vl2, const Geo& g, double* U, Ctrl* ctrl, int nsteps, hipStream_t s) {
    if (g.n[0] > kRun1dMost || geo_nblk(g) != 1) return hipErrorInvalidValue;
    const dim3 block((g.n[0] + 63) / 64 * 64);
    if (vl2)
        hipLaunchKernelGGL((run_1d_kernel<R, true>), dim3(1), block, 0, s, g, U, ctrl, nsteps);
    else
        hipLaunchKernelGGL((run_1d_kernel<R, false>), dim3(1), block, 0, s, g, U, ctrl, nsteps);
    return hipGetLastError();
}
}  // namespace
#endif

#if HYDRO_PART == 1
hipError_t launch_run_1d_fp64(int vl2, const Geo& g, double* U, Ctrl* ctrl, int nsteps, hipStream_t s) {
    return launch_run_1d<double>(vl2, g, U, ctrl, nsteps, s);
}
hipError_t launch_stage_1d_fp64(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s) {
    return launch_stage_mode<1, double>(mode, t, L, s);
}
#elif HYDRO_PART == 2
hipError_t launch_run_1d_mixed(int vl2, const Geo& g, double* U, Ctrl* ctrl, int nsteps, hipStream_t s) {
    return launch_run_1d<float>(vl2, g, U, ctrl, nsteps, s);
}
hipError_t launch_stage_1d_mixed(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s) {
    return launch_stage_mode<1, float>(mode, t, L, s);
}
#elif HYDRO_PART == 3
hipError_t launch_stage_2d_fp64(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s) {
    return launch_stage_mode<2, double>(mode, t, L, s);
}
#elif HYDRO_PART == 4
hipError_t launch_stage_2d_mixed(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s) {
    return launch_stage_mode<2, float>(mode, t, L, s);
}
#elif HYDRO_PART == 5
hipError_t launch_stage_3d_fp64(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s) {
    return launch_stage_mode<3, double>(mode, t, L, s);
}
#elif HYDRO_PART == 6
hipError_t launch_stage_3d_mixed(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s) {
    return launch_stage_mode<3, float>(mode, t, L, s);
}
#else

namespace {
hipError_t launch_any(int ndim, int precision, int mode, const Tile& t, const LaunchCtx& L,
                      hipStream_t s) {
    switch (2 * ndim + (precision == 0 ? 0 : 1)) {
        case 2: return launch_stage_1d_fp64(mode, t, L, s);
        case 3: return launch_stage_1d_mixed(mode, t, L, s);
        case 4: return launch_stage_2d_fp64(mode, t, L, s);
        case 5: return launch_stage_2d_mixed(mode, t, L, s);
        case 6: return launch_stage_3d_fp64(mode, t, L, s);
        case 7: return launch_stage_3d_mixed(mode, t, L, s);
        default: return hipErrorInvalidValue;
    }
}
}  // namespace

Slots stage_residency(int ndim, int precision, int mode, const Tile& t) {
    Slots o{0, 0, 0};
    LaunchCtx L{nullptr, nullptr, nullptr, 0, nullptr, &o};
    if (launch_any(ndim, precision, mode, t, L, nullptr) != hipSuccess) return Slots{0, 0, 0};
    return o;
}

int stage_kz(int precision, int mode, const Tile& t, const StageArgs& a) {
    if (t.kz > 0) return t.kz;
    int tx, ty, cz, kz;
    plan_tiles(a.geo, t, tx, ty, cz, kz);
    const MarchCols m{(long long)tx * ty * (a.conc > a.nblk ? a.conc : a.nblk), a.geo.n[2], a.nblk == 8 && !a.side};
    return auto_kz(a.geo.ndim, stage_residency(a.geo.ndim, precision, mode, t), &m, 1);
}

hipError_t launch_stage(int precision, int mode, const Tile& t, StageArgs a, hipStream_t s) {
    const Tile r{t.tx, t.ty, stage_kz(precision, mode, t, a)};
    plan_tiles(a.geo, r, a.tiles_x, a.tiles_y, a.chunks_z, a.kz);
    LaunchCtx L{&a, nullptr, nullptr, 0, nullptr, nullptr};
    return launch_any(a.geo.ndim, precision, mode, r, L, s);
}

hipError_t plan_stage_launch(int precision, int mode, const Tile& t, StageArgs a, StageLaunch* out) {
    if (!out) return hipErrorInvalidValue;
    const Tile r{t.tx, t.ty, stage_kz(precision, mode, t, a)};
    plan_tiles(a.geo, r, a.tiles_x, a.tiles_y, a.chunks_z, a.kz);
    LaunchCtx L{&a, nullptr, nullptr, 0, out, nullptr};
    return launch_any(a.geo.ndim, precision, mode, r, L, nullptr);
}

hipError_t launch_stage_batch(int ndim, int precision, int mode, const Tile& tile, const MeshDesc* d,
                              const int2* blk, int nblk, hipStream_t s) {
    if (mode == MODE_RHS) return hipErrorInvalidValue;
    LaunchCtx L{nullptr, d, blk, nblk, nullptr, nullptr};
    return launch_any(ndim, precision, mode, tile, L, s);
}

hipError_t launch_status_gather(const MeshDesc* d, int n, unsigned long long* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(status_gather_kernel, dim3((n + 255) / 256), dim3(256), 0, s, d, n, out);
    return hipGetLastError();
}

hipError_t launch_ctrl_batch(const MeshDesc* d, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(ctrl_batch_kernel, dim3(n), dim3(64), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_dt_levels(const Geo& g0, const LevelStarts& starts, int nblk, const double* U, Ctrl* ctrl,
                            hipStream_t s) {
    if (nblk < 1) return hipSuccess;
    const dim3 grid(grid_for(g0.ncells, 256, (2048 + nblk - 1) / nblk), nblk);
    switch (g0.ndim) {
        case 1: hipLaunchKernelGGL(dt_kernel<1>, grid, dim3(256), 0, s, g0, starts, U, ctrl); break;
        case 2: hipLaunchKernelGGL(dt_kernel<2>, grid, dim3(256), 0, s, g0, starts, U, ctrl); break;
        case 3: hipLaunchKernelGGL(dt_kernel<3>, grid, dim3(256), 0, s, g0, starts, U, ctrl); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_ctrl(Ctrl* c, int op, double a0, double a1, double cfl, hipStream_t s) {
    hipLaunchKernelGGL(ctrl_kernel, dim3(1), dim3(64), 0, s, c, op, a0, a1, cfl);
    return hipGetLastError();
}

namespace {
// Partials pass then the tree over them; sums or out as in totals_pass2.
hipError_t totals_launch(const Geo& g, const double* U, double* parts, int nparts, double* sums, double* out,
                         double dV, hipStream_t s) {
    // nparts partials shared out over the blocks (at least one each)
    const int nblk = geo_nblk(g);
    if (nblk > nparts) return hipErrorInvalidValue;
    const int nb = grid_for(g.ncells, 256, nparts / nblk);
    const dim3 grid(nb, nblk);
    const int np = nb * nblk;
    const int NC = g.ndim + 2;
    switch (NC) {
        case 3:
            hipLaunchKernelGGL(totals_pass1<3>, grid, dim3(256), 0, s, g.ncells, U, parts);
            hipLaunchKernelGGL(totals_pass2<3>, dim3(1), dim3(256), 0, s, np, parts, sums, out, dV);
            break;
        case 4:
            hipLaunchKernelGGL(totals_pass1<4>, grid, dim3(256), 0, s, g.ncells, U, parts);
            hipLaunchKernelGGL(totals_pass2<4>, dim3(1), dim3(256), 0, s, np, parts, sums, out, dV);
            break;
        case 5:
            hipLaunchKernelGGL(totals_pass1<5>, grid, dim3(256), 0, s, g.ncells, U, parts);
            hipLaunchKernelGGL(totals_pass2<5>, dim3(1), dim3(256), 0, s, np, parts, sums, out, dV);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_totals(const Geo& g, const double* U, double* parts, int nparts, Ctrl* ctrl,
                         hipStream_t s) {
    return totals_launch(g, U, parts, nparts, ctrl->sums, nullptr, 0.0, s);
}

hipError_t launch_totals_out(const Geo& g, const double* U, double* parts, int nparts, double* out, double dV,
                             hipStream_t s) {
    if (!out) return hipErrorInvalidValue;
    return totals_launch(g, U, parts, nparts, nullptr, out, dV, s);
}

hipError_t launch_prim_to_cons(const Geo& g0, const LevelStarts& starts, int nblk, const double* W, double* U,
                               int mesh_layout, Ctrl* ctrl, hipStream_t s) {
    const dim3 grid(grid_for(g0.ncells, 256, (1024 + nblk - 1) / nblk), nblk);
#define PC(ND, M) hipLaunchKernelGGL((prim_to_cons_kernel<ND, M>), grid, dim3(256), 0, s, g0, starts, W, U, ctrl)
    switch (2 * g0.ndim + (mesh_layout ? 1 : 0)) {
        case 2: PC(1, false); break;
        case 3: PC(1, true); break;
        case 4: PC(2, false); break;
        case 5: PC(2, true); break;
        case 6: PC(3, false); break;
        case 7: PC(3, true); break;
        default: return hipErrorInvalidValue;
    }
#undef PC
    return hipGetLastError();
}

hipError_t launch_relayout(const Geo& g, double* mesh, double* blk, int to_blocks, hipStream_t s) {
    const int nb = grid_for(g.ncells * geo_nblk(g), 256, 4096);
    hipLaunchKernelGGL(relayout_kernel, dim3(nb), dim3(256), 0, s, g, g.ndim + 2, mesh, blk, to_blocks);
    return hipGetLastError();
}

hipError_t launch_padded_prim(const Geo& g, int precision, const double* U, double* Wp, Ctrl* ctrl,
                              hipStream_t s) {
    const int nb = grid_for(g.ncells * geo_nblk(g) * 2 + 4096, 256, 4096);
#define PP(ND, RT) hipLaunchKernelGGL((padded_prim_kernel<ND, RT>), dim3(nb), dim3(256), 0, s, g, U, Wp, ctrl)
    if (precision == 0) {
        switch (g.ndim) {
            case 1: PP(1, double); break;
            case 2: PP(2, double); break;
            case 3: PP(3, double); break;
            default: return hipErrorInvalidValue;
        }
    } else {
        switch (g.ndim) {
            case 1: PP(1, float); break;
            case 2: PP(2, float); break;
            case 3: PP(3, float); break;
            default: return hipErrorInvalidValue;
        }
    }
#undef PP
    return hipGetLastError();
}

hipError_t launch_smr_restrict(const Geo& g, const double* U, double* gbuf, long long gcs, const GhostTask* tasks,
                               int n, Ctrl* ctrl, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    // one thread per ghost of the largest slot (gcs = its two layers)
    const dim3 grid(n, (unsigned)((gcs + 63) / 64));
    switch (g.ndim) {
        case 1: hipLaunchKernelGGL(smr_restrict_kernel<1>, grid, dim3(64), 0, s, g, U, gbuf, gcs, tasks, ctrl); break;
        case 2: hipLaunchKernelGGL(smr_restrict_kernel<2>, grid, dim3(64), 0, s, g, U, gbuf, gcs, tasks, ctrl); break;
        case 3: hipLaunchKernelGGL(smr_restrict_kernel<3>, grid, dim3(64), 0, s, g, U, gbuf, gcs, tasks, ctrl); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_smr_prolong(const Geo& g, const double* U, const int* side, double* gbuf, long long gcs,
                              const GhostTask* tasks, int n, Ctrl* ctrl, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    // one thread per coarse cell across the largest side
    const long long cells = (gcs / 2) >> (g.ndim - 1);
    const dim3 grid(n, (unsigned)((cells + 63) / 64));
    switch (g.ndim) {
        case 1: hipLaunchKernelGGL(smr_prolong_kernel<1>, grid, dim3(64), 0, s, g, U, side, gbuf, gcs, tasks, ctrl); break;
        case 2: hipLaunchKernelGGL(smr_prolong_kernel<2>, grid, dim3(64), 0, s, g, U, side, gbuf, gcs, tasks, ctrl); break;
        case 3: hipLaunchKernelGGL(smr_prolong_kernel<3>, grid, dim3(64), 0, s, g, U, side, gbuf, gcs, tasks, ctrl); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_smr_correct(int precision, int first, const Geo& g, const double* in, double* out, double factor,
                              int use_device_dt, double dt_host, const int* side, const double* gbuf, long long gcs,
                              const GhostTask* tasks, int nres, int want_dt, Ctrl* ctrl, hipStream_t s) {
    if (nres <= 0) return hipSuccess;
    // one thread per fine face across the largest side
    const long long faces = (gcs / 2) << (g.ndim - 1);
    const dim3 grid(nres, (unsigned)((faces + 63) / 64));
#define RF(ND, RT, FO)                                                                                        \
    hipLaunchKernelGGL((smr_correct_kernel<ND, RT, FO>), grid, dim3(64), 0, s, g, in, out, factor, use_device_dt, \
                       dt_host, side, gbuf, gcs, tasks, nres, want_dt, ctrl)
    switch ((g.ndim * 2 + (precision == 0 ? 0 : 1)) * 2 + (first ? 1 : 0)) {
        case 4: RF(1, double, false); break;
        case 5: RF(1, double, true); break;
        case 6: RF(1, float, false); break;
        case 7: RF(1, float, true); break;
        case 8: RF(2, double, false); break;
        case 9: RF(2, double, true); break;
        case 10: RF(2, float, false); break;
        case 11: RF(2, float, true); break;
        case 12: RF(3, double, false); break;
        case 13: RF(3, double, true); break;
        case 14: RF(3, float, false); break;
        case 15: RF(3, float, true); break;
        default: return hipErrorInvalidValue;
    }
#undef RF
    return hipGetLastError();
}

hipError_t launch_riemann(int precision, int ntan, double gamma, long long n, const double* WL,
                          const double* WR, double* F, hipStream_t s) {
    const int nb = grid_for(n, 256, 4096);
#define RK(RT, NTAN) \
    hipLaunchKernelGGL((riemann_kernel<RT, NTAN>), dim3(nb), dim3(256), 0, s, gamma, n, WL, WR, F)
    if (precision == 0) {
        switch (ntan) {
            case 0: RK(double, 0); break;
            case 1: RK(double, 1); break;
            case 2: RK(double, 2); break;
            default: return hipErrorInvalidValue;
        }
    } else {
        switch (ntan) {
            case 0: RK(float, 0); break;
            case 1: RK(float, 1); break;
            case 2: RK(float, 2); break;
            default: return hipErrorInvalidValue;
        }
    }
#undef RK
    return hipGetLastError();
}

#endif  // HYDRO_PART

}  // namespace hydro
