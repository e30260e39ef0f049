// Per-cell stencil code shared by the forward sweep and its adjoint: the
// coefficient struct, the stars of one cell, the residual of Eq. 1-3, the
// wall ghost rules and the stars of one cell read from global memory.
// Included by sweep.hip and adjoint.hip only; both are built with
// -ffp-contract=off.
#pragma once

#include "cavity_internal.h"

namespace cav {

// Coefficients in the arithmetic type of the sweep.
template <typename Real>
struct CoefR {
    Real hx2, hy2, hz2, ix2, iy2, iz2, eps4, beta2_floor, nu, alpha, t_inf, cfl, dt_visc, t_hot, t_cold;
    const double* t_hot_field;    // NULL or nj*nk hot-wall temperatures, j fastest
};

template <typename Real>
__device__ __forceinline__ CoefR<Real> coef_as(const Coef& c)
{
    return CoefR<Real>{(Real)c.hx2, (Real)c.hy2, (Real)c.hz2, (Real)c.ix2, (Real)c.iy2, (Real)c.iz2,
                       (Real)c.eps4, (Real)c.beta2_floor, (Real)c.nu, (Real)c.alpha, (Real)c.t_inf,
                       (Real)c.cfl, (Real)c.dt_visc, (Real)c.t_hot, (Real)c.t_cold, c.t_hot_field};
}

// Temperature of the hot wall x = 0 next to row j of plane k.
template <typename Real>
__device__ __forceinline__ Real hot_wall(const CoefR<Real>& c, const Dims& d, int j, int k)
{
    return c.t_hot_field ? (Real)c.t_hot_field[j + (long long)d.nj * k] : c.t_hot;
}

// ---------------------------------------------------------------------------
// Per-cell residual.  Inputs: the 13-point pressure star and the 7-point
// stars of u, v, w, T.  Outputs: R_p (Eq. 1 times beta^2, with the
// dissipation -eps4 * lambda_x * F_x p / h_x per axis), R_u, R_v, R_w
// (Eq. 2, advective form, buoyancy +(T - t_inf) along z) and R_T (Eq. 3),
// and the local pseudo-time step.
template <typename Real>
struct Star {
    Real p, pxm, pxp, pxm2, pxp2, pym, pyp, pym2, pyp2, pzm, pzp, pzm2, pzp2;
    Real u, uxm, uxp, uym, uyp, uzm, uzp;
    Real v, vxm, vxp, vym, vyp, vzm, vzp;
    Real w, wxm, wxp, wym, wyp, wzm, wzp;
    Real t, txm, txp, tym, typ, tzm, tzp;
};

template <typename Real>
__device__ __forceinline__ Real lap3(const CoefR<Real>& c, Real q, Real xm, Real xp, Real ym,
                                       Real yp, Real zm, Real zp)
{
    // (L_x + L_y + L_z) q with L_x q = ((q_{i+1} + q_{i-1}) - 2 q_i) / h_x^2
    return fma(c.ix2, fma(Real(-2), q, xp + xm), fma(c.iy2, fma(Real(-2), q, yp + ym), c.iz2 * fma(Real(-2), q, zp + zm)));
}

// Square root of a positive argument: hardware reciprocal-square-root
// estimate refined by Goldschmidt's iteration (one coupled step for
// sqrt(x) and 1/(2 sqrt(x)), then a final residual correction), within an
// ulp of the correctly rounded result.  Arguments below 1e-300 are clamped.
__device__ __forceinline__ double sqrt_pos(double x)
{
    x = fmax(x, 1e-300);
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    const double d = fma(-g, g, x);
    return fma(h, d, g);
}

// 1/x for x > 0: hardware estimate refined by two Newton steps.
__device__ __forceinline__ double recip_pos(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    double e = fma(-x, y, 1.0);
    y = fma(y, e, y);
    e = fma(-x, y, 1.0);
    return fma(y, e, y);
}

// FP32 forms: the hardware square root (within 1 ulp; the argument is kept
// above the denormal range) and a reciprocal estimate refined by one Newton
// step.
__device__ __forceinline__ float sqrt_pos(float x) { return __builtin_amdgcn_sqrtf(fmaxf(x, 1e-30f)); }

__device__ __forceinline__ float recip_pos(float x)
{
    const float y = __builtin_amdgcn_rcpf(x);
    return fmaf(y, fmaf(-x, y, 1.0f), y);
}

template <typename Real>
__device__ __forceinline__ void cell_residual(const CoefR<Real>& c, const Star<Real>& s, Real R[NF], Real& dt)
{
    // first differences (times 2h)
    const Real dxu = s.uxp - s.uxm, dyu = s.uyp - s.uym, dzu = s.uzp - s.uzm;
    const Real dxv = s.vxp - s.vxm, dyv = s.vyp - s.vym, dzv = s.vzp - s.vzm;
    const Real dxw = s.wxp - s.wxm, dyw = s.wyp - s.wym, dzw = s.wzp - s.wzm;
    const Real dxt = s.txp - s.txm, dyt = s.typ - s.tym, dzt = s.tzp - s.tzm;
    const Real dxp = s.pxp - s.pxm, dyp = s.pyp - s.pym, dzp = s.pzp - s.pzm;

    // advecting velocity scaled by 1/(2h): V . grad q = su*dxq + sv*dyq + sw*dzq
    const Real su = s.u * c.hx2, sv = s.v * c.hy2, sw = s.w * c.hz2;

    // artificial compressibility and characteristic speeds over h
    const Real u2 = s.u * s.u, v2 = s.v * s.v, w2 = s.w * s.w;
    const Real beta2 = fmax((u2 + v2) + w2, c.beta2_floor);
    const Real b4 = Real(4) * beta2;
    const Real lxn = (fabs(s.u) + sqrt_pos(u2 + b4)) * c.hx2;   // lambda_x / h_x
    const Real lyn = (fabs(s.v) + sqrt_pos(v2 + b4)) * c.hy2;
    const Real lzn = (fabs(s.w) + sqrt_pos(w2 + b4)) * c.hz2;
    dt = c.cfl * fmin(recip_pos((lxn + lyn) + lzn), c.dt_visc);

    // continuity (Eq. 1 times beta^2) with fourth-difference dissipation
    const Real div = fma(dxu, c.hx2, fma(dyv, c.hy2, dzw * c.hz2));
    const Real fx = fma(Real(6), s.p, fma(Real(-4), s.pxp + s.pxm, s.pxp2 + s.pxm2));
    const Real fy = fma(Real(6), s.p, fma(Real(-4), s.pyp + s.pym, s.pyp2 + s.pym2));
    const Real fz = fma(Real(6), s.p, fma(Real(-4), s.pzp + s.pzm, s.pzp2 + s.pzm2));
    const Real diss = fma(lxn, fx, fma(lyn, fy, lzn * fz));
    R[FP] = fma(-beta2, div, -c.eps4 * diss);

    // momentum (Eq. 2) and energy (Eq. 3)
    const Real adu = fma(su, dxu, fma(sv, dyu, sw * dzu));
    const Real adv = fma(su, dxv, fma(sv, dyv, sw * dzv));
    const Real adw = fma(su, dxw, fma(sv, dyw, sw * dzw));
    const Real adt = fma(su, dxt, fma(sv, dyt, sw * dzt));
    R[FU] = fma(c.nu, lap3(c, s.u, s.uxm, s.uxp, s.uym, s.uyp, s.uzm, s.uzp), -fma(dxp, c.hx2, adu));
    R[FV] = fma(c.nu, lap3(c, s.v, s.vxm, s.vxp, s.vym, s.vyp, s.vzm, s.vzp), -fma(dyp, c.hy2, adv));
    R[FW] = fma(c.nu, lap3(c, s.w, s.wxm, s.wxp, s.wym, s.wyp, s.wzm, s.wzp),
                (s.t - c.t_inf) - fma(dzp, c.hz2, adw));
    R[FT] = fma(c.alpha, lap3(c, s.t, s.txm, s.txp, s.tym, s.typ, s.tzm, s.tzp), -adt);
}

// ---------------------------------------------------------------------------
// Wall ghosts on the fly (Sec. 2).  The state in HBM holds only interior
// cells that the sweep reads; a face-ghost value g = 1, 2 layers beyond a
// wall is derived from the interior cells m0 (next to the wall) and m1:
//   p:        g1 = 2 q(m0) - q(m1), g2 = 2 g1 - q(m0)  (one-sided linear
//             extrapolation, second order)
//   u, v, w:  g = -q(m_{g-1})                          (no-slip)
//   T:        g = 2 T_wall - q(m_{g-1}) on the hot (x = 0) and cold (x = 1)
//             walls, g = q(m_{g-1}) on the adiabatic walls.
// The wall ghosts of one cell's stars along axis AX, by these rules from the
// star's own values: m0 of a ghost is the cell itself or its neighbour
// towards the wall, m1 the next one (the extents are >= 2).  x: the cell's
// coordinate along the axis, n its extent; j, k: its hot-wall row.
template <int AX, typename Real>
__device__ __forceinline__ void star_ghosts_axis(int x, int n, Star<Real>& s, const CoefR<Real>& c, const Dims& d, int j,
                                                 int k)
{
#define STAR_AX(nm, sfx) (AX == 0 ? s.nm##x##sfx : (AX == 1 ? s.nm##y##sfx : s.nm##z##sfx))
    if (x == 0) {
        STAR_AX(p, m) = Real(2) * s.p - STAR_AX(p, p);
        STAR_AX(u, m) = -s.u;
        STAR_AX(v, m) = -s.v;
        STAR_AX(w, m) = -s.w;
        STAR_AX(t, m) = AX == 0 ? Real(2) * hot_wall(c, d, j, k) - s.t : s.t;
    }
    if (x == n - 1) {
        STAR_AX(p, p) = Real(2) * s.p - STAR_AX(p, m);
        STAR_AX(u, p) = -s.u;
        STAR_AX(v, p) = -s.v;
        STAR_AX(w, p) = -s.w;
        STAR_AX(t, p) = AX == 0 ? Real(2) * c.t_cold - s.t : s.t;
    }
    if (x <= 1) STAR_AX(p, m2) = Real(2) * STAR_AX(p, m) - s.p;
    if (x >= n - 2) STAR_AX(p, p2) = Real(2) * STAR_AX(p, p) - s.p;
#undef STAR_AX
}

// A cell's place in the grid and the byte offsets, from element `base` of a
// field, of it and of its neighbours one and two cells away per axis (its own
// offset where that neighbour lies beyond a wall).  32-bit offsets from a
// uniform base cost one register and no 64-bit arithmetic per load; the
// caller picks base so that they fit.
struct PointCell {
    int i, j, k, base;
    uint32_t o, xm, xp, xm2, xp2, ym, yp, ym2, yp2, zm, zp, zm2, zp2;
};

template <typename Real>
__device__ __forceinline__ PointCell point_cell(const Dims& d, int i, int j, int k, int base)
{
    PointCell e;
    e.i = i; e.j = j; e.k = k; e.base = base;
    const uint32_t B = sizeof(Real), sy = d.sy * B, sz = d.sz * B;
    e.o = (uint32_t)(cell_off(d, i, j, k) - base) * B;
    e.xm = i > 0 ? e.o - B : e.o;         e.xm2 = i > 1 ? e.o - 2 * B : e.o;
    e.xp = i < d.ni - 1 ? e.o + B : e.o;  e.xp2 = i < d.ni - 2 ? e.o + 2 * B : e.o;
    e.ym = j > 0 ? e.o - sy : e.o;        e.ym2 = j > 1 ? e.o - 2 * sy : e.o;
    e.yp = j < d.nj - 1 ? e.o + sy : e.o; e.yp2 = j < d.nj - 2 ? e.o + 2 * sy : e.o;
    e.zm = k > 0 ? e.o - sz : e.o;        e.zm2 = k > 1 ? e.o - 2 * sz : e.o;
    e.zp = k < d.nk - 1 ? e.o + sz : e.o; e.zp2 = k < d.nk - 2 ? e.o + 2 * sz : e.o;
    return e;
}

// The centre cell of the rescale (Sec. 2).  Its star lies within two planes.
template <typename Real>
__device__ __forceinline__ PointCell centre_cell(const Dims& d)
{
    const int i = d.ni / 2, j = d.nj / 2, k = d.nk / 2;
    return point_cell<Real>(d, i, j, k, cell_off(d, i, j, k) - 2 * d.sz);
}

// The value of the lane below (UP = false) or above in the wavefront; the
// lane at its end keeps `end`.
template <bool UP>
__device__ __forceinline__ uint32_t lane_next(uint32_t v, uint32_t end)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)end, (int)v, UP ? 0x130 : 0x138, 0xf, 0xf, false);
}
template <bool UP>
__device__ __forceinline__ float lane_next(float v, float end)
{
    return __builtin_bit_cast(float, lane_next<UP>(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, end)));
}
template <bool UP>
__device__ __forceinline__ double lane_next(double v, double end)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, v), b = __builtin_bit_cast(uint64_t, end);
    const uint64_t lo = lane_next<UP>((uint32_t)a, (uint32_t)b), hi = lane_next<UP>((uint32_t)(a >> 32), (uint32_t)(b >> 32));
    return __builtin_bit_cast(double, lo | hi << 32);
}

// The stars of one cell straight from global memory, all loads independent
// of each other, then its wall ghosts.  ROW: the wavefront's lanes hold
// 64 consecutive cells, so the x neighbours are the adjacent lanes' cells
// (moved, not loaded: 29 loads instead of 41) and only the two end lanes load
// theirs; every lane must be active.
template <typename Real, bool ROW = false>
__device__ __forceinline__ void point_star(const Dims& d, const CStateT<Real>& q, const CoefR<Real>& c,
                                           const PointCell& e, Star<Real>& s)
{
    auto at = [&](int f, uint32_t off) __attribute__((always_inline)) {
        return *reinterpret_cast<const Real*>(reinterpret_cast<const char*>(q.f[f] + e.base) + off);
    };
    Real end1[NF], end2 = Real(0);
    if constexpr (ROW) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int f = 0; f < NF; ++f) end1[f] = Real(0);
        if (lane == 0 || lane == 63) {
            end2 = at(FP, lane ? e.xp2 : e.xm2);
#pragma unroll
            for (int f = 0; f < NF; ++f) end1[f] = at(f, lane ? e.xp : e.xm);
        }
    }
    s.p = at(FP, e.o);
    s.pym = at(FP, e.ym); s.pyp = at(FP, e.yp); s.pym2 = at(FP, e.ym2); s.pyp2 = at(FP, e.yp2);
    s.pzm = at(FP, e.zm); s.pzp = at(FP, e.zp); s.pzm2 = at(FP, e.zm2); s.pzp2 = at(FP, e.zp2);
#define POINT_STAR5(F, nm)                                \
    s.nm = at(F, e.o);                                    \
    s.nm##ym = at(F, e.ym); s.nm##yp = at(F, e.yp);       \
    s.nm##zm = at(F, e.zm); s.nm##zp = at(F, e.zp);
    POINT_STAR5(FU, u) POINT_STAR5(FV, v) POINT_STAR5(FW, w) POINT_STAR5(FT, t)
#undef POINT_STAR5
#define POINT_X(F, nm)                                                                                  \
    s.nm##xm = ROW ? lane_next<false>(s.nm, end1[F]) : at(F, e.xm);                                     \
    s.nm##xp = ROW ? lane_next<true>(s.nm, end1[F]) : at(F, e.xp);
    POINT_X(FP, p) POINT_X(FU, u) POINT_X(FV, v) POINT_X(FW, w) POINT_X(FT, t)
#undef POINT_X
    s.pxm2 = ROW ? lane_next<false>(s.pxm, end2) : at(FP, e.xm2);
    s.pxp2 = ROW ? lane_next<true>(s.pxp, end2) : at(FP, e.xp2);
    star_ghosts_axis<0>(e.i, d.ni, s, c, d, e.j, e.k);
    star_ghosts_axis<1>(e.j, d.nj, s, c, d, e.j, e.k);
    star_ghosts_axis<2>(e.k, d.nk, s, c, d, e.j, e.k);
}

// Map hardware block ids (dispatched round-robin over the 8 XCDs) to tiles
// so that each XCD works on one contiguous range of tiles and neighbouring
// tiles share that XCD's L2.
__device__ __forceinline__ int xcd_block(int bid, int nb)
{
    const int per = nb >> 3, rem = nb & 7;
    const int x = bid & 7, y = bid >> 3;
    return x * per + min(x, rem) + y;
}


}  // namespace cav
