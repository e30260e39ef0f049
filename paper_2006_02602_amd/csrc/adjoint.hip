// Discrete adjoint (reverse mode) of one pseudo-time step and of the mean
// hot-wall Nusselt number, in FP64.
//
// One step maps the state q^n to q^{n+1} (Sec. 2, Eq. 1-3): wall ghosts G
// from the interior cells and the hot-wall temperatures Theta, per cell the
// residual R(S) and local step dt(S) of its stars S, q* = q + dt R, and the
// pressure rescale p^{n+1} = p* - p*(centre).  Given the cotangent lambda of
// q^{n+1}, the reverse step returns the cotangent of q^n and adds the
// cotangents of Theta and of Ra.
//
// Seeds: a_f = lambda_f dt of R_f and b = sum_f lambda_f R_f of dt.  The star
// cotangents of a cell m are linear in a few numbers of m:
//   p:      centre -6 (Xx + Xy + Xz); at +-1 along x: -+a_u/(2h_x) + 4 Xx;
//           at +-2 along x: -Xx (y, z alike with a_v, a_w)
//   u:      centre ub + ctr nu a_u; at +-1 along x: -+(su a_u + Bp/(2h_x))
//           + nu a_u/h_x^2; along y: -+sv a_u + nu a_u/h_y^2; z alike
//   v, w:   likewise, with the Bp term along y for v and along z for w
//   T:      centre a_w + ctr alpha a_T; along each axis -+s a_T + alpha a_T/h^2
// with Xi = eps4 a_p lambda_i/h_i, Bp = beta^2 a_p, (su, sv, sw) = V/(2h),
// ctr = -2 sum 1/h^2, "-+" meaning - at +1 and + at -1.  Only ub, vb, wb
// depend on m's stars, and only m itself needs them; the rest follows from
// m's velocity and lambda (cell_d).  So one pass does the step: a cell forms
// its own dt, X, Bp and ub, vb, wb and gathers the star cotangents that land
// on it from its neighbours' lambda, velocity, dt, X and Bp; cells within two
// of a wall add the transposed wall rules of the ghosts their neighbours read
// (and the x = 0 wall rows add to dJ/dTheta).  The transpose of the rescale
// (the centre cell's p seed is lambda_p minus the sum of lambda_p over the
// grid) and the Ra sum follow in a small second launch.
//
// Non-smooth points take one side: |u| has slope +1 at u = 0; beta^2 =
// max(|V|^2, floor) follows |V|^2 only where strictly larger; dt follows the
// convective limit only where strictly smaller than the viscous one.
// Every sum runs in a fixed order, so results are run-to-run identical.
#include "cavity_internal.h"
#include "stencil.h"
#include "sweep_tile.h"      // TileBox, tile_box

#include <algorithm>
#include <type_traits>

namespace cav {

namespace {

constexpr int NREC = 8;            // doubles of workspace per cell (see adjoint_ws_doubles)
constexpr int ADJ_THREADS = 256;

// What a cell's velocity and lambda_p alone determine: dt, the dissipation
// terms Xx, Xy, Xz and Bp (dt by the formulas of cell_residual).
struct CellD {
    double dt, X[3], Bp;
};
__device__ __forceinline__ CellD cell_d(const CoefR<double>& c, double u, double v, double w, double lp)
{
    const double u2 = u * u, v2 = v * v, w2 = w * w;
    const double beta2 = fmax((u2 + v2) + w2, c.beta2_floor);
    const double b4 = 4.0 * beta2;
    const double lxn = (fabs(u) + sqrt_pos(u2 + b4)) * c.hx2;
    const double lyn = (fabs(v) + sqrt_pos(v2 + b4)) * c.hy2;
    const double lzn = (fabs(w) + sqrt_pos(w2 + b4)) * c.hz2;
    CellD D;
    D.dt = c.cfl * fmin(recip_pos((lxn + lyn) + lzn), c.dt_visc);
    const double ap = lp * D.dt;
    const double dissb = -c.eps4 * ap;
    D.X[0] = -lxn * dissb;
    D.X[1] = -lyn * dissb;
    D.X[2] = -lzn * dissb;
    D.Bp = beta2 * ap;
    return D;
}

struct RaFactors {
    double nu, alpha, dtv;        // d(nu)/dRa, d(alpha)/dRa, d(dt_visc)/dRa
};

// The cotangent a cell collects.
struct GatherAcc {
    double Lp, Lu, Lv, Lw, Lt;
};

// Coefficients of the reverse step; the products are formed on the host (in
// the kernel they would be loop invariants in vector registers).
struct RevCoef : CoefR<double> {
    RaFactors rf;
    double nu_i2[3], al_i2[3];    // nu/h^2, alpha/h^2 per axis
    double nu_c, al_c;            // -2 nu sum 1/h^2, -2 alpha sum 1/h^2
};

struct SeedTerms {
    double ub, vb, wb;            // the cell's own centre terms
    double ra;                    // its term of the Ra cotangent
};

// The reverse of one cell's residual and step, given lambda at the cell: seeds
// a_f = lambda_f dt of R_f and b = sum_f lambda_f R_f of dt.  Of the stars
// only a few sums are needed, taken axis by axis (so that few star values are
// live at once): G[ax] = sum_f lambda_f D_ax f over u, v, w, T (advection),
// sn and st (lambda-weighted Laplacians of the velocity and of T), the
// weighted pressure gradient, the divergence and the fourth differences of p.
struct ReverseCell {
    double G[3], F[3], sn, st, gp, div;

    // fm, fp: u, v, w, T one cell below and above; p likewise, and two away
    template <int AX>
    __device__ __forceinline__ void axis(const RevCoef& c, const double l[NF - 1], const double f0[NF - 1], double p0,
                                         const double fm[NF - 1], const double fp[NF - 1], double pm, double pp, double pm2,
                                         double pp2)
    {
        const double h2 = AX == 0 ? c.hx2 : (AX == 1 ? c.hy2 : c.hz2);
        const double i2 = AX == 0 ? c.ix2 : (AX == 1 ? c.iy2 : c.iz2);
        double g = 0.0, n = 0.0;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            g = fma(l[f], fp[f] - fm[f], g);
            n = fma(l[f], fma(-2.0, f0[f], fp[f] + fm[f]), n);
        }
        G[AX] = fma(l[3], fp[3] - fm[3], g);
        const double t = l[3] * fma(-2.0, f0[3], fp[3] + fm[3]);
        const double gpx = (l[AX] * h2) * (pp - pm), dv = (fp[AX] - fm[AX]) * h2;
        F[AX] = fma(6.0, p0, fma(-4.0, pp + pm, pp2 + pm2));
        sn = AX == 0 ? i2 * n : fma(i2, n, sn);
        st = AX == 0 ? i2 * t : fma(i2, t, st);
        gp = AX == 0 ? gpx : gp + gpx;
        div = AX == 0 ? dv : div + dv;
    }

    __device__ __forceinline__ SeedTerms finish(const RevCoef& c, const double l[NF - 1],
                                                const double f0[NF - 1], double lp, double dt) const
    {
        const double u = f0[0], v = f0[1], w = f0[2];
        const double u2 = u * u, v2 = v * v, w2 = w * w;
        const double vv = (u2 + v2) + w2;
        const bool beta_free = vv > c.beta2_floor;
        const double beta2 = fmax(vv, c.beta2_floor);
        const double b4 = 4.0 * beta2;
        const double rx = sqrt_pos(u2 + b4), ry = sqrt_pos(v2 + b4), rz = sqrt_pos(w2 + b4);
        const double lxn = (fabs(u) + rx) * c.hx2, lyn = (fabs(v) + ry) * c.hy2, lzn = (fabs(w) + rz) * c.hz2;
        const double inv = recip_pos((lxn + lyn) + lzn);
        const bool convective = inv < c.dt_visc;
        // b = sum_f lambda_f R_f: diffusion, buoyancy, advection and pressure
        // gradient, and R_p = -beta^2 div - eps4 sum_ax lambda_ax/h_ax F_ax p
        double b = fma(c.nu, sn, fma(c.alpha, st, fma(l[2], f0[3] - c.t_inf, -gp)));
        b = fma(-(u * c.hx2), G[0], fma(-(v * c.hy2), G[1], fma(-(w * c.hz2), G[2], b)));
        b = fma(lp, fma(-beta2, div, -c.eps4 * fma(lxn, F[0], fma(lyn, F[1], lzn * F[2]))), b);
        const double ap = lp * dt, dissb = -c.eps4 * ap, cb = c.cfl * b;
        SeedTerms o;
        o.ra = dt * fma(sn, c.rf.nu, st * c.rf.alpha);
        // dt = cfl min(1 / (lxn + lyn + lzn), dt_visc)
        const double lsb = convective ? -cb * inv * inv : 0.0;
        if (!convective) o.ra = fma(cb, c.rf.dtv, o.ra);
        const double rxb = c.hx2 * fma(F[0], dissb, lsb), ryb = c.hy2 * fma(F[1], dissb, lsb);
        const double rzb = c.hz2 * fma(F[2], dissb, lsb);
        // lambda_i / h_i = (|V_i| + sqrt(V_i^2 + 4 beta^2)) / (2 h_i); the
        // advecting velocity (R_f holds -V_i D_i f / (2 h_i))
        const double tx = 0.5 * rxb * recip_pos(rx), ty = 0.5 * ryb * recip_pos(ry), tz = 0.5 * rzb * recip_pos(rz);
        const double beta2b = beta_free ? fma(4.0, (tx + ty) + tz, -div * ap) : 0.0;
        o.ub = fma(2.0 * u, tx + beta2b, fma(-dt * c.hx2, G[0], u < 0.0 ? -rxb : rxb));
        o.vb = fma(2.0 * v, ty + beta2b, fma(-dt * c.hy2, G[1], v < 0.0 ? -ryb : ryb));
        o.wb = fma(2.0 * w, tz + beta2b, fma(-dt * c.hz2, G[2], w < 0.0 ? -rzb : rzb));
        return o;
    }
};

// What the gather needs from a neighbour m along an axis: lambda_u ..
// lambda_T and dt (their products are the seeds a_u .. a_T), that axis's
// dissipation term X, Bp, and m's velocity along the axis times 1/(2h).
struct Nbr {
    double l[NF - 1], dt, X, Bp, s;
};

// The cotangents cell b's star puts on the cell one step from b in direction
// DIR along axis AX, times SIGN, added to a: for DIR = +1 the slot "+", so
//   p: -a_ax/(2h) + 4 X;  u .. T: a_f (nu/h^2 - s) (alpha for T);
//   the velocity along the axis also -Bp/(2h);  DIR = -1 with the signs of
//   the first differences turned.
template <int AX, int DIR>
__device__ __forceinline__ void add_star(GatherAcc& a, const RevCoef& c, const Nbr& b)
{
    const double H = AX == 0 ? c.hx2 : (AX == 1 ? c.hy2 : c.hz2);
    const double Hs = DIR > 0 ? -H : H, s = DIR > 0 ? -b.s : b.s;
    const double fn = b.dt * (c.nu_i2[AX] + s), ft = b.dt * (c.al_i2[AX] + s);
    a.Lp = fma(4.0, b.X, fma(b.l[AX] * b.dt, Hs, a.Lp));
    a.Lu = fma(b.l[0], fn, a.Lu);
    a.Lv = fma(b.l[1], fn, a.Lv);
    a.Lw = fma(b.l[2], fn, a.Lw);
    a.Lt = fma(b.l[3], ft, a.Lt);
    (AX == 0 ? a.Lu : (AX == 1 ? a.Lv : a.Lw)) += Hs * b.Bp;
}

// The transposed wall rules along axis AX at the wall in direction DIR for a
// cell at x = m0 (next to the wall) or m1 (the next one): ghosts g1, g2
// beyond the wall carry the cotangents of the stars that read them; the rules
// move them onto m0 and m1:
//   p: m0 += 2 g1 + 3 g2, m1 -= g1 + 2 g2;  u v w: m0 -= g1;
//   T: m0 -= g1 on x walls (and Theta += 2 g1 at x = 0), m0 += g1 on others.
// b0: cell m0; X1: m1's dissipation term; dth: where Theta's term goes, or NULL.
template <int AX, int DIR>
__device__ __forceinline__ void add_wall(GatherAcc& a, const RevCoef& c, int x, int n, const Nbr& b0, double X1,
                                         double* dth)
{
    // g1 collects m0's one-step and m1's two-step reach past the wall, g2
    // m0's two-step reach
    GatherAcc t{0.0, 0.0, 0.0, 0.0, 0.0};
    add_star<AX, DIR>(t, c, b0);
    const double g1p = t.Lp - X1, g2p = -b0.X;
    if (x == (DIR > 0 ? n - 1 : 0)) {
        a.Lp += 2.0 * g1p + 3.0 * g2p;
        a.Lu -= t.Lu;
        a.Lv -= t.Lv;
        a.Lw -= t.Lw;
        if (AX == 0) {
            a.Lt -= t.Lt;
            if (DIR < 0 && dth) *dth = 2.0 * t.Lt;
        } else {
            a.Lt += t.Lt;
        }
    } else {
        a.Lp -= g1p + 2.0 * g2p;
    }
}

// The wall ghosts of one axis of a cell's stars (star_ghosts_axis for values
// held per axis).  wall: the hot-wall temperature of the cell's row.
template <int AX>
__device__ __forceinline__ void axis_ghosts(const RevCoef& c, int x, int n, double wall, const double f0[NF - 1], double p0, double fm[NF - 1], double fp[NF - 1],
                                            double& pm, double& pp, double& pm2, double& pp2)
{
    if (x == 0) {
        pm = 2.0 * p0 - pp;
#pragma unroll
        for (int f = 0; f < 3; ++f) fm[f] = -f0[f];
        fm[3] = AX == 0 ? 2.0 * wall - f0[3] : f0[3];
    }
    if (x == n - 1) {
        pp = 2.0 * p0 - pm;
#pragma unroll
        for (int f = 0; f < 3; ++f) fp[f] = -f0[f];
        fp[3] = AX == 0 ? 2.0 * c.t_cold - f0[3] : f0[3];
    }
    if (x <= 1) pm2 = 2.0 * pm - p0;
    if (x >= n - 2) pp2 = 2.0 * pp - p0;
}

// Keeps the compiler from moving work across a phase of the tile's plane:
// left alone it issues every LDS read of a plane first and spills.
#define PHASE() __builtin_amdgcn_sched_barrier(0)

// A copy made here, in a register of its own.
__device__ __forceinline__ double moved(double x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// The value at 32-bit byte offset off from a uniform base.
__device__ __forceinline__ double ldo(const double* base, uint32_t off)
{
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + off);
}

// The pass as a k-marching LDS tile: a block of 64 x TJ threads marches its
// (i, j) columns through a k chunk.  Each plane, every thread puts what its
// in-plane neighbours need into LDS, the block's threads add the tile's halo
// (two rows above and below, two columns left and right), and after one
// barrier every cell reads its x and y neighbours from there; the z
// neighbours are register queues, and a cell's dt, X and Bp are formed when
// its plane is two ahead.  So every value is read from memory once per tile
// plus the halo, and nothing is stored but lambda: 120 B per cell at least,
// where a pass that stored the centre terms and one that gathered with them
// moved 259 (256^3: 515 + 595 us in two passes, 535 in one).  160 KB of LDS
// (one block per CU) and 236 VGPRs: the z neighbours' dt and Bp and the
// in-plane X stay in LDS for their three planes rather than in registers.
// Its loads run a plane ahead without conditions (with them every plane began
// by waiting for all loads in flight: 660 us); what is left is the 616 VALU
// and 78 LDS instructions a wavefront issues per plane, two to a SIMD.
template <int TJ>
struct ReverseTile {
    static constexpr int THREADS = 64 * TJ;
    // One plane in LDS.  Two alternate: eight values with one halo cell per
    // side (index r1), p with two.  Three rotate, since a cell's own thread
    // writes them two planes ahead and reads them until the plane is done: dt
    // and Bp (r1), the x dissipation term with two halo columns (xx) and the
    // y one with two halo rows (xy).
    enum { U, V, W, T, LU, LV, LW, LT };
    enum { DT, BP };
    static constexpr int W1 = 66, S1 = (TJ + 2) * W1, WP = 68;
    static constexpr int OP = 8 * S1, TWO = OP + (TJ + 4) * WP;
    static constexpr int OXX = 2 * S1, OXY = OXX + TJ * WP, THREE = OXY + (TJ + 4) * 64;
    static constexpr int LDS = 2 * TWO + 3 * THREE;
    __device__ static int r1(int row, int col) { return (row + 1) * W1 + col + 1; }
    __device__ static int p(int row, int col) { return OP + (row + 2) * WP + col + 2; }
    __device__ static int xx(int row, int col) { return OXX + row * WP + col + 2; }
    __device__ static int xy(int row, int col) { return OXY + (row + 2) * 64 + col; }
    // halo slots per plane, five loads each: rows -1 and TJ and columns -1
    // and 64 twice (velocity, p, lambda_p; T, lambda_u .. lambda_T), rows -2
    // and TJ+1 and columns -2 and 65 once (velocity, p, lambda_p)
    static constexpr int RING = 2 * 64 + 2 * TJ, SLOTS = 3 * RING;
    static_assert(SLOTS <= THREADS, "one halo slot per thread");
};

template <int TJ>
__global__ __launch_bounds__(64 * TJ) void reverse_tile_kernel(Dims d, RevCoef c, SweepGeom g, long long sf,
                                                               const double* __restrict__ q,
                                                               const double* __restrict__ lam, double* __restrict__ out,
                                                               double* __restrict__ part, double* __restrict__ cx,
                                                               double* __restrict__ rows)
{
    using RT = ReverseTile<TJ>;
    __shared__ double L[RT::LDS];
    const TileBox tb = tile_box<64, TJ>(d, g.tiles_i, g.tiles_j, g.kc, xcd_block(blockIdx.x, g.nblocks));
    const int lane = threadIdx.x, row = threadIdx.y, tid = lane + 64 * row;
    const int i = tb.i0 + lane, j = tb.j0 + row;
    // threads past the grid work on a real cell (clamped), take part in every
    // barrier, and store nothing; no cell of the grid reads their LDS slots
    const bool active = i < d.ni && j < d.nj;
    const int ic = min(i, d.ni - 1), jc = min(j, d.nj - 1);
    // byte offsets within a plane (a plane is under 2^32 bytes)
    const uint32_t ocol = (uint32_t)((jc + NG) * d.sy + d.lead + ic) * 8u;
    const long long Z = d.sz;
    const int k0 = tb.k0, k1 = tb.k1, nk = d.nk;
    const bool bnd_i = tb.i0 == 0 || tb.i0 + 66 > d.ni, bnd_j = tb.j0 == 0 || tb.j0 + TJ + 2 > d.nj;

    const bool centre_col = i == d.ni / 2 && j == d.nj / 2;

    // this thread's halo slot: kind -1 none or outside the grid, 0 ring 1
    // (velocity, p, lambda_p), 1 ring 1 (T, lambda_u .. lambda_T), 2 ring 2
    int hkind = -1, hr = 0, hc = 0;
    {
        const int kind = tid / RT::RING, r = tid % RT::RING, far = kind == 2;
        if (r < 128) { hr = r < 64 ? -1 - far : TJ + far; hc = r & 63; }
        else { hr = (r - 128) % TJ; hc = r - 128 < TJ ? -1 - far : 64 + far; }
        const int gi = tb.i0 + hc, gj = tb.j0 + hr;
        if (kind < 3 && gi >= 0 && gi < d.ni && gj >= 0 && gj < d.nj) hkind = kind;
    }
    const bool hrow = hr < 0 || hr >= TJ;
    const uint32_t ohalo = hkind < 0 ? ocol : (uint32_t)((tb.j0 + hr + NG) * d.sy + d.lead + tb.i0 + hc) * 8u;
    const int hr1 = RT::r1(hr, hc), hp = RT::p(hr, hc), hx = hrow ? RT::xy(hr, hc) : RT::xx(hr, hc);
    struct Halo {
        double v[5];
    };
    // the slot's five values: T, lambda_u .. lambda_T, or u, v, w, lambda_p, p.
    // Every thread loads five (its own cell's where it has no slot): loads
    // under a condition would be counted as missing in the waits that follow.
    const double* hsrc[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        const double* a = m == 0 ? q + FT * sf : lam + m * sf;
        const double* b = m < 3 ? q + (FU + m) * sf : (m == 3 ? lam : q);
        hsrc[m] = reinterpret_cast<const double*>(reinterpret_cast<const char*>(hkind == 1 ? a : b) + ohalo);
    }
    auto load_halo = [&](int k, Halo& H) __attribute__((always_inline)) {
        const long long kz = (k + NG) * Z;
#pragma unroll
        for (int m = 0; m < 5; ++m) H.v[m] = hsrc[m][kz];
    };
    auto store_halo = [&](const Halo& H, double* B, double* Q) __attribute__((always_inline)) {
        if (hkind == 1) {
            B[hr1 + RT::T * RT::S1] = H.v[0];
#pragma unroll
            for (int f = 0; f < 4; ++f) B[hr1 + (RT::LU + f) * RT::S1] = H.v[1 + f];
        } else if (hkind >= 0) {
            const CellD D = cell_d(c, H.v[0], H.v[1], H.v[2], H.v[3]);
            B[hp] = H.v[4];
            Q[hx] = hrow ? D.X[1] : D.X[0];
            if (hkind == 0) {
                B[hr1 + RT::U * RT::S1] = H.v[0];
                B[hr1 + RT::V * RT::S1] = H.v[1];
                B[hr1 + RT::W * RT::S1] = H.v[2];
                Q[hr1 + RT::DT * RT::S1] = D.dt;
                Q[hr1 + RT::BP * RT::S1] = D.Bp;
            }
        }
    };

    struct Col {
        double u, v, w, p, lp;         // loaded three planes before their plane is the current one
        double t, l[NF - 1];           // loaded two planes before
        double X;                      // the z dissipation term, formed two planes before
    };
    auto load = [&](int k, Col& C) __attribute__((always_inline)) {
        const long long kz = (k + NG) * Z;
        C.u = ldo(q + FU * sf + kz, ocol);
        C.v = ldo(q + FV * sf + kz, ocol);
        C.w = ldo(q + FW * sf + kz, ocol);
        C.lp = ldo(lam + FP * sf + kz, ocol);
        C.p = ldo(q + FP * sf + kz, ocol);
    };
    auto load_l = [&](int k, Col& C) __attribute__((always_inline)) {
        const long long kz = (k + NG) * Z;
        C.t = ldo(q + FT * sf + kz, ocol);
#pragma unroll
        for (int f = FU; f <= FT; ++f) C.l[f - FU] = ldo(lam + f * sf + kz, ocol);
    };
    const int o1 = RT::r1(row, lane), op = RT::p(row, lane), ox = RT::xx(row, lane), oy = RT::xy(row, lane);
    // the cell's dt, Bp and dissipation terms, into its place of the rotating planes
    auto derive = [&](Col& C, double* Q) __attribute__((always_inline)) {
        const CellD D = cell_d(c, C.u, C.v, C.w, C.lp);
        Q[o1 + RT::DT * RT::S1] = D.dt;
        Q[o1 + RT::BP * RT::S1] = D.Bp;
        Q[ox] = D.X[0];
        Q[oy] = D.X[1];
        C.X = D.X[2];
    };
    // what plane k-1 (and k-2) leave for plane k: the seeds a_u .. a_T, X, Bp
    // and values at k-1
    double pa[NF - 1] = {0.0, 0.0, 0.0, 0.0}, pX = 0.0, pBp = 0.0;
    double fm[NF - 1] = {0.0, 0.0, 0.0, 0.0}, pm = 0.0, pm2 = 0.0, xm2 = 0.0;
    Col cur, nxt, nn2;
    Halo H;
    double* const Q0 = L + 2 * RT::TWO;
    // the hot-wall temperature of this row, loaded a plane ahead
    const double* const wsrc = c.t_hot_field ? c.t_hot_field + jc : q;
    const long long wstep = c.t_hot_field ? d.nj : 0;
    double wall = wsrc[k0 * wstep];
    load(k0, cur);
    load_l(k0, cur);
    load_halo(k0, H);
    if (k0 + 1 < nk) {
        load(k0 + 1, nxt);
        load_l(k0 + 1, nxt);
    }
    if (k0 >= 2) {
        load(k0 - 2, nn2);
        xm2 = cell_d(c, nn2.u, nn2.v, nn2.w, nn2.lp).X[2];
        pm2 = nn2.p;
    }
    if (k0 >= 1) {
        load(k0 - 1, nn2);
        load_l(k0 - 1, nn2);
        const CellD D = cell_d(c, nn2.u, nn2.v, nn2.w, nn2.lp);
#pragma unroll
        for (int f = 0; f < NF - 1; ++f) pa[f] = nn2.l[f] * D.dt;
        pX = D.X[2];
        pBp = D.Bp;
        fm[0] = nn2.u; fm[1] = nn2.v; fm[2] = nn2.w; fm[3] = nn2.t;
        pm = nn2.p;
    }
    if (k0 + 2 < nk) load(k0 + 2, nn2);
    derive(cur, Q0);
    if (k0 + 1 < nk) derive(nxt, Q0 + RT::THREE);
    double acc_ra = 0.0, acc_s = 0.0;
    // the last plane the chunk needs; loads past it repeat it (a load under a
    // condition would be waited for at once, to be merged with the old value)
    const int klast = min(k1 + 1, nk - 1);

    // One plane per iteration; the sets of planes k, k+1, k+2 are moved down
    // once their values have arrived and the next loads go straight into
    // their set (unrolled by three with rotating sets the kernel spilled 44
    // registers: the LDS addresses of three planes, held across the loop).
    int oq = 0, oqn = RT::THREE, oqnn = 2 * RT::THREE;
    // all loads so far done (vmcnt 0): were some still in flight here, every
    // iteration would start with a wait for them, and with it for its own
    __builtin_amdgcn_s_waitcnt(0x0f70);
    for (int k = k0; k < k1; ++k) {
        double* const B = L + ((k - k0) & 1) * RT::TWO;
        double* const Q = Q0 + oq;
        double* const Qn = Q0 + oqn;
        double* const Qnn = Q0 + oqnn;
        B[o1 + RT::U * RT::S1] = cur.u;
        B[o1 + RT::V * RT::S1] = cur.v;
        B[o1 + RT::W * RT::S1] = cur.w;
        B[o1 + RT::T * RT::S1] = cur.t;
#pragma unroll
        for (int f = 0; f < 4; ++f) B[o1 + (RT::LU + f) * RT::S1] = cur.l[f];
        B[op] = cur.p;
        store_halo(H, B, Q);
        load_halo(min(k + 1, k1 - 1), H);
        __syncthreads();

        const double tw = c.t_hot_field ? wall : c.t_hot;

        // e's own terms, then axis by axis the stars landing on e and e's own
        const double dt = Q[o1 + RT::DT * RT::S1], f0[NF - 1] = {cur.u, cur.v, cur.w, cur.t};
        Nbr me{{cur.l[0], cur.l[1], cur.l[2], cur.l[3]}, dt, 0.0, Q[o1 + RT::BP * RT::S1], 0.0};
        GatherAcc a;
        {
            const double fn = fma(c.nu_c, dt, 1.0), ft = fma(c.al_c, dt, 1.0);
            a = GatherAcc{fma(-6.0, (Q[ox] + Q[oy]) + cur.X, cur.lp), cur.l[0] * fn, cur.l[1] * fn, cur.l[2] * fn,
                          fma(cur.l[3], ft, cur.l[2] * dt)};
        }
        ReverseCell r;
        // the neighbour at LDS offset o, its X at oX; its velocity and T into f
        auto nbr = [&](int o, int oX, double f[NF - 1], int ax, double h2) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < NF - 1; ++m) f[m] = B[o + m * RT::S1];
            return Nbr{{B[o + RT::LU * RT::S1], B[o + RT::LV * RT::S1], B[o + RT::LW * RT::S1], B[o + RT::LT * RT::S1]},
                       Q[o + RT::DT * RT::S1], Q[oX], Q[o + RT::BP * RT::S1], f[ax] * h2};
        };
        // one in-plane axis: d1, dp, dX the LDS steps of the three layouts
        auto in_plane = [&](auto axis, int x, int n, bool bnd, int d1, int dp, int oX, int dX) __attribute__((always_inline)) {
            constexpr int AX = decltype(axis)::value;
            const double h2 = AX == 0 ? c.hx2 : c.hy2;
            double fl[NF - 1], fh[NF - 1];
            me.X = Q[oX];
            me.s = f0[AX] * h2;
            PHASE();
            {
                const Nbr lo = nbr(o1 - d1, oX - dX, fl, AX, h2);
                if (!bnd || x > 0) add_star<AX, 1>(a, c, lo);
                if (bnd && x <= 1) add_wall<AX, -1>(a, c, x, n, x == 0 ? me : lo, x == 0 ? Q[oX + dX] : me.X,
                                                    (AX == 0 && rows && active) ? &rows[j + (long long)d.nj * k] : nullptr);
            }
            PHASE();
            {
                const Nbr hi = nbr(o1 + d1, oX + dX, fh, AX, h2);
                if (!bnd || x < n - 1) add_star<AX, -1>(a, c, hi);
                if (bnd && x >= n - 2) add_wall<AX, 1>(a, c, x, n, x == n - 1 ? me : hi, x == n - 1 ? Q[oX - dX] : me.X, nullptr);
            }
            PHASE();
            if (!bnd || x >= 2) a.Lp -= Q[oX - 2 * dX];
            if (!bnd || x < n - 2) a.Lp -= Q[oX + 2 * dX];
            double pl = B[op - dp], ph = B[op + dp], pl2 = B[op - 2 * dp], ph2 = B[op + 2 * dp];
            if (bnd) axis_ghosts<AX>(c, x, n, tw, f0, cur.p, fl, fh, pl, ph, pl2, ph2);
            r.axis<AX>(c, cur.l, f0, cur.p, fl, fh, pl, ph, pl2, ph2);
            PHASE();
        };
        in_plane(std::integral_constant<int, 0>{}, i, d.ni, bnd_i, 1, 1, ox, 1);
        in_plane(std::integral_constant<int, 1>{}, j, d.nj, bnd_j, RT::W1, RT::WP, oy, 64);
        derive(nn2, Qnn);
        me.X = cur.X;
        me.s = cur.w * c.hz2;
        {
            const Nbr prv{{pa[0], pa[1], pa[2], pa[3]}, 1.0, pX, pBp, fm[2] * c.hz2};
            const Nbr hi{{nxt.l[0], nxt.l[1], nxt.l[2], nxt.l[3]}, Qn[o1 + RT::DT * RT::S1], nxt.X,
                         Qn[o1 + RT::BP * RT::S1], nxt.w * c.hz2};
            double fh[NF - 1] = {nxt.u, nxt.v, nxt.w, nxt.t}, ph = nxt.p, ph2 = nn2.p;
            if (k > 0) add_star<2, 1>(a, c, prv);
            if (k < nk - 1) add_star<2, -1>(a, c, hi);
            if (k >= 2) a.Lp -= xm2;
            if (k < nk - 2) a.Lp -= nn2.X;
            if (k <= 1) add_wall<2, -1>(a, c, k, nk, k == 0 ? me : prv, k == 0 ? hi.X : me.X, nullptr);
            if (k >= nk - 2) add_wall<2, 1>(a, c, k, nk, k == nk - 1 ? me : hi, k == nk - 1 ? prv.X : me.X, nullptr);
            if (k <= 1 || k >= nk - 2) axis_ghosts<2>(c, k, nk, 0.0, f0, cur.p, fm, fh, pm, ph, pm2, ph2);
            r.axis<2>(c, cur.l, f0, cur.p, fm, fh, pm, ph, pm2, ph2);
        }
        PHASE();
        const SeedTerms t = r.finish(c, cur.l, f0, cur.lp, dt);
        if (k == nk / 2 && centre_col) {
            // what the centre's unit p seed terms need, finished after the march
            // (here they cost registers the loop does not have)
            cx[0] = r.F[0]; cx[1] = r.F[1]; cx[2] = r.F[2]; cx[3] = r.div;
            cx[4] = f0[0]; cx[5] = f0[1]; cx[6] = f0[2]; cx[7] = dt;
        }
        a.Lu += t.ub;
        a.Lv += t.vb;
        a.Lw += t.wb;
        if (active) {
            acc_ra += t.ra;
            acc_s += cur.lp;
            const double v[NF] = {a.Lp, a.Lu, a.Lv, a.Lw, a.Lt};
            const long long kz = (k + NG) * Z;
#pragma unroll
            for (int f = 0; f < NF; ++f)
                __builtin_nontemporal_store(v[f], reinterpret_cast<double*>(reinterpret_cast<char*>(out + f * sf + kz) + ocol));
        }
        // Move the sets down a plane, before the next loads are issued: left to
        // the end of the loop, these copies make the loads write elsewhere, and
        // be waited for at once, to be copied in their turn.
        xm2 = moved(pX);
        pX = moved(cur.X);
        pBp = me.Bp;
#pragma unroll
        for (int f = 0; f < NF - 1; ++f) pa[f] = cur.l[f] * dt;
        fm[0] = moved(cur.u); fm[1] = moved(cur.v); fm[2] = moved(cur.w); fm[3] = moved(cur.t);
        pm2 = moved(pm);
        pm = moved(cur.p);
        cur.u = moved(nxt.u); cur.v = moved(nxt.v); cur.w = moved(nxt.w); cur.t = moved(nxt.t);
        cur.p = moved(nxt.p); cur.lp = moved(nxt.lp); cur.X = moved(nxt.X);
#pragma unroll
        for (int f = 0; f < NF - 1; ++f) cur.l[f] = moved(nxt.l[f]);
        nxt.u = moved(nn2.u); nxt.v = moved(nn2.v); nxt.w = moved(nn2.w);
        nxt.p = moved(nn2.p); nxt.lp = moved(nn2.lp); nxt.X = moved(nn2.X);
        PHASE();
        wall = wsrc[min(k + 1, k1 - 1) * wstep];
        load_l(min(k + 2, klast), nxt);
        load(min(k + 3, klast), nn2);
        const int t3 = oq;
        oq = oqn;
        oqn = oqnn;
        oqnn = t3;
    }

    if (centre_col && k0 <= nk / 2 && nk / 2 < k1) {
        // the centre's terms for a unit p seed (a_p = dt, b = R_p)
        const ReverseCell r1{{0.0, 0.0, 0.0}, {cx[0], cx[1], cx[2]}, 0.0, 0.0, 0.0, cx[3]};
        const double zero[NF - 1] = {0.0, 0.0, 0.0, 0.0}, f0[NF - 1] = {cx[4], cx[5], cx[6], c.t_inf};
        const SeedTerms t1 = r1.finish(c, zero, f0, 1.0, cx[7]);
        const CellD D1 = cell_d(c, f0[0], f0[1], f0[2], 1.0);
        cx[0] = t1.ub; cx[1] = t1.vb; cx[2] = t1.wb; cx[3] = t1.ra;
        cx[4] = D1.X[0]; cx[5] = D1.X[1]; cx[6] = D1.X[2]; cx[7] = D1.Bp;
    }

    // the block's Ra term and sum of lambda_p
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) {
        acc_ra += __shfl_xor(acc_ra, m, 64);
        acc_s += __shfl_xor(acc_s, m, 64);
    }
    __syncthreads();
    if (lane == 0) {
        L[2 * row] = acc_ra;
        L[2 * row + 1] = acc_s;
    }
    __syncthreads();
    if (tid < 2) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < TJ; ++w) t += L[2 * w + tid];
        part[(size_t)tb.pidx * NF + tid] = t;
    }
}

// The transpose of the centre rescale and the Ra sum, after the pass.  The
// pass seeds the centre cell with lambda_p; its seed is lambda_p - S, S the
// sum of lambda_p over the grid, and everything is linear in the seeds, so S
// times the response to a unit p seed is subtracted: 1 on lambda_p at the
// centre, and the centre's star cotangents for a_p = dt, b = R_p, all other
// seeds 0 (cx: ub, vb, wb, the Ra term, the dissipation terms, Bp), which
// land on the cells within two of the centre along an axis (a wall's ghosts
// map back onto such cells).  Lane 5 ax + step + 2 of the first wavefront
// holds the cell at `step` along axis ax.  One block; the sums run in a fixed
// order.  It is a chain of latencies (~5 us), so the code is kept short: with
// the centre's terms formed here it took 8.3 us.  Beside it, blocks from the
// second on add the wall rows' terms to dJ/dTheta, a row a thread, by plain
// loads and stores: the pass itself would wait for the old values (loaded a
// plane ahead, 256^3 1646 us for three steps against 1631), and an atomic add
// there is dropped in memory that is not the device's own.
constexpr int FIX_THREADS = 256;
__global__ __launch_bounds__(FIX_THREADS) void rescale_adjoint_kernel(Dims d, double hx2, double hy2, double hz2,
                                                                      const double* __restrict__ part, int nblocks,
                                                                      const double* __restrict__ cx, long long sf,
                                                                      double* __restrict__ out, double* __restrict__ dra,
                                                                      int nrows, const double* __restrict__ rows,
                                                                      double* __restrict__ dthot)
{
    if (blockIdx.x > 0) {
        const int r = (blockIdx.x - 1) * FIX_THREADS + threadIdx.x;
        if (r < nrows) dthot[r] += rows[r];
        return;
    }
    __shared__ double red[FIX_THREADS / 64][2];
    const int tid = threadIdx.x;
    double ra = 0.0, S = 0.0;
    for (int b = tid; b < nblocks; b += FIX_THREADS) {
        ra += part[(size_t)b * NF];
        S += part[(size_t)b * NF + 1];
    }
    // this lane's cell and its two values to change
    const int ax = min(tid / 5, 2), st = tid % 5 - 2;
    const int x = (ax == 0 ? d.ni : (ax == 1 ? d.nj : d.nk)) / 2 + st, n = ax == 0 ? d.ni : (ax == 1 ? d.nj : d.nk);
    const bool mine = tid < 15 && x >= 0 && x < n;
    double* const P = out + (mine ? cell_off(d, d.ni / 2 + (ax == 0 ? st : 0), d.nj / 2 + (ax == 1 ? st : 0),
                                             d.nk / 2 + (ax == 2 ? st : 0))
                                  : cell_off(d, 0, 0, 0));
    double* const V = P + (FU + ax) * sf;
    const double p0 = *P, v0 = *V;
    const double X = cx[4 + ax], B = cx[7] * (ax == 0 ? hx2 : (ax == 1 ? hy2 : hz2)), own = cx[ax], ura = cx[3];
    double Lp = st == 0 ? 0.0 : (st == 1 || st == -1 ? 4.0 * X : -X);
    double Lv = st == 1 ? -B : (st == -1 ? B : 0.0);
    // the wall rules: is m0, is m1 the centre
    auto wall = [&](bool at_m0, bool m0, bool m1, double Bs) __attribute__((always_inline)) {
        const double g1 = (m0 ? 4.0 * X : 0.0) - (m1 ? X : 0.0), g2 = m0 ? -X : 0.0;
        Lp += at_m0 ? 2.0 * g1 + 3.0 * g2 : -(g1 + 2.0 * g2);
        if (at_m0 && m0) Lv -= Bs;
    };
    if (x <= 1) wall(x == 0, st == (x == 0 ? 0 : 1), st == (x == 0 ? -1 : 0), B);
    if (x >= n - 2) wall(x == n - 1, st == (x == n - 1 ? 0 : -1), st == (x == n - 1 ? 1 : 0), -B);
    if (tid < 64) {
        const double c3 = (__shfl(Lp, 2, 64) + __shfl(Lp, 7, 64)) + __shfl(Lp, 12, 64);
        if (st == 0) {
            Lp = ((1.0 - 6.0 * ((cx[4] + cx[5]) + cx[6])) + c3);
            Lv += own;
        }
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) {
        ra += __shfl_xor(ra, m, 64);
        S += __shfl_xor(S, m, 64);
    }
    if ((tid & 63) == 0) {
        red[tid >> 6][0] = ra;
        red[tid >> 6][1] = S;
    }
    __syncthreads();
    ra = S = 0.0;
#pragma unroll
    for (int w = 0; w < FIX_THREADS / 64; ++w) {
        ra += red[w][0];
        S += red[w][1];
    }
    if (tid == 0 && dra) dra[0] += ra - S * ura;
    if (!mine) return;
    if (st != 0 || ax == 0) *P = p0 - S * Lp;
    if (st > -2 && st < 2) *V = v0 - S * Lv;
}

// ---- cotangent of the mean hot-wall Nusselt number ----
// Nu = sum over (j, k) of -(9 T_0 - T_1 - 8 T_wall) * ni / 3 / (nj nk dT):
// writes lambda (zero except T at i = 0, 1) and adds dNu/dT_wall.
__global__ __launch_bounds__(ADJ_THREADS) void nusselt_seed_kernel(Dims d, double scale, StateT<double> lam,
                                                                   double* __restrict__ dthot)
{
    const long long n = (long long)d.ni * d.nj * d.nk;
    const long long idx = (long long)blockIdx.x * ADJ_THREADS + threadIdx.x;
    if (idx >= n) return;
    const int i = (int)(idx % d.ni);
    const long long r = idx / d.ni;
    const int j = (int)(r % d.nj), k = (int)(r / d.nj);
    const int o = cell_off(d, i, j, k);
#pragma unroll
    for (int f = FP; f < FT; ++f) lam.f[f][o] = 0.0;
    lam.f[FT][o] = i == 0 ? -9.0 * scale : (i == 1 ? scale : 0.0);
    if (i == 0 && dthot) dthot[j + (long long)d.nj * k] += 8.0 * scale;
}

// Partials of the pass: one per block of any k-chunk tiling (the chunking
// never yields more than nk/CAV_MIN_KC chunks per tile column), NF doubles
// apart.
long long reverse_partials(const Dims& d)
{
    const long long tiles = (long long)((d.ni + SW_TI - 1) / SW_TI) * ((d.nj + SW_TJ - 1) / SW_TJ);
    return tiles * std::max(1, d.nk / CAV_MIN_KC) * NF;
}

}  // namespace

// ---------------------------------------------------------------------------
// The size callers have allocated since the step stored 8 values per cell; it
// uses the 8 head doubles, the partials and a double per wall row.
size_t adjoint_ws_doubles(const Dims& d)
{
    const long long n = (long long)d.ni * d.nj * d.nk;
    return (size_t)(8 + (reverse_partials(d) + 7) / 8 * 8 + (long long)NREC * n);
}

hipError_t launch_adjoint_step(const Dims& d, const Coef& c, const SweepGeom& g, double Ra, CStateT<double> q,
                               CStateT<double> lam_in, StateT<double> lam_out, double* ws, double* dthot, double* dra,
                               hipStream_t s)
{
    double* cx = ws;                         // the centre's unit p seed terms
    double* part = ws + 8;
    double* rows = dthot ? part + (reverse_partials(d) + 7) / 8 * 8 : nullptr;     // the wall rows' terms
    const int nrows = dthot ? d.nj * d.nk : 0;
    if ((long long)g.nblocks * NF > reverse_partials(d)) return hipErrorInvalidValue;
    const long long sf = q.f[1] - q.f[0];
    const RevCoef rc{{c.hx2, c.hy2, c.hz2, c.ix2, c.iy2, c.iz2, c.eps4, c.beta2_floor, c.nu, c.alpha, c.t_inf, c.cfl,
                      c.dt_visc, c.t_hot, c.t_cold, c.t_hot_field},
                     {-c.nu / (2.0 * Ra), -c.alpha / (2.0 * Ra), c.dt_visc / (2.0 * Ra)},
                     {c.nu * c.ix2, c.nu * c.iy2, c.nu * c.iz2},
                     {c.alpha * c.ix2, c.alpha * c.iy2, c.alpha * c.iz2},
                     -2.0 * c.nu * ((c.ix2 + c.iy2) + c.iz2),
                     -2.0 * c.alpha * ((c.ix2 + c.iy2) + c.iz2)};
    reverse_tile_kernel<SW_TJ><<<g.nblocks, dim3(SW_TI, SW_TJ), 0, s>>>(d, rc, g, sf, q.f[0], lam_in.f[0], lam_out.f[0],
                                                                        part, cx, rows);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    rescale_adjoint_kernel<<<1 + (nrows + FIX_THREADS - 1) / FIX_THREADS, FIX_THREADS, 0, s>>>(
        d, c.hx2, c.hy2, c.hz2, part, g.nblocks, cx, sf, lam_out.f[0], dra, nrows, rows, dthot);
    return hipGetLastError();
}

hipError_t launch_nusselt_seed(const Dims& d, double scale, StateT<double> lam, double* dthot, hipStream_t s)
{
    const long long n = (long long)d.ni * d.nj * d.nk;
    nusselt_seed_kernel<<<(unsigned)((n + ADJ_THREADS - 1) / ADJ_THREADS), ADJ_THREADS, 0, s>>>(d, scale, lam,
                                                                                               dthot);
    return hipGetLastError();
}

}  // namespace cav
