// The k-marching tile of the sweep (sweep.hip: the step, the batched form and
// the interior/exterior split); its tile boxes serve the adjoint's tile too.
// Built with -ffp-contract=off.
#pragma once

#include "cavity_internal.h"
#include "stencil.h"

namespace cav {

// ---------------------------------------------------------------------------
// The sweep.  Block = one TI x TJ tile of (i, j) columns, i along the lanes
// (64 x 8: one wavefront per j row; narrower tiles put 64 / TI rows in a
// wavefront) marching over a chunk of k planes.  Plane k of
// all five fields lives in LDS with its i/j halo (2 for p, 1 for the rest);
// the k neighbours come from per-thread register queues (p: k-2..k+2,
// others k-1..k+1).  The LDS planes are double-buffered: plane k+1 is
// written into one buffer while plane k is computed from the other, so each
// plane costs one barrier; global loads run two planes ahead.  Wall ghosts
// are derived from interior cells (in each cell's star for the i/j walls, by
// recurrences on the queues for the k walls); no ghost cell is read from HBM.
// LDS of one sweep block of TI x TJ threads: two planes of p (halo 2) and
// of u, v, w, T (halo 1), and one norm slot per wavefront.
template <typename Real, int TI_ = SW_TI, int TJ_ = SW_TJ>
struct SweepLds {
    static constexpr int TI = TI_, TJ = TJ_;
    static constexpr int PW = TI + 4;              // row pitch, p
    static constexpr int UW = TI + 2;              // row pitch, u v w T
    static constexpr int PPL = (TJ + 4) * PW;      // plane, p
    static constexpr int UPL = (TJ + 2) * UW;      // plane, one of u v w T
    static constexpr int NWAVE = TI * TJ / 64;
    Real p[2 * PPL];
    Real u[2 * 4 * UPL];
    double red[NWAVE][NF];
};

// What a sweep does with each cell's stars and residual: the pseudo-time
// update of Sec. 2 (q + dt R, then the centre rescale of p) streamed into
// qn, and R^2 into the norm accumulators.
// STREAM: by non-temporal stores (stream_out; compiled in, since of the two
// kinds of store under a condition the compiler makes one).
template <typename Real, bool STREAM>
struct StepEpi {
    StateT<Real> qn;
    Real pc_new;
    __device__ __forceinline__ void store(const Real v[NF], int o)
    {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (STREAM) __builtin_nontemporal_store(v[f], &qn.f[f][o]);
            else qn.f[f][o] = v[f];
        }
    }
    // New pressure at the centre cell, recomputed with the same arithmetic
    // as its owner, so that every block subtracts the identical value.
    __device__ __forceinline__ void prepare(const Dims& d, const CStateT<Real>& q, const CoefR<Real>& c)
    {
        Star<Real> s;
        point_star(d, q, c, centre_cell<Real>(d), s);
        Real R[NF], dt;
        cell_residual(c, s, R, dt);
        pc_new = fma(dt, R[FP], s.p);
    }
    __device__ __forceinline__ void cell(const CoefR<Real>&, const Star<Real>& s, const Real R[NF], Real dt, int o,
                                         int, int, int, double acc[NF])
    {
        const Real v[NF] = {fma(dt, R[FP], s.p) - pc_new, fma(dt, R[FU], s.u), fma(dt, R[FV], s.v),
                            fma(dt, R[FW], s.w), fma(dt, R[FT], s.t)};
        store(v, o);
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f] = fma((double)R[f], (double)R[f], acc[f]);
    }
};

// Where one block works: columns [i0, i0+TI) x [j0, j0+TJ), planes
// [k0, k1); its norm partial goes to slot pidx.
struct TileBox {
    int i0, j0, k0, k1, pidx;
};

// Logical tile b of the regular TI x TJ tiling with k chunks of length kc.
template <int TI = SW_TI, int TJ = SW_TJ>
__device__ __forceinline__ TileBox tile_box(const Dims& d, int tiles_i, int tiles_j, int kc, int b)
{
    const int bi = b % tiles_i;
    const int bj = (b / tiles_i) % tiles_j;
    const int bk = b / (tiles_i * tiles_j);
    TileBox t;
    t.i0 = bi * TI;
    t.j0 = bj * TJ;
    t.k0 = bk * kc;
    t.k1 = min(t.k0 + kc, d.nk);
    t.pidx = b;
    return t;
}

// Every cell of the box is updated.  column(i, j): whether any updated cell
// reads column (i, j).
struct OwnAll {
    __device__ __forceinline__ bool operator()(int, int, int) const { return true; }
    __device__ __forceinline__ bool column(int, int) const { return true; }
};

// One tile box: planes of its k range, cells for which own(i, j, k) holds
// are updated (and enter the norm).  Used by the single-cavity sweep, the
// batched kernel and the interior/exterior split.  The block has TI x TJ =
// 512 or 256 threads, launched as SW_TI x (TI TJ / SW_TI): thread t = lane +
// TI * row works on column (i0 + lane, j0 + row).
// Where a thread's column comes from: the state.  (A sweep that does the
// exchange of a split along i has another, sweep.hip.)
template <typename Real>
struct StateColumn {
    const Real* p[NF];
    long long Z;
    __device__ __forceinline__ void init(const Dims& d, const CStateT<Real>& q, const TileBox&, int, int, int off)
    {
#pragma unroll
        for (int f = 0; f < NF; ++f) p[f] = q.f[f] + off;
        Z = d.sz;
    }
    __device__ __forceinline__ Real operator()(int f, int k) const { return p[f][k * Z]; }
};

template <typename Real, bool NORM, typename Own, typename Epi, int TI = SW_TI, int TJ = SW_TJ,
          typename Column = StateColumn<Real>>
__device__ __forceinline__ void sweep_tile(const Dims& d, const CoefR<Real>& c, const TileBox& tb, const Own& own,
                                           const CStateT<Real>& q, Epi& epi, double* partials,
                                           SweepLds<Real, TI, TJ>& L, Column C = Column{})
{
    constexpr int THREADS = TI * TJ;
    static_assert((THREADS == 512 || THREADS == 256) && TJ >= 8 && 4 * TI + 12 * TJ <= THREADS,
                  "512- or 256-thread tiles whose halo is two loads a thread");
    using Lds = SweepLds<Real, TI, TJ>;
    constexpr int PW = Lds::PW, UW = Lds::UW;
    constexpr int PPL = Lds::PPL, UPL = Lds::UPL;
    Real* const sP = L.p;
    Real* const sU = L.u;

    const int i0 = tb.i0, j0 = tb.j0;
    const int k0 = tb.k0, k1 = tb.k1;

    // launched as SW_TI x (TI TJ / SW_TI) threads; other shapes re-split the block
    const int tid = threadIdx.x + SW_TI * threadIdx.y;
    const int lane = TI == SW_TI ? (int)threadIdx.x : tid % TI;
    const int row = TI == SW_TI ? (int)threadIdx.y : tid / TI;
    const int i = i0 + lane, j = j0 + row;
    // columns no owned cell's star reaches are not computed
    const bool active = i < d.ni && j < d.nj && own.column(i, j);

    // ---- what this thread loads (fixed for the whole march) ----
    // Per plane every thread loads the five fields of its column and two halo
    // values, whatever its place: threads past the grid, or with no halo value
    // of their own, repeat a neighbour's address.  A load under a condition
    // would be taken as not issued by the waits that follow it, which then
    // wait for younger loads too and undo the look-ahead.  Only interior cells
    // are loaded.  LDS cells beyond a wall are read only into star values that
    // star_ghosts_axis then replaces; the k neighbours beyond the z walls come
    // by recurrences on the queues.
    auto interior = [&](int ii, int jj) { return ii >= 0 && ii < d.ni && jj >= 0 && jj < d.nj; };
    const int off_c = cell_off(d, min(i, d.ni - 1), min(j, d.nj - 1), 0);
    const long long fs = q.f[FU] - q.f[FP];          // elements per field
    // halo value A: u v w T rows j0-1, j0+TJ, slot s = tid / TI = 0..7 is
    // field 1 + s/2, side s&1
    const Real* srcA = q.f[FP] + off_c;
    bool hasA = false;
    int dstA = 0;
    if (tid < 8 * TI) {
        const int sl = tid / TI, ul = (sl & 1) ? TJ + 1 : 0, uj = j0 - 1 + ul, ui = i0 + tid % TI;
        hasA = interior(ui, uj) && own.column(ui, uj);
        dstA = (sl >> 1) * UPL + ul * UW + tid % TI + 1;
        if (hasA) srcA = q.f[FP] + (FU + (sl >> 1)) * fs + cell_off(d, ui, uj, 0);
    }
    // halo value B: p rows j0-2, j0-1, j0+TJ, j0+TJ+1, then the columns: per
    // row, p at i0-2, i0-1, i0+TI, i0+TI+1 and u v w T at i0-1, i0+TI
    const Real* srcB = q.f[FP] + off_c;
    bool hasB = false, pB = true;
    int dstB = 0;
    if (tid < 4 * TI) {
        const int r = tid / TI, pl = r < 2 ? r : TJ + r, pj = j0 - 2 + pl, pi = i0 + tid % TI;
        hasB = interior(pi, pj) && own.column(pi, pj);
        dstB = pl * PW + tid % TI + 2;
        if (hasB) srcB = q.f[FP] + cell_off(d, pi, pj, 0);
    } else if (tid < 4 * TI + 12 * TJ) {
        const int h = tid - 4 * TI, r = h / 12, m = h % 12;
        int f = FP, cc, ci;
        if (m < 4) {
            cc = m < 2 ? m : TI + m;
            ci = i0 - 2 + cc;
            dstB = (r + 2) * PW + cc;
        } else {
            const int t = m - 4;
            f = FU + (t >> 1);
            cc = (t & 1) ? TI + 1 : 0;
            ci = i0 - 1 + cc;
            dstB = (t >> 1) * UPL + (r + 1) * UW + cc;
            pB = false;
        }
        hasB = interior(ci, j0 + r);
        if (hasB) srcB = q.f[FP] + f * fs + cell_off(d, ci, j0 + r, 0);
    }
    C.init(d, q, tb, i, j, off_c);
    const long long Z = d.sz;

    // tiles whose stars reach past an i or j wall (block-uniform)
    const bool bnd_i = i0 == 0 || i0 + TI + 2 > d.ni, bnd_j = j0 == 0 || j0 + TJ + 2 > d.nj;

    // ---- register queues ----
    Real p0, p1, p2, p3;                                 // p at k-2, k-1, k, k+1
    Real u0, u1, v0, v1, w0, w1, t0, t1;                 // at k-1, k
    const int lc_p = (row + 2) * PW + lane + 2;            // this cell in an LDS p plane
    const int lc_u = (row + 1) * UW + lane + 1;            // this cell in an LDS u v w T plane
    {
        // planes k0-2 .. k0+1 of this column; planes beyond the z walls
        // follow from the wall rules (recurrences along k)
        Real P[4], U[2], V[2], W[2], T[2];
        for (int m = 0; m < 4; ++m) P[m] = C(FP, max(0, min(k0 - 2 + m, d.nk - 1)));
        for (int m = 0; m < 2; ++m) {
            const int kk = max(0, k0 - 1 + m);
            U[m] = C(FU, kk);
            V[m] = C(FV, kk);
            W[m] = C(FW, kk);
            T[m] = C(FT, kk);
        }
        if (k0 + 1 >= d.nk) P[3] = Real(2) * P[2] - P[1];
        for (int m = 1; m >= 0; --m)
            if (k0 - 2 + m < 0) P[m] = Real(2) * P[m + 1] - P[m + 2];
        if (k0 - 1 < 0) { U[0] = -U[1]; V[0] = -V[1]; W[0] = -W[1]; T[0] = T[1]; }
        p0 = P[0]; p1 = P[1]; p2 = P[2]; p3 = P[3];
        u0 = U[0]; u1 = U[1]; v0 = V[0]; v1 = V[1]; w0 = W[0]; w1 = W[1]; t0 = T[0]; t1 = T[1];
    }
    // plane k0 into LDS buffer 0
    sP[lc_p] = p2;
    sU[0 * UPL + lc_u] = u1;
    sU[1 * UPL + lc_u] = v1;
    sU[2 * UPL + lc_u] = w1;
    sU[3 * UPL + lc_u] = t1;
    if (hasA) sU[dstA] = srcA[k0 * Z];
    if (hasB) (pB ? sP : sU)[dstB] = srcB[k0 * Z];

    // Loads run two planes ahead: what the iteration for plane k needs from
    // memory (queue heads p(k+2), uvwT(k+1), halo values of plane k+1) is
    // issued while plane k-2 is computed; two register sets alternate.
    struct InFlight {
        Real p, u, v, w, t, a, b;
    };
    const int kp = min(k1 + 1, d.nk - 1), ku = min(k1, d.nk - 1), kh = k1 - 1;   // last planes needed
    auto issue = [&](InFlight& F, int k) __attribute__((always_inline)) {
        const int kk = min(k + 1, ku);
        const long long hz = min(k + 1, kh) * Z;
        F.p = C(FP, min(k + 2, kp));
        F.u = C(FU, kk);
        F.v = C(FV, kk);
        F.w = C(FW, kk);
        F.t = C(FT, kk);
        F.a = srcA[hz];
        F.b = srcB[hz];
    };
    InFlight X, Y;
    issue(X, k0);
    issue(Y, k0 + 1);
    // the epilogue's per-block setup (for the step: the centre cell's new
    // pressure, a star gathered from L2) overlaps the loads in flight
    epi.prepare(d, q, c);
    __syncthreads();

    double acc[NF] = {0.0, 0.0, 0.0, 0.0, 0.0};
    int buf = 0;

    auto plane = [&](InFlight& F, int k) __attribute__((always_inline)) {
        // complete the queues; planes past the top wall follow the wall rules
        const Real p4 = k + 2 < d.nk ? F.p : Real(2) * p3 - p2;
        const bool in1 = k + 1 < d.nk;
        const Real u2 = in1 ? F.u : -u1, v2 = in1 ? F.v : -v1, w2 = in1 ? F.w : -w1, t2 = in1 ? F.t : t1;
        if (k + 1 < k1) {
            // plane k+1 into the other LDS buffer (its last readers finished
            // before the barrier that ended the previous plane)
            Real* const nP = sP + (buf ^ 1) * PPL;
            Real* const nU = sU + (buf ^ 1) * 4 * UPL;
            nP[lc_p] = p3;
            nU[0 * UPL + lc_u] = u2;
            nU[1 * UPL + lc_u] = v2;
            nU[2 * UPL + lc_u] = w2;
            nU[3 * UPL + lc_u] = t2;
            if (hasA) nU[dstA] = F.a;
            if (hasB) (pB ? nP : nU)[dstB] = F.b;
        }
        issue(F, k + 2);

        Real* const cP = sP + buf * PPL;
        Real* const cU = sU + buf * 4 * UPL;
        if (active && own(i, j, k)) {
            Star<Real> s;
            s.p = p2;
            s.pxm = cP[lc_p - 1]; s.pxp = cP[lc_p + 1]; s.pxm2 = cP[lc_p - 2]; s.pxp2 = cP[lc_p + 2];
            s.pym = cP[lc_p - PW]; s.pyp = cP[lc_p + PW]; s.pym2 = cP[lc_p - 2 * PW]; s.pyp2 = cP[lc_p + 2 * PW];
            s.pzm = p1; s.pzp = p3; s.pzm2 = p0; s.pzp2 = p4;
#define STAR_LDS(nm, pl, c0, cm, cp)                                               \
            s.nm = c0; s.nm##zm = cm; s.nm##zp = cp;                               \
            s.nm##xm = cU[pl * UPL + lc_u - 1]; s.nm##xp = cU[pl * UPL + lc_u + 1]; \
            s.nm##ym = cU[pl * UPL + lc_u - UW]; s.nm##yp = cU[pl * UPL + lc_u + UW];
            STAR_LDS(u, 0, u1, u0, u2)
            STAR_LDS(v, 1, v1, v0, v2)
            STAR_LDS(w, 2, w1, w0, w2)
            STAR_LDS(t, 3, t1, t0, t2)
#undef STAR_LDS
            if (bnd_i && __any(i < 2 || i >= d.ni - 2)) star_ghosts_axis<0>(i, d.ni, s, c, d, j, k);
            if (bnd_j && __any(j < 2 || j >= d.nj - 2)) star_ghosts_axis<1>(j, d.nj, s, c, d, j, k);
            Real R[NF], dt;
            cell_residual(c, s, R, dt);
            epi.cell(c, s, R, dt, off_c + k * d.sz, i, j, k, acc);
        }
        __syncthreads();
        buf ^= 1;
        p0 = p1; p1 = p2; p2 = p3; p3 = p4;
        u0 = u1; u1 = u2; v0 = v1; v1 = v2; w0 = w1; w1 = w2; t0 = t1; t1 = t2;
    };

    // pairs of planes, then a last odd one (a way out of the middle of the
    // loop would join its back edge with one set of loads not yet issued)
    int k = k0;
    for (; k + 1 < k1; k += 2) {
        plane(X, k);
        plane(Y, k + 1);
    }
    if (k < k1) plane(X, k);

    if (NORM) {
        // fixed-order block reduction: butterfly within the wavefront, then
        // the wavefront sums in order
        auto& red = L.red;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            double v = acc[f];
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
            acc[f] = v;
        }
        const int wl = tid & 63, wv = tid >> 6;
        if (wl == 0) {
#pragma unroll
            for (int f = 0; f < NF; ++f) red[wv][f] = acc[f];
        }
        __syncthreads();
        if (tid < NF) {
            double t = 0.0;
#pragma unroll
            for (int r = 0; r < Lds::NWAVE; ++r) t += red[r][tid];
            partials[(size_t)tb.pidx * NF + tid] = t;
        }
    }
}

}  // namespace cav
