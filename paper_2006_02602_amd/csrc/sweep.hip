// Residual + Euler-update sweep kernels (single cavity, interior/exterior
// split, batched), wall boundary conditions, seeded init, the hot-wall
// Nusselt integral and the residual-norm finalize for gfx950, in FP64 and
// FP32 (the per-cell code is in stencil.h, the k-marching tile in
// sweep_tile.h).
//
// The method (Xue & Roy, arXiv:2006.02602): artificial-compressibility
// Boussinesq equations (Sec. 2, Eq. 1-3), second-order central differences
// with a fourth-difference pressure dissipation (5-point p stencil, 3-point
// stencils for u, v, w, T; Sec. 3.1), first-order explicit Euler in pseudo
// time, wall boundary conditions and the pressure rescale at the cavity
// centre in every iteration (Sec. 2).
//
// This file is compiled with -ffp-contract=off: every fused multiply-add is
// written out with fma(), so two inlined copies of the per-cell update round
// identically (the centre-cell rescale relies on that).
#include "cavity_internal.h"
#include "stencil.h"
#include "sweep_tile.h"

namespace cav {

// Tile of the step sweep: FP64 64 x 8 (eight wavefronts; at its register
// count, 196, one block per compute unit), FP32 32 x 8 (four wavefronts; 135
// registers, three resident blocks per compute unit, whose barriers
// interleave; 126 and four blocks measured the same).
template <typename Real>
struct StepTile {
    static constexpr int TI = sizeof(Real) == 4 ? F32_TI : F64_TI;
    static constexpr int TJ = sizeof(Real) == 4 ? F32_TJ : F64_TJ;
    static constexpr int THREADS = TI * TJ;
};

// The exchange of a split along i only, inside the sweep (Sec. 4.5: the
// noncontiguous i faces that "Optimized V1" packs).  A lane whose column lies
// within a face width of a cut takes its column's values from the halo buffer
// instead of the state (the unpack), and stores the new values of its cell at
// their places in the buffer as well (the pack of the next step's exchange;
// the layout is halo_pack's).  Needs every subdomain extent along i >= 2 x the
// largest width, so that a column lies in at most one face box.
struct XGeom {
    int ex, pi;          // subdomain extent along i, subdomains along i
    int nj;              // face rows per plane (the split is along i only)
    int area;            // face area nj * nk
    int wsum;
    int w[NF], wpre[NF];
};

// A column's place in the buffer.
struct XColumn {
    int dd = -1;     // distance of the column to its cut (< the largest width), or -1: no face
    int face;        // 0: the -i face of the column's subdomain, 1: its +i face
    int seg;         // element offset of that face's segment in the buffer

    __device__ __forceinline__ void init(const XGeom& x, const Dims& d, int i, int j)
    {
        dd = -1;
        if (i >= d.ni || j >= d.nj) return;
        int wmax = 0;
#pragma unroll
        for (int f = 0; f < NF; ++f) wmax = max(wmax, x.w[f]);
        const int a = i / x.ex;
        const int lo = i - a * x.ex, hi = x.ex - 1 - lo;
        if (a > 0 && lo < wmax) { face = 0; dd = lo; }
        else if (a < x.pi - 1 && hi < wmax) { face = 1; dd = hi; }
        // segments in subdomain order, -i before +i face (buffer layout):
        // subdomain 0 has only its +i face, the others both (the last one
        // only its -i face)
        seg = (a > 0 ? 2 * a - 1 + face : 0) * x.area * x.wsum;
    }
    __device__ __forceinline__ bool has(const XGeom& x, int f) const { return dd >= 0 && dd < x.w[f]; }
    // element of field f at row j, plane k
    __device__ __forceinline__ int at(const XGeom& x, int f, int j, int k) const
    {
        const int w = x.w[f];
        return seg + x.wpre[f] * x.area + (k * x.nj + j) * w + (face ? w - 1 - dd : dd);
    }
};

// The unpack, in the column's loads: planes of this block's own chunk come
// from the buffer.  (Planes of a neighbouring chunk come from the state, which
// holds the same values: that chunk's block may already be packing its new
// ones.  A cell's own place is read before it is written, by this thread.)
template <typename Real>
struct ExchangedColumn {
    StateColumn<Real> s;
    const Real* buf;
    XGeom x;
    XColumn c;
    int j, k0, k1;
    __device__ __forceinline__ void init(const Dims& d, const CStateT<Real>& q, const TileBox& tb, int i, int jj, int off)
    {
        s.init(d, q, tb, i, jj, off);
        c.init(x, d, i, jj);
        j = jj;
        k0 = tb.k0;
        k1 = tb.k1;
    }
    __device__ __forceinline__ Real operator()(int f, int k) const
    {
        const Real* a = s.p[f] + k * s.Z;
        if (c.has(x, f) && k >= k0 && k < k1) a = buf + c.at(x, f, j, k);
        return *a;
    }
};

// The pack, in the step's epilogue.
template <typename Real, bool STREAM>
struct StepXPackEpi : StepEpi<Real, STREAM> {
    Real* buf;
    XColumn c;
    XGeom x;
    __device__ __forceinline__ void cell(const CoefR<Real>&, const Star<Real>& s, const Real R[NF], Real dt, int o,
                                         int, int j, int k, double acc[NF])
    {
        const Real nv[NF] = {fma(dt, R[FP], s.p) - this->pc_new, fma(dt, R[FU], s.u), fma(dt, R[FV], s.v),
                             fma(dt, R[FW], s.w), fma(dt, R[FT], s.t)};
        this->store(nv, o);
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f] = fma((double)R[f], (double)R[f], acc[f]);
        if (c.dd < 0) return;
#pragma unroll
        for (int f = 0; f < NF; ++f)
            if (c.has(x, f)) buf[c.at(x, f, j, k)] = nv[f];
    }
};

// FIELD = false: the hot wall is the scalar t_hot, known at compile time to
// need no field loads (the kernel the uniform-wall problem runs).  X: 1 the
// exchange's unpack in the loads, 2 also the next one's pack in the epilogue
// (buffer xbuf, geometry xg).
template <typename Real, bool NORM, bool FIELD, int X, bool STREAM>
__global__ __launch_bounds__(StepTile<Real>::THREADS) void sweep_kernel(
    Dims d, Coef cd, SweepGeom g, CStateT<Real> q, StateT<Real> qn, double* partials, XGeom xg, Real* xbuf)
{
    constexpr int TI = StepTile<Real>::TI, TJ = StepTile<Real>::TJ;
    __shared__ SweepLds<Real, TI, TJ> L;
    CoefR<Real> c = coef_as<Real>(cd);
    if constexpr (!FIELD) c.t_hot_field = nullptr;
    const TileBox tb = tile_box<TI, TJ>(d, g.tiles_i, g.tiles_j, g.kc, xcd_block(blockIdx.x, g.nblocks));
    if constexpr (X) {
        ExchangedColumn<Real> col;
        col.buf = xbuf;
        col.x = xg;
        if constexpr (X == 2) {
            StepXPackEpi<Real, STREAM> epi;
            epi.qn = qn;
            epi.pc_new = Real(0);
            epi.x = xg;
            epi.buf = xbuf;
            const int tid = threadIdx.x + SW_TI * threadIdx.y;
            epi.c.init(xg, d, tb.i0 + tid % TI, tb.j0 + tid / TI);
            sweep_tile<Real, NORM, OwnAll, StepXPackEpi<Real, STREAM>, TI, TJ>(d, c, tb, OwnAll{}, q, epi, partials, L, col);
        } else {
            StepEpi<Real, STREAM> epi{qn, Real(0)};
            sweep_tile<Real, NORM, OwnAll, StepEpi<Real, STREAM>, TI, TJ>(d, c, tb, OwnAll{}, q, epi, partials, L, col);
        }
    } else {
        StepEpi<Real, STREAM> epi{qn, Real(0)};
        sweep_tile<Real, NORM, OwnAll, StepEpi<Real, STREAM>, TI, TJ>(d, c, tb, OwnAll{}, q, epi, partials, L);
    }
}

// ---------------------------------------------------------------------------
// The step of a small grid: one cell per thread, its star read straight from
// global memory (L2 and the memory-side cache hold the state), no k march.
// A launch of the marching tile lasts ~8 us (FP64) however few planes its
// blocks march: start-up of the queues and planes, then a chain of barriers.
// Here the chain is one round of independent loads, one residual and the
// stores.  Per step, without norms, marching tile -> this kernel: FP64 16^3
// 7.9 -> 4.6 us, 48^3 8.3 -> 6.2, 80^3 16.1 -> 14.9; FP32 16^3 5.4 -> 4.4,
// 64^3 6.1 -> 5.9, 84x88x94 12.8 -> 10.2.
//
// A block is CELLS cells, consecutive in (k, j, i) order whatever the extents
// (no idle lanes at ragged ones), and one more wavefront that updates the
// centre cell for the rescale while the others update theirs.  FP64 is bound
// by the loads of its stars (41 of 512 bytes a wavefront): the x neighbours
// are moved between lanes (29 loads; 96^3 24.0 -> 21.4 us), and 7 + 1
// wavefronts make two blocks fill a compute unit at four wavefronts per SIMD
// (106 registers).  FP32 is bound by its instructions and loads all 41 (moves:
// 160^3 38 -> 40 us).  SMALL (FP64, up to 128 blocks of 448 cells): 192 cells
// a block, which spread over more units: 16^3 5.5 -> 4.6 us, 36^3 5.7 -> 5.0;
// 40^3 is even (5.6) and 48^3 loses (5.9 -> 6.7).  The norm pass writes a partial
// per 512 (FP64) or 256 (FP32) cells, which the workspace always holds.
template <typename Real, bool NORM, bool SMALL>
struct PointSweep {
    static constexpr bool F32 = sizeof(Real) == 4;
    static constexpr int CELLS = NORM ? (F32 ? 256 : 512) : (SMALL ? 192 : POINT_CELLS);
    static constexpr int THREADS = CELLS + 64;
};

template <typename Real, bool NORM, bool SMALL>
__device__ __forceinline__ void point_sweep(const Dims& d, const CoefR<Real>& c, const CStateT<Real>& q,
                                            const StateT<Real>& qn, int blk, double* partials)
{
    constexpr int CELLS = PointSweep<Real, NORM, SMALL>::CELLS;
    __shared__ Real pc;
    __shared__ double red[NORM ? CELLS / 64 : 1][NF];
    const int tid = threadIdx.x;
    const int n = d.ni * d.nj * d.nk;
    // the last wavefront's cells: 64 consecutive ones with the centre among them
    const bool extra = tid >= CELLS;
    const int mc = d.ni / 2 + d.ni * (d.nj / 2 + d.nj * (d.nk / 2));
    const int m = extra ? max(0, min(mc - 32, n - 64)) + tid - CELLS : blk * CELLS + tid;
    const bool in = !extra && m < n;
    const int mm = min(m, n - 1);
    const int r = mm / d.ni;
    const int i = mm - r * d.ni, k = r / d.nj, j = r - k * d.nj;
    const PointCell e = point_cell<Real>(d, i, j, k, 0);
    Star<Real> s;
    point_star<Real, !PointSweep<Real, NORM, SMALL>::F32>(d, q, c, e, s);
    Real R[NF], dt;
    cell_residual(c, s, R, dt);
    if (extra && m == mc) pc = fma(dt, R[FP], s.p);
    __syncthreads();
    auto put = [&](int f, Real v) __attribute__((always_inline)) {
        *reinterpret_cast<Real*>(reinterpret_cast<char*>(qn.f[f]) + e.o) = v;
    };
    if (in) {
        put(FP, fma(dt, R[FP], s.p) - pc);
        put(FU, fma(dt, R[FU], s.u));
        put(FV, fma(dt, R[FV], s.v));
        put(FW, fma(dt, R[FW], s.w));
        put(FT, fma(dt, R[FT], s.t));
    }
    if (NORM) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            double v = in ? (double)R[f] * (double)R[f] : 0.0;
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) v += __shfl_xor(v, x, 64);
            if ((tid & 63) == 0 && !extra) red[tid >> 6][f] = v;
        }
        __syncthreads();
        if (tid < NF) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < CELLS / 64; ++w) t += red[w][tid];
            partials[(size_t)blk * NF + tid] = t;
        }
    }
}

template <typename Real, bool NORM, bool SMALL>
__global__ __launch_bounds__((PointSweep<Real, NORM, SMALL>::THREADS)) void point_sweep_kernel(
    Dims d, Coef cd, CStateT<Real> q, StateT<Real> qn, double* partials)
{
    point_sweep<Real, NORM, SMALL>(d, coef_as<Real>(cd), q, qn, xcd_block(blockIdx.x, gridDim.x), partials);
}

// The step sweep's memory streams without its work: the same tiles, block
// order, k chunks and prefetch depth, and per interior cell the five fields
// read once and written once (non-temporal) -- no halo loads, no LDS, no
// arithmetic.  Its rate is the ceiling of the sweep's access pattern on the
// device it runs on where the sweep streams as well: on states past the
// caches (stream_out).  Where the sweep leaves its state in the caches, or
// runs one cell per thread, the sweep may be the faster.
template <typename Real>
__global__ __launch_bounds__(StepTile<Real>::THREADS) void stream_copy_kernel(Dims d, SweepGeom g, CStateT<Real> q,
                                                                              StateT<Real> qn)
{
    constexpr int TI = StepTile<Real>::TI, TJ = StepTile<Real>::TJ, DEPTH = 2;   // the sweep's look-ahead
    const TileBox tb = tile_box<TI, TJ>(d, g.tiles_i, g.tiles_j, g.kc, xcd_block(blockIdx.x, g.nblocks));
    const int tid = threadIdx.x + SW_TI * threadIdx.y;
    const int i = tb.i0 + tid % TI, j = tb.j0 + tid / TI;
    if (i >= d.ni || j >= d.nj) return;
    const int o0 = cell_off(d, i, j, 0), Z = d.sz;
    Real v[DEPTH][NF];
#pragma unroll
    for (int s = 0; s < DEPTH; ++s)
        if (tb.k0 + s < tb.k1)
#pragma unroll
            for (int f = 0; f < NF; ++f) v[s][f] = q.f[f][o0 + (tb.k0 + s) * Z];
    for (int k = tb.k0; k < tb.k1; k += DEPTH) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            if (k + s < tb.k1) {
                const int o = o0 + (k + s) * Z;
#pragma unroll
                for (int f = 0; f < NF; ++f) __builtin_nontemporal_store(v[s][f], &qn.f[f][o]);
                if (k + s + DEPTH < tb.k1)
#pragma unroll
                    for (int f = 0; f < NF; ++f) v[s][f] = q.f[f][o + DEPTH * Z];
            }
        }
    }
}

template <typename Real>
hipError_t launch_stream_copy(const Dims& d, const SweepGeom& g, CStateT<Real> q, StateT<Real> qn, hipStream_t s)
{
    dim3 block(SW_TI, StepTile<Real>::THREADS / SW_TI), grid(g.nblocks);
    stream_copy_kernel<Real><<<grid, block, 0, s>>>(d, g, q, qn);
    return hipGetLastError();
}
template hipError_t launch_stream_copy<double>(const Dims&, const SweepGeom&, CStateT<double>, StateT<double>,
                                               hipStream_t);
template hipError_t launch_stream_copy<float>(const Dims&, const SweepGeom&, CStateT<float>, StateT<float>,
                                              hipStream_t);

// The sweep's square root and reciprocal (stencil.h) on an array: out[2m] =
// sqrt_pos(x[m]), out[2m+1] = recip_pos(x[m]).
__global__ __launch_bounds__(256) void math_kernel(const double* __restrict__ x, double* __restrict__ out, int n)
{
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m >= n) return;
    out[2 * m] = sqrt_pos(x[m]);
    out[2 * m + 1] = recip_pos(x[m]);
}

hipError_t launch_math(const double* x, double* out, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    math_kernel<<<(n + 255) / 256, 256, 0, s>>>(x, out, n);
    return hipGetLastError();
}

SweepGeom sweep_geom(const Dims& d, int cus, int ti, int tj, int per_cu, bool streams_f64)
{
    SweepGeom g;
    g.tiles_i = (d.ni + ti - 1) / ti;
    g.tiles_j = (d.nj + tj - 1) / tj;
    const int tiles = g.tiles_i * g.tiles_j, slots = cus * per_cu;
    // Split the k columns into nkc chunks so that the launch finishes
    // earliest: blocks run in rounds of `slots` (the blocks resident at
    // once), a block costs its planes plus ~3 planes of start-up (the queue
    // and halo planes it loads before its first plane).  An FP64 sweep whose
    // two states exceed the 256 MB memory-side cache is bound by HBM, which
    // four fifths of the blocks keep busy: there the planes of all blocks count,
    // until the rounds at that rate take longer (192^3: 3 chunks 117 us, the 7
    // that minimise the rounds 123; 224^3 187 against 202).  Below that size
    // the rule does harm (136^3 54 against 44 us, 140x140x150 78 against 65),
    // and in FP32, with three blocks per CU (176^3 68 against 62 us, 224^3 121
    // against 109; 256^3 142 against 152).
    const int overhead = 3;
    const bool hbm = streams_f64 && 2.0 * NF * sizeof(double) * d.ni * d.nj * d.nk > 256e6;
    double best_cost = -1.0;
    int best = 1;
    const int max_nkc = max(1, d.nk / CAV_MIN_KC);
    for (int nkc = 1; nkc <= max_nkc; ++nkc) {
        const int kc = (d.nk + nkc - 1) / nkc;
        const long long blocks = (long long)tiles * ((d.nk + kc - 1) / kc);
        const long long rounds = (blocks + slots - 1) / slots;
        double cost = (double)rounds * (kc + overhead) * slots;
        if (hbm) cost = fmax(0.8 * cost, (double)blocks * (kc + overhead));
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = nkc;
        }
    }
    g.kc = (d.nk + best - 1) / best;
    g.nkc = (d.nk + g.kc - 1) / g.kc;
    g.nblocks = tiles * g.nkc;
    g.point = g.point_norm = g.stream = false;
    g.npart = g.nblocks;
    return g;
}

template <typename Real>
SweepGeom tile_geom(const Dims& d, int cus)
{
    // resident blocks per compute unit of the step kernel (registers and LDS
    // decide it); the same for every launch on this device
    static int per_cu = 0;
    if (per_cu == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sweep_kernel<Real, false, false, 0, true>,
                                                         StepTile<Real>::THREADS, 0) != hipSuccess ||
            n < 1)
            n = 1;
        per_cu = n;
    }
    SweepGeom g = sweep_geom(d, cus, StepTile<Real>::TI, StepTile<Real>::TJ, per_cu, sizeof(Real) == 8);
    g.stream = stream_out<Real>((double)d.ni * d.nj * d.nk);
    return g;
}
template SweepGeom tile_geom<double>(const Dims&, int);
template SweepGeom tile_geom<float>(const Dims&, int);

// The tile, or one cell per thread where that is faster.  FP32: while the L2s
// hold both states, 0.8 million cells (84x88x94 10.2 against 12.8 us; 99^3 15.4
// against 14.7, 33x180x150 18.6 against 16.4, 131x67x201 23.0 against 19.1).
// FP64: by both kernels' measured cost in us: the tile 4.9 + 1.55 a plane of
// its blocks (48^3 8.3, 72^3 14.6, 96^3 20.6, 130^3 41.6, 91x212x209 86), the
// other 4.5 + 20 per million cells (6.2, 12.7, 21.4), 30 for those past 1.5
// million, where its stars begin to miss the caches (130^3 51, 70x200x220 100
// against the tile's 76, 91x212x209 141); they cross twice, near 56^3, where
// the tile's chunks reach their shortest, and near 88^3, for rows just wider
// than a tile later (70x150x200 48 against 54).  (A grid of 4.2 million
// cells has at most 48 (FP64) or 96 (FP32) padded elements a cell, so that
// kernel's byte offsets fit in 32 bits.)  With norms only up to 150 thousand
// cells: each wavefront's five butterflies cost as much as its residual
// (161x97x130: 190 us against the tile's 125 for a step, its norms and the
// copy back).
template <typename Real>
SweepGeom step_geom(const Dims& d, int cus)
{
    SweepGeom g = tile_geom<Real>(d, cus);
    const long long n = (long long)d.ni * d.nj * d.nk;
    constexpr int CELLS = PointSweep<Real, true, false>::CELLS;
    const int rounds = (g.nblocks + cus - 1) / cus;
    const double cost = 4.5 + 20e-6 * (double)n + 10e-6 * fmax((double)n - 1.5e6, 0.0);
    g.point = sizeof(Real) == 4 ? n <= 800000 : n <= 4200000 && cost < 4.9 + 1.55 * rounds * g.kc;
    g.point_norm = g.point && n <= 150000;
    if (g.point_norm) g.npart = (int)((n + CELLS - 1) / CELLS);
    return g;
}
template SweepGeom step_geom<double>(const Dims&, int);
template SweepGeom step_geom<float>(const Dims&, int);

// g comes from step_geom<Real> or tile_geom<Real>.  xh, xbuf: the exchange of a split along i
// inside the sweep (NULL: none; never with one cell per thread); xpack: with
// the pack of the next step's exchange (never with norms).
template <typename Real>
hipError_t launch_sweep(const Dims& d, const Coef& c, const SweepGeom& g, CStateT<Real> q, StateT<Real> qn,
                        double* partials, bool with_norm, hipStream_t s, const HaloGeom* xh, Real* xbuf, bool xpack)
{
    if (with_norm ? g.point_norm : g.point) {
        const int n = d.ni * d.nj * d.nk;
        const bool small = sizeof(Real) == 8 && n <= 448 * 128;
#define POINT_LAUNCH(NRM, SM)                                                                              \
    do {                                                                                                   \
        using P = PointSweep<Real, NRM, SM>;                                                               \
        point_sweep_kernel<Real, NRM, SM><<<(n + P::CELLS - 1) / P::CELLS, P::THREADS, 0, s>>>(d, c, q, qn, partials); \
    } while (0)
        if (with_norm) POINT_LAUNCH(true, false);
        else if (small) POINT_LAUNCH(false, sizeof(Real) == 8);
        else POINT_LAUNCH(false, false);
#undef POINT_LAUNCH
        return hipGetLastError();
    }
    dim3 block(SW_TI, StepTile<Real>::THREADS / SW_TI), grid(g.nblocks);
    XGeom xg{};
    if (xh) {
        xg.ex = xh->e[0];
        xg.pi = xh->P[0];
        xg.nj = d.nj;
        xg.area = (int)xh->area[0];
        xg.wsum = xh->wsum;
        for (int f = 0; f < NF; ++f) {
            xg.w[f] = xh->w[f];
            xg.wpre[f] = xh->wpre[f];
        }
    }
    auto go = [&](auto field, auto stream) {
        constexpr bool F = decltype(field)::value, S = decltype(stream)::value;
        if (with_norm && xh) sweep_kernel<Real, true, F, 1, S><<<grid, block, 0, s>>>(d, c, g, q, qn, partials, xg, xbuf);
        else if (with_norm) sweep_kernel<Real, true, F, 0, S><<<grid, block, 0, s>>>(d, c, g, q, qn, partials, xg, xbuf);
        else if (xh && xpack) sweep_kernel<Real, false, F, 2, S><<<grid, block, 0, s>>>(d, c, g, q, qn, partials, xg, xbuf);
        else if (xh) sweep_kernel<Real, false, F, 1, S><<<grid, block, 0, s>>>(d, c, g, q, qn, partials, xg, xbuf);
        else sweep_kernel<Real, false, F, 0, S><<<grid, block, 0, s>>>(d, c, g, q, qn, partials, xg, xbuf);
    };
    auto pick = [&](auto stream) {
        if (c.t_hot_field) go(std::true_type{}, stream);
        else go(std::false_type{}, stream);
    };
    if (g.stream) pick(std::true_type{});
    else pick(std::false_type{});
    return hipGetLastError();
}
template hipError_t launch_sweep<double>(const Dims&, const Coef&, const SweepGeom&, CStateT<double>,
                                         StateT<double>, double*, bool, hipStream_t, const HaloGeom*, double*, bool);
template hipError_t launch_sweep<float>(const Dims&, const Coef&, const SweepGeom&, CStateT<float>,
                                        StateT<float>, double*, bool, hipStream_t, const HaloGeom*, float*, bool);

// ---------------------------------------------------------------------------
// Interior/exterior split (Sec. 4.7): with a halo exchange in the step, the
// cells whose stars reach no cell the unpack writes (the interior) are
// updated by one launch that may run while the exchange is in flight; the
// rest (the exterior: cells within `m` of a cut) by a second launch after
// it.  Each cell is computed by exactly one launch with the same per-cell
// code as the unsplit sweep, so the new state is bit-identical to it.

// Tile shape of the exterior x slabs (2m <= 8 owned columns).
constexpr int XS_TI = 16, XS_TJ = 32;

// Cell x along `axis` lies within m of a cut between two subdomains.
__device__ __forceinline__ bool near_cut(const SplitGeom& sg, int axis, int x)
{
    const int e = sg.e[axis];
    const int a = x / e, local = x - a * e;
    return (a > 0 && local < sg.m) || (a < sg.P[axis] - 1 && local >= e - sg.m);
}

struct OwnInterior {
    SplitGeom sg;
    __device__ __forceinline__ bool operator()(int i, int j, int k) const
    {
        return !(near_cut(sg, 0, i) || near_cut(sg, 1, j) || near_cut(sg, 2, k));
    }
    __device__ __forceinline__ bool column(int, int) const { return true; }
};

// The slab [cut - m, cut + m) along `axis`; cells also near a cut of a lower
// axis belong to that axis's slab.
struct OwnSlab {
    SplitGeom sg;
    int axis, cut;
    __device__ __forceinline__ bool operator()(int i, int j, int k) const
    {
        const int x = axis == 0 ? i : (axis == 1 ? j : k);
        if (x < cut - sg.m || x >= cut + sg.m) return false;
        if (axis >= 1 && near_cut(sg, 0, i)) return false;
        if (axis == 2 && near_cut(sg, 1, j)) return false;
        return true;
    }
    // an x slab's cells read columns up to 2 cells beyond it
    __device__ __forceinline__ bool column(int i, int) const
    {
        return axis != 0 || (i >= cut - sg.m - 2 && i < cut + sg.m + 2);
    }
};

// The interior launch runs the step sweep's tile of its type (g from
// tile_geom<Real>).
template <typename Real, bool NORM, bool FIELD, bool STREAM>
__global__ __launch_bounds__(StepTile<Real>::THREADS) void interior_kernel(Dims d, Coef cd, SweepGeom g, SplitGeom sg,
                                                                           CStateT<Real> q, StateT<Real> qn,
                                                                           double* partials, int)
{
    constexpr int TI = StepTile<Real>::TI, TJ = StepTile<Real>::TJ;
    __shared__ SweepLds<Real, TI, TJ> L;
    CoefR<Real> c = coef_as<Real>(cd);
    if constexpr (!FIELD) c.t_hot_field = nullptr;
    const TileBox tb = tile_box<TI, TJ>(d, g.tiles_i, g.tiles_j, g.kc, xcd_block(blockIdx.x, g.nblocks));
    StepEpi<Real, STREAM> epi{qn, Real(0)};
    sweep_tile<Real, NORM, OwnInterior, StepEpi<Real, STREAM>, TI, TJ>(d, c, tb, OwnInterior{sg}, q,
                                                                                     epi, partials, L);
}

// Exterior work items, block b: first the x slabs (per cut: 16 x 32 tiles,
// j tiles x k chunks of kce planes), then the y slabs (per cut: i tiles x k
// chunks), then the z slabs (per cut: i x j tiles, the 2m planes around the
// cut).
// Norm partials follow the interior launch's, at pidx = pidx0 + b (pidx0:
// the interior launch's block count).  g: the 64 x 8 tiling (sweep_geom).
template <typename Real, bool NORM, bool FIELD, bool STREAM>
__global__ __launch_bounds__(SW_TI * SW_TJ) void exterior_kernel(Dims d, Coef cd, SweepGeom g, SplitGeom sg,
                                                                 CStateT<Real> q, StateT<Real> qn,
                                                                 double* partials, int pidx0)
{
    __shared__ union {
        SweepLds<Real> yz;                       // 64 x 8 tiles for the y and z slabs
        SweepLds<Real, XS_TI, XS_TJ> x;          // 16 x 32 tiles for the x slabs
    } L;
    CoefR<Real> c = coef_as<Real>(cd);
    if constexpr (!FIELD) c.t_hot_field = nullptr;
    const int b = blockIdx.x;
    const int nkce = (d.nk + sg.kce - 1) / sg.kce;
    const int tjx = (d.nj + XS_TJ - 1) / XS_TJ;
    const int per0 = tjx * nkce, per1 = g.tiles_i * nkce, per2 = g.tiles_i * g.tiles_j;
    const int n0 = (sg.P[0] - 1) * per0, n1 = (sg.P[1] - 1) * per1;
    TileBox tb;
    int axis, cut;
    if (b < n0) {
        axis = 0;
        const int r = b % per0;
        cut = (b / per0 + 1) * sg.e[0];
        tb.i0 = cut - sg.m;
        tb.j0 = (r % tjx) * XS_TJ;
        tb.k0 = (r / tjx) * sg.kce;
        tb.k1 = min(tb.k0 + sg.kce, d.nk);
    } else if (b < n0 + n1) {
        axis = 1;
        const int r = (b - n0) % per1;
        cut = ((b - n0) / per1 + 1) * sg.e[1];
        tb.i0 = (r % g.tiles_i) * SW_TI;
        tb.j0 = cut - sg.m;
        tb.k0 = (r / g.tiles_i) * sg.kce;
        tb.k1 = min(tb.k0 + sg.kce, d.nk);
    } else {
        axis = 2;
        const int r = (b - n0 - n1) % per2;
        cut = ((b - n0 - n1) / per2 + 1) * sg.e[2];
        tb.i0 = (r % g.tiles_i) * SW_TI;
        tb.j0 = (r / g.tiles_i) * SW_TJ;
        tb.k0 = cut - sg.m;
        tb.k1 = cut + sg.m;
    }
    tb.pidx = pidx0 + b;
    StepEpi<Real, STREAM> epi{qn, Real(0)};
    if (axis == 0)          // 2m <= 8 owned columns: a narrow tile wastes fewer lanes
        sweep_tile<Real, NORM, OwnSlab, StepEpi<Real, STREAM>, XS_TI, XS_TJ>(d, c, tb, OwnSlab{sg, axis, cut}, q, epi,
                                                                      partials, L.x);
    else
        sweep_tile<Real, NORM>(d, c, tb, OwnSlab{sg, axis, cut}, q, epi, partials, L.yz);
}

int exterior_blocks(const Dims& d, const SweepGeom& g, const SplitGeom& sg)
{
    const int nkce = (d.nk + sg.kce - 1) / sg.kce;
    return (sg.P[0] - 1) * ((d.nj + XS_TJ - 1) / XS_TJ) * nkce + (sg.P[1] - 1) * g.tiles_i * nkce +
           (sg.P[2] - 1) * g.tiles_i * g.tiles_j;
}

// gi: the interior launch's geometry (tile_geom<Real>); g: the 64 x 8 tiling
// the exterior slabs are decoded from (sweep_geom).
template <typename Real>
hipError_t launch_split(const Dims& d, const Coef& c, const SweepGeom& gi, const SweepGeom& g, const SplitGeom& sg,
                        bool exterior, CStateT<Real> q, StateT<Real> qn, double* partials, bool with_norm,
                        hipStream_t s)
{
    const dim3 block = exterior ? dim3(SW_TI, SW_TJ) : dim3(SW_TI, StepTile<Real>::THREADS / SW_TI);
    const SweepGeom& gl = exterior ? g : gi;
    const int nb = exterior ? exterior_blocks(d, g, sg) : gi.nblocks;
    const int pidx0 = gi.nblocks;
    if (nb == 0) return hipSuccess;
    const bool fld = c.t_hot_field != nullptr;
#define SPLIT_LAUNCH(K, S)                                                                                    \
    do {                                                                                                      \
        if (fld) {                                                                                            \
            if (with_norm) K<Real, true, true, S><<<nb, block, 0, s>>>(d, c, gl, sg, q, qn, partials, pidx0);  \
            else K<Real, false, true, S><<<nb, block, 0, s>>>(d, c, gl, sg, q, qn, partials, pidx0);           \
        } else {                                                                                              \
            if (with_norm) K<Real, true, false, S><<<nb, block, 0, s>>>(d, c, gl, sg, q, qn, partials, pidx0); \
            else K<Real, false, false, S><<<nb, block, 0, s>>>(d, c, gl, sg, q, qn, partials, pidx0);          \
        }                                                                                                     \
    } while (0)
    if (exterior) {
        if (gl.stream) SPLIT_LAUNCH(exterior_kernel, true);
        else SPLIT_LAUNCH(exterior_kernel, false);
    } else {
        if (gl.stream) SPLIT_LAUNCH(interior_kernel, true);
        else SPLIT_LAUNCH(interior_kernel, false);
    }
#undef SPLIT_LAUNCH
    return hipGetLastError();
}
template hipError_t launch_split<double>(const Dims&, const Coef&, const SweepGeom&, const SweepGeom&,
                                         const SplitGeom&, bool, CStateT<double>, StateT<double>, double*, bool,
                                         hipStream_t);
template hipError_t launch_split<float>(const Dims&, const Coef&, const SweepGeom&, const SweepGeom&,
                                        const SplitGeom&, bool, CStateT<float>, StateT<float>, double*, bool,
                                        hipStream_t);

// ---------------------------------------------------------------------------
// Batched form: a persistent grid walks the work list of all members; each
// item is one tile column's k chunk of one member, computed by the same
// sweep_tile as the single-cavity sweep.  `parity` selects which of q and
// q_tmp holds the current state of every member.
template <typename Real>
struct BatchTiles {
    static constexpr bool F32 = sizeof(Real) == 4;
    static constexpr int THREADS = batch_threads(F32);
    static constexpr int WTI = batch_wide_ti(F32), WTJ = batch_tj(F32, WTI);
    static constexpr int NTI = batch_narrow_ti(F32), NTJ = batch_tj(F32, NTI);
    // waves per SIMD the one-shape FP32 kernels must fit (three 256-thread
    // blocks per CU, as the FP32 step sweep; 0: the compiler's choice)
    static constexpr int MINW1 = F32 ? 3 : 0;
};

// The item walk of one block: with at least BATCH_SEGS blocks, block b
// (on XCD b % 8) takes every (blocks on its XCD)-th item of segment b % 8;
// with fewer blocks, block b walks whole segments b, b + gridDim.x, ...
template <typename F>
__device__ __forceinline__ void for_each_item(const int* __restrict__ segs, F&& body)
{
    const int G = gridDim.x, b = blockIdx.x;
    if (G >= BATCH_SEGS) {
        const int s = b % BATCH_SEGS, lb = b / BATCH_SEGS;
        const int nbs = (G - s + BATCH_SEGS - 1) / BATCH_SEGS;      // blocks on segment s
        for (int it = segs[s] + lb; it < segs[s + 1]; it += nbs) body(it);
    } else {
        for (int s = b; s < BATCH_SEGS; s += G)
            for (int it = segs[s]; it < segs[s + 1]; ++it) body(it);
    }
}

// SHAPES: 3 = each member's tile shape (both compiled in; FP32: 164 registers
// and three blocks per CU, with norms 175 and two), 1 = the wide shape only, 2
// = the narrow one only (FP32: 141 registers, with norms 168, three blocks).
template <typename Real, bool NORM, int SHAPES, bool STREAM>
__global__ __launch_bounds__(BatchTiles<Real>::THREADS, SHAPES == 3 ? 0 : BatchTiles<Real>::MINW1) void batch_kernel(
    const BatchCav* __restrict__ cavs, const int* __restrict__ segs, const BatchItem* __restrict__ items, int parity)
{
    using BT = BatchTiles<Real>;
    using Wide = SweepLds<Real, BT::WTI, BT::WTJ>;
    using Narrow = SweepLds<Real, BT::NTI, BT::NTJ>;
    __shared__ union {
        Wide wide;
        Narrow narrow;
    } L;
    for_each_item(segs, [&](int it) {
        const BatchItem w = items[it];
        const BatchCav& cv = cavs[w.cav];
        const Dims d = cv.d;
        const CoefR<Real> c = coef_as<Real>(cv.c);
        const Real* cur = static_cast<const Real*>(parity ? cv.q_tmp : cv.q);
        Real* nxt = static_cast<Real*>(parity ? cv.q : cv.q_tmp);
        CStateT<Real> qs;
        StateT<Real> qn;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            qs.f[f] = cur + f * cv.fstride;
            qn.f[f] = nxt + f * cv.fstride;
        }
        StepEpi<Real, STREAM> epi{qn, Real(0)};
        if (SHAPES == 2 || (SHAPES == 3 && cv.ti == BT::NTI)) {
            const TileBox tb = tile_box<BT::NTI, BT::NTJ>(d, cv.tiles_i, cv.tiles_j, cv.kc, w.tile);
            sweep_tile<Real, NORM, OwnAll, StepEpi<Real, STREAM>, BT::NTI, BT::NTJ>(
                d, c, tb, OwnAll{}, qs, epi, cv.ws + WS_HEAD_DOUBLES, L.narrow);
        } else {
            const TileBox tb = tile_box<BT::WTI, BT::WTJ>(d, cv.tiles_i, cv.tiles_j, cv.kc, w.tile);
            sweep_tile<Real, NORM, OwnAll, StepEpi<Real, STREAM>, BT::WTI, BT::WTJ>(
                d, c, tb, OwnAll{}, qs, epi, cv.ws + WS_HEAD_DOUBLES, L.wide);
        }
        __syncthreads();                  // LDS is reused by the next item
    });
}

template <typename Real>
hipError_t launch_batch(const BatchCav* cavs, const int* segs, const BatchItem* items, int parity, bool with_norm,
                        int nblocks, int shapes, bool stream, hipStream_t s)
{
    dim3 block(SW_TI, BatchTiles<Real>::THREADS / SW_TI), grid(nblocks);
#define BATCH_LAUNCH(SH)                                                                                \
    do {                                                                                                \
        if (with_norm && stream) batch_kernel<Real, true, SH, true><<<grid, block, 0, s>>>(cavs, segs, items, parity);  \
        else if (with_norm) batch_kernel<Real, true, SH, false><<<grid, block, 0, s>>>(cavs, segs, items, parity);      \
        else if (stream) batch_kernel<Real, false, SH, true><<<grid, block, 0, s>>>(cavs, segs, items, parity);         \
        else batch_kernel<Real, false, SH, false><<<grid, block, 0, s>>>(cavs, segs, items, parity);                    \
    } while (0)
    if (shapes == 1) BATCH_LAUNCH(1);
    else if (shapes == 2) BATCH_LAUNCH(2);
    else BATCH_LAUNCH(3);
#undef BATCH_LAUNCH
    return hipGetLastError();
}
template hipError_t launch_batch<double>(const BatchCav*, const int*, const BatchItem*, int, bool, int, int,
                                         bool, hipStream_t);
template hipError_t launch_batch<float>(const BatchCav*, const int*, const BatchItem*, int, bool, int, int,
                                        bool, hipStream_t);

// The batch's step with one cell per thread (as for a small grid, and bound
// alike): every block is POINT_CELLS cells of one member, so no lanes idle at
// ragged extents and no unit waits for a column to end.  A block finds its
// member among the first blocks of all of them, 64 at a time (one load's
// latency up to 64 members; a list of items would be one more).  8 FP64
// members of 0.75 M cells together: 48 -> 25 us a step.
template <typename Real>
__global__ __launch_bounds__((PointSweep<Real, false, false>::THREADS)) void batch_point_kernel(
    const BatchCav* __restrict__ cavs, int members, int parity)
{
    const int blk = xcd_block(blockIdx.x, gridDim.x), lane = threadIdx.x & 63;
    int lo = 0;
    for (int span = members; span > 1;) {
        const int step = (span + 63) >> 6, m = lo + lane * step;
        const bool at_or_before = lane * step < span && cavs[min(m, members - 1)].pstart <= blk;
        const int at = (__popcll(__ballot(at_or_before)) - 1) * step;
        lo += at;
        span = min(step, span - at);
    }
    const BatchCav& cv = cavs[__builtin_amdgcn_readfirstlane(lo)];
    const Dims d = cv.d;
    const Real* cur = static_cast<const Real*>(parity ? cv.q_tmp : cv.q);
    Real* nxt = static_cast<Real*>(parity ? cv.q : cv.q_tmp);
    CStateT<Real> qs;
    StateT<Real> qn;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        qs.f[f] = cur + f * cv.fstride;
        qn.f[f] = nxt + f * cv.fstride;
    }
    point_sweep<Real, false, false>(d, coef_as<Real>(cv.c), qs, qn, blk - cv.pstart, nullptr);
}

template <typename Real>
hipError_t launch_batch_points(const BatchCav* cavs, int members, int points, int parity, hipStream_t s)
{
    static_assert(PointSweep<Real, false, false>::CELLS == POINT_CELLS, "the table's blocks are the kernel's");
    batch_point_kernel<Real><<<points, PointSweep<Real, false, false>::THREADS, 0, s>>>(cavs, members, parity);
    return hipGetLastError();
}
template hipError_t launch_batch_points<double>(const BatchCav*, int, int, int, hipStream_t);
template hipError_t launch_batch_points<float>(const BatchCav*, int, int, int, hipStream_t);

// Residual norms from per-block partials: fixed-order sums (each thread its
// strided blocks in order, all fields of a block at once so that its loads
// are independent; a butterfly within the wavefront; the wavefronts in
// order), RMS over ncell.  Run by one block of T threads.  One field after the
// other, with one load in flight per thread, 4000 partials took ~90 us.
template <int T>
__device__ __forceinline__ void finalize_norms(const double* __restrict__ part, int nb, double ncell,
                                               double* __restrict__ out)
{
    __shared__ double red[T / 64][NF];
    const int t = threadIdx.x;
    double s[NF] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int b = t; b < nb; b += T)
#pragma unroll
        for (int f = 0; f < NF; ++f) s[f] += part[(size_t)b * NF + f];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) s[f] += __shfl_xor(s[f], m, 64);
        if ((t & 63) == 0) red[t >> 6][f] = s[f];
    }
    __syncthreads();
    if (t < NF) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < T / 64; ++w) v += red[w][t];
        out[t] = sqrt(v / ncell);
    }
}

// Residual norms of every member of a batch: one block per member.
__global__ __launch_bounds__(256) void batch_norm_kernel(const BatchCav* __restrict__ cavs)
{
    const BatchCav& cv = cavs[blockIdx.x];
    finalize_norms<256>(cv.ws + WS_HEAD_DOUBLES, cv.ntiles, (double)cv.d.ni * cv.d.nj * cv.d.nk, cv.ws);
}

hipError_t launch_batch_norms(const BatchCav* cavs, int members, hipStream_t s)
{
    batch_norm_kernel<<<members, 256, 0, s>>>(cavs);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Wall ghost layers (Sec. 2), written into the state by cavity_init: one
// thread per wall-adjacent line of cells, all five fields, both layers.
template <typename Real>
__global__ __launch_bounds__(256) void bc_kernel(Dims d, Bcs bc, StateT<Real> q)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long nx = 2LL * d.nj * d.nk, ny = 2LL * d.ni * d.nk, nz = 2LL * d.ni * d.nj;
    int o, s, axis;
    bool high;
    double tw_lo = bc.t_hot;
    if (t < nx) {                                   // x walls: (j, k, side), j fastest
        axis = 0;
        const int j = (int)(t % d.nj);
        const long long r = t / d.nj;
        const int k = (int)(r % d.nk);
        high = r >= d.nk;
        if (bc.t_hot_field) tw_lo = bc.t_hot_field[j + (long long)d.nj * k];
        o = cell_off(d, high ? d.ni - 1 : 0, j, k);
        s = high ? -1 : 1;
    } else if (t < nx + ny) {                       // y walls: (i, k, side), i fastest
        axis = 1;
        const long long u = t - nx;
        const int i = (int)(u % d.ni);
        const long long r = u / d.ni;
        const int k = (int)(r % d.nk);
        high = r >= d.nk;
        o = cell_off(d, i, high ? d.nj - 1 : 0, k);
        s = high ? -d.sy : d.sy;
    } else if (t < nx + ny + nz) {                  // z walls: (i, j, side), i fastest
        axis = 2;
        const long long u = t - nx - ny;
        const int i = (int)(u % d.ni);
        const long long r = u / d.ni;
        const int j = (int)(r % d.nj);
        high = r >= d.nj;
        o = cell_off(d, i, j, high ? d.nk - 1 : 0);
        s = high ? -d.sz : d.sz;
    } else {
        return;
    }
    // p: one-sided linear extrapolation, second order
    {
        Real* A = q.f[FP];
        const Real a = A[o], b = A[o + s];
        const Real g1 = Real(2) * a - b;
        A[o - s] = g1;
        A[o - 2 * s] = Real(2) * g1 - a;
    }
    // u, v, w: no-slip (odd reflection)
#pragma unroll
    for (int f = FU; f <= FW; ++f) {
        Real* A = q.f[f];
        const Real a = A[o], b = A[o + s];
        A[o - s] = -a;
        A[o - 2 * s] = -b;
    }
    // T: fixed value on the hot/cold walls, zero gradient elsewhere
    {
        Real* A = q.f[FT];
        const Real a = A[o], b = A[o + s];
        if (axis == 0) {
            const Real tw = (Real)(high ? bc.t_cold : tw_lo);
            A[o - s] = Real(2) * tw - a;
            A[o - 2 * s] = Real(2) * tw - b;
        } else {
            A[o - s] = a;
            A[o - 2 * s] = b;
        }
    }
}

template <typename Real>
hipError_t launch_bc(const Dims& d, const Bcs& b, StateT<Real> q, hipStream_t s)
{
    const long long n = 2LL * ((long long)d.nj * d.nk + (long long)d.ni * d.nk + (long long)d.ni * d.nj);
    bc_kernel<Real><<<(unsigned)((n + 255) / 256), 256, 0, s>>>(d, b, q);
    return hipGetLastError();
}
template hipError_t launch_bc<double>(const Dims&, const Bcs&, StateT<double>, hipStream_t);
template hipError_t launch_bc<float>(const Dims&, const Bcs&, StateT<float>, hipStream_t);

// ---------------------------------------------------------------------------
// Seeded initial state: SplitMix64 (Steele, Lea & Flood 2014), output number
// f*2^40 + idx of the stream seeded with `seed`.  Computed in FP64; an FP32
// state stores the rounded values.
__device__ __forceinline__ double noise(uint64_t seed, int f, uint64_t idx, double amp)
{
    uint64_t z = seed + ((((uint64_t)f) << 40) + idx + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z = z ^ (z >> 31);
    const double r = (double)(z >> 11) * 0x1.0p-53;
    return (2.0 * r - 1.0) * amp;
}

template <typename Real>
__global__ __launch_bounds__(256) void init_kernel(Dims d, double t_hot, double t_cold, uint64_t seed,
                                                   double amp, StateT<Real> q)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long long)d.ni * d.nj * d.nk) return;
    const int i = (int)(idx % d.ni);
    const long long r = idx / d.ni;
    const int j = (int)(r % d.nj);
    const int k = (int)(r / d.nj);
    const int o = cell_off(d, i, j, k);
    const double xc = ((double)i + 0.5) / (double)d.ni;
    q.f[FP][o] = (Real)0.0;
    q.f[FU][o] = (Real)noise(seed, 1, (uint64_t)idx, amp);
    q.f[FV][o] = (Real)noise(seed, 2, (uint64_t)idx, amp);
    q.f[FW][o] = (Real)noise(seed, 3, (uint64_t)idx, amp);
    q.f[FT][o] = (Real)((t_hot + (t_cold - t_hot) * xc) + noise(seed, 4, (uint64_t)idx, amp));
}

template <typename Real>
hipError_t launch_init(const Dims& d, double t_hot, double t_cold, uint64_t seed, double amp, StateT<Real> q,
                       hipStream_t s)
{
    const long long n = (long long)d.ni * d.nj * d.nk;
    init_kernel<Real><<<(unsigned)((n + 255) / 256), 256, 0, s>>>(d, t_hot, t_cold, seed, amp, q);
    return hipGetLastError();
}
template hipError_t launch_init<double>(const Dims&, double, double, uint64_t, double, StateT<double>, hipStream_t);
template hipError_t launch_init<float>(const Dims&, double, double, uint64_t, double, StateT<float>, hipStream_t);

// ---------------------------------------------------------------------------
// Mean Nusselt number of the hot wall x = 0 in FP64: -dT/dx at the wall from
// the second-order one-sided difference (9 T_0 - T_1 - 8 T_w) / (3h) through
// the wall value and the first two cell centres, averaged over the wall and
// divided by t_hot - t_cold.  The wall value is the hot-wall field where one
// is given.  One block; fixed-order reduction.
template <typename Real>
__global__ __launch_bounds__(1024) void nusselt_kernel(Dims d, Bcs bc, CStateT<Real> q, double* out)
{
    __shared__ double red[1024];
    const int t = threadIdx.x;
    const long long n = (long long)d.nj * d.nk;
    const double three_h = 3.0 / (double)d.ni;
    double acc = 0.0;
    for (long long e = t; e < n; e += 1024) {
        const int j = (int)(e % d.nj), k = (int)(e / d.nj);
        const int o = cell_off(d, 0, j, k);
        const double t0 = (double)q.f[FT][o], t1 = (double)q.f[FT][o + 1];
        const double tw = bc.t_hot_field ? bc.t_hot_field[e] : bc.t_hot;
        acc += -((9.0 * t0 - t1 - 8.0 * tw) / three_h);
    }
    red[t] = acc;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    if (t == 0) out[0] = red[0] / ((double)d.nj * (double)d.nk) / (bc.t_hot - bc.t_cold);
}

template <typename Real>
hipError_t launch_nusselt(const Dims& d, const Bcs& b, CStateT<Real> q, double* out, hipStream_t s)
{
    nusselt_kernel<Real><<<1, 1024, 0, s>>>(d, b, q, out);
    return hipGetLastError();
}
template hipError_t launch_nusselt<double>(const Dims&, const Bcs&, CStateT<double>, double*, hipStream_t);
template hipError_t launch_nusselt<float>(const Dims&, const Bcs&, CStateT<float>, double*, hipStream_t);

// ---------------------------------------------------------------------------
// Residual norms of one cavity.
__global__ __launch_bounds__(1024) void norm_finalize_kernel(const double* part, int nb, double ncell, double* out)
{
    finalize_norms<1024>(part, nb, ncell, out);
}

hipError_t launch_norm_finalize(const double* partials, int nblocks, double ncell, double* out,
                                hipStream_t s)
{
    norm_finalize_kernel<<<1, 1024, 0, s>>>(partials, nblocks, ncell, out);
    return hipGetLastError();
}

// The end of an odd number of steps: the interior cells of src copied to dst,
// VE elements (16 bytes, or one element of an unaligned state) a lane, row by
// row in whole 128-byte lines (a row's last one takes ghost and padding cells
// along: part of a line costs more to write; 170^3 FP32 95 -> 90 us for one
// step).  Bound by memory: COPY_CHUNKS chunks of a plane a block, four in
// flight a lane.  With norms (out not NULL) the first block finalizes them
// meanwhile, in norm_finalize_kernel's order.  STREAM: as the sweep's stores;
// the loads too, which otherwise leave src cached for the next step to write
// (161x97x130: 76 -> 67 us).  One step with its norms, by a copy of the whole
// array after the norms against this: FP64 64^3 24.5 -> 20, 128^3 74 -> 59,
// 256^3 554 -> 473; FP32 64^3 19.7 -> 14.7, 256^3 325 -> 270.
// A launch has to stay below 2^32 threads, which one block per plane and field
// passes on deep thin grids (2 x 2 x 838861): past COPY_MAX_BLOCKS a block
// takes every so many-th piece.
constexpr int COPY_THREADS = 1024, COPY_UNROLL = 4, COPY_CHUNKS = COPY_THREADS * COPY_UNROLL;
constexpr int COPY_MAX_BLOCKS = 1 << 21;

template <typename Real, bool STREAM, int VE>
__global__ __launch_bounds__(COPY_THREADS) void copy_back_kernel(Dims d, long long fs, int bpp, const Real* __restrict__ src,
                                                                 Real* __restrict__ dst, const double* part, int nb,
                                                                 double ncell, double* out)
{
    typedef Real Vec __attribute__((ext_vector_type(VE)));
    const int first = out ? 1 : 0;
    if (out && blockIdx.x == 0) {
        finalize_norms<COPY_THREADS>(part, nb, ncell, out);
        return;
    }
    constexpr int LINE = ROW_ALIGN_BYTES / sizeof(Real);
    const int cpr = (d.ni + LINE - 1) / LINE * (LINE / VE), n = d.nj * cpr;
    const int pieces = NF * d.nk * bpp;
    for (int blk = blockIdx.x - first; blk < pieces; blk += gridDim.x - first) {
        const int plane = blk / bpp, seg = blk - plane * bpp;
        const int f = plane / d.nk, k = plane - f * d.nk;
        const long long base = f * fs + cell_off(d, 0, 0, k);
        const int t0 = seg * COPY_CHUNKS + threadIdx.x;
        Vec v[COPY_UNROLL];
        int o[COPY_UNROLL];
#pragma unroll
        for (int r = 0; r < COPY_UNROLL; ++r) {
            const int t = min(t0 + r * COPY_THREADS, n - 1), row = t / cpr;
            o[r] = row * d.sy + (t - row * cpr) * VE;
            const Vec* a = reinterpret_cast<const Vec*>(src + base + o[r]);
            v[r] = STREAM ? __builtin_nontemporal_load(a) : *a;
        }
#pragma unroll
        for (int r = 0; r < COPY_UNROLL; ++r) {
            if (t0 + r * COPY_THREADS >= n) break;
            if (STREAM) __builtin_nontemporal_store(v[r], reinterpret_cast<Vec*>(dst + base + o[r]));
            else *reinterpret_cast<Vec*>(dst + base + o[r]) = v[r];
        }
    }
}

template <typename Real>
hipError_t launch_copy_back(const Dims& d, long long fs, const Real* src, Real* dst, bool stream, const double* partials,
                            int nblocks, double ncell, double* out, hipStream_t s)
{
    auto go = [&](auto str, auto width) {
        constexpr int VE = decltype(width)::value;
        constexpr int LINE = ROW_ALIGN_BYTES / sizeof(Real);
        const int bpp = (d.nj * ((d.ni + LINE - 1) / LINE * (LINE / VE)) + COPY_CHUNKS - 1) / COPY_CHUNKS;
        const int grid = min(NF * d.nk * bpp, COPY_MAX_BLOCKS) + (out ? 1 : 0);
        copy_back_kernel<Real, decltype(str)::value, VE>
            <<<grid, COPY_THREADS, 0, s>>>(d, fs, bpp, src, dst, partials, nblocks, ncell, out);
    };
    // rows are at multiples of 128 bytes of the state, which the caller may
    // have aligned to one element only
    const bool wide = (reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % 16 == 0;
    auto pick = [&](auto str) {
        if (wide) go(str, std::integral_constant<int, 16 / sizeof(Real)>{});
        else go(str, std::integral_constant<int, 1>{});
    };
    if (stream) pick(std::true_type{});
    else pick(std::false_type{});
    return hipGetLastError();
}
template hipError_t launch_copy_back<double>(const Dims&, long long, const double*, double*, bool, const double*, int,
                                             double, double*, hipStream_t);
template hipError_t launch_copy_back<float>(const Dims&, long long, const float*, float*, bool, const double*, int,
                                            double, double*, hipStream_t);

}  // namespace cav
