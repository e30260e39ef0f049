// In-device halo pack / unpack for gfx950 (Xue & Roy, arXiv:2006.02602,
// Sec. 4.5: "Optimized V1" packs the noncontiguous i faces into a contiguous
// buffer in parallel on the device, "V2" sends each field with its own
// stencil width, "V3" extends the buffers to the j and k faces).
//
// One launch covers every cut face of the virtual split and nothing else:
// the grid is three ranges of blocks, one per axis, each (cut faces normal
// to that axis) x (blocks per face, sized to that axis' face area).  A
// thread moves HALO_ROWS tangential cells of one face, 256 cells apart, with
// all fields and layers of each: every load of the thread is in flight
// before its first store.  On j and k faces the lanes run along i, so loads
// and stores are coalesced rows.  On i faces a lane's layers are adjacent
// in memory (one 16-byte access for two FP64 layers when aligned) and
// consecutive lanes take consecutive rows, whose buffer entries are
// adjacent: the buffer side is coalesced, the state side moves one short
// run per row.  The buffer layout is in halo_layout.h.
//
// Where a pack is followed by its unpack with nothing between (the exchange
// inside a step: all virtual subdomains live in one array), one launch does
// both: the unpack stores, into the receiver's box, the values the pack has
// just stored into the buffer, from the same registers.
#include "cavity_internal.h"
#include "halo_layout.h"

#include <type_traits>

namespace cav {

template <typename Real>
struct Pair;
template <>
struct Pair<double> {
    using T = double2;
};
template <>
struct Pair<float> {
    using T = float2;
};

// Face `fidx` of the cut faces normal to `axis`: cut m (between subdomain
// coordinates m and m+1 along the axis), transverse subdomain pair tr, and
// side 0 = the +axis face of the lower subdomain, 1 = the -axis face of the
// upper one.
__device__ __forceinline__ void face_of(const HaloGeom& h, int axis, int fidx, int& a, int& b, int& c, int& face)
{
    const int side = fidx & 1, pair = fidx >> 1;
    const int cut = pair % (h.P[axis] - 1), tr = pair / (h.P[axis] - 1);
    const int m = cut + side;
    face = 2 * axis + (side ? 0 : 1);
    if (axis == 0) { a = m; b = tr % h.P[1]; c = tr / h.P[1]; }
    else if (axis == 1) { a = tr % h.P[0]; b = m; c = tr / h.P[0]; }
    else { a = tr % h.P[0]; b = tr / h.P[0]; c = m; }
}

template <typename Real, HaloMode MODE>
__global__ __launch_bounds__(HALO_THREADS) void halo_kernel(Dims d, HaloGeom h, StateT<Real> q, Real* buf)
{
    using R2 = typename Pair<Real>::T;
    int blk = blockIdx.x;
    const int axis = blk < h.blk_end[0] ? 0 : (blk < h.blk_end[1] ? 1 : 2);
    if (axis > 0) blk -= h.blk_end[axis - 1];
    const int fidx = blk / h.bpf[axis], fblk = blk - fidx * h.bpf[axis];
    int a, b, c, face;
    face_of(h, axis, fidx, a, b, c, face);
    const bool high = face & 1;
    const int area = (int)h.area[axis];

    // offset (in tangential cells) of this face's segment
    const long long u = face_offset(h, a, b, c, face);
    Real* __restrict__ B = buf + u * h.wsum;

    const int ex = h.e[0], ey = h.e[1], ez = h.e[2];
    // per field: state offset of the face's first layer at tangential cell
    // 0, and the buffer offset of its box
    int qbase[NF];
    long long bbase[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int w = h.w[f];
        bbase[f] = (long long)h.wpre[f] * area;
        if (axis == 0) qbase[f] = cell_off(d, high ? (a + 1) * ex - w : a * ex, b * ey, c * ez);
        else if (axis == 1) qbase[f] = cell_off(d, a * ex, high ? (b + 1) * ey - w : b * ey, c * ez);
        else qbase[f] = cell_off(d, a * ex, b * ey, high ? (c + 1) * ez - w : c * ez);
    }
    // this thread's tangential cells: (ta, tb) = (j, k) on i faces, (i, k)
    // on j faces, (i, j) on k faces, and their state offsets from qbase
    const int t0 = fblk * (HALO_THREADS * HALO_ROWS) + threadIdx.x;
    const int ne = axis == 0 ? ey : ex;
    int ta[HALO_ROWS], tb[HALO_ROWS], qo[HALO_ROWS];
    bool ok[HALO_ROWS];
#pragma unroll
    for (int r = 0; r < HALO_ROWS; ++r) {
        const int t = t0 + r * HALO_THREADS;
        ok[r] = t < area;
        ta[r] = t % ne;
        tb[r] = t / ne;
        qo[r] = axis == 0 ? tb[r] * d.sz + ta[r] * d.sy : (axis == 1 ? tb[r] * d.sz + ta[r] : tb[r] * d.sy + ta[r]);
    }
    // stride between layers in the state
    const int lay_q = axis == 0 ? 1 : (axis == 1 ? d.sy : d.sz);

    // buffer element of (tangential cell r, layer l) of field f: the box in
    // (k, j, i) order, i fastest
    auto bidx = [&](int f, int r, int l) -> long long {
        const int w = h.w[f];
        if (axis == 0) return bbase[f] + ((long long)tb[r] * ey + ta[r]) * w + l;
        if (axis == 1) return bbase[f] + ((long long)tb[r] * w + l) * ex + ta[r];
        return bbase[f] + (long long)l * area + (long long)tb[r] * ex + ta[r];
    };
    // two layers of an i face move as one pair where the address allows
    auto paired = [&](const Real* p) { return axis == 0 && (reinterpret_cast<uintptr_t>(p) % sizeof(R2)) == 0; };

    Real v[HALO_ROWS][NF][2];
    auto get_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < HALO_ROWS; ++r) {
            if (!ok[r]) continue;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const Real* __restrict__ Q = q.f[f] + qbase[f] + qo[r];
                const int w = h.w[f];
                if (w == 2 && paired(Q)) {
                    const R2 x = *reinterpret_cast<const R2*>(Q);
                    v[r][f][0] = x.x;
                    v[r][f][1] = x.y;
                } else {
                    if (w > 0) v[r][f][0] = Q[0];
                    if (w > 1) v[r][f][1] = Q[lay_q];
                }
            }
        }
    };
    auto get_buffer = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < HALO_ROWS; ++r) {
            if (!ok[r]) continue;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int w = h.w[f];
                const long long o = bidx(f, r, 0);
                if (w == 2 && paired(B + o)) {
                    const R2 x = *reinterpret_cast<const R2*>(B + o);
                    v[r][f][0] = x.x;
                    v[r][f][1] = x.y;
                } else {
                    if (w > 0) v[r][f][0] = B[o];
                    if (w > 1) v[r][f][1] = B[bidx(f, r, 1)];
                }
            }
        }
    };
    auto put_buffer = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < HALO_ROWS; ++r) {
            if (!ok[r]) continue;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int w = h.w[f];
                const long long o = bidx(f, r, 0);
                if (w == 2 && paired(B + o)) {
                    R2 x;
                    x.x = v[r][f][0];
                    x.y = v[r][f][1];
                    *reinterpret_cast<R2*>(B + o) = x;
                } else {
                    if (w > 0) B[o] = v[r][f][0];
                    if (w > 1) B[bidx(f, r, 1)] = v[r][f][1];
                }
            }
        }
    };
    auto put_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < HALO_ROWS; ++r) {
            if (!ok[r]) continue;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                Real* __restrict__ Q = q.f[f] + qbase[f] + qo[r];
                const int w = h.w[f];
                if (w == 2 && paired(Q)) {
                    R2 x;
                    x.x = v[r][f][0];
                    x.y = v[r][f][1];
                    *reinterpret_cast<R2*>(Q) = x;
                } else {
                    if (w > 0) Q[0] = v[r][f][0];
                    if (w > 1) Q[lay_q] = v[r][f][1];
                }
            }
        }
    };
    if (MODE == HALO_UNPACK) get_buffer();
    else get_state();
    if (MODE != HALO_UNPACK) put_buffer();
    if (MODE != HALO_PACK) put_state();
}

// The same with one field a thread, for small exchanges: those are bound by a
// launch's start, of which the code fetched before the first load is a large
// part, and by the few loads in flight (pack, us: 16^3 2x2x2 4.2 -> 3.3, 64^3
// 6.7 -> 4.0, 96^3 6.9 -> 5.3; the exchange of a 16^3 step 6.2 -> 4.0).
template <typename Real, HaloMode MODE>
__global__ __launch_bounds__(HALO_THREADS) void halo_field_kernel(Dims d, HaloGeom h, long long fs,
                                                                  Real* __restrict__ q,
                                                                  Real* __restrict__ buf)
{
    using R2 = typename Pair<Real>::T;
    // blocks of one axis: faces, then fields, then the face's cells
    int blk = blockIdx.x;
    const int axis = blk < h.blk_end[0] * NF ? 0 : (blk < h.blk_end[1] * NF ? 1 : 2);
    if (axis > 0) blk -= h.blk_end[axis - 1] * NF;
    const int r1 = blk >> 1, r2 = r1 / NF, f = r1 - r2 * NF;
    const int pair = r2 / h.bpf[axis], fblk = r2 - pair * h.bpf[axis];
    const int fidx = 2 * pair + (blk & 1);
    const int w = h.w[f];
    if (w == 0) return;
    int a, b, c, face;
    face_of(h, axis, fidx, a, b, c, face);
    const bool high = face & 1;
    const int area = (int)h.area[axis];
    const int ex = h.e[0], ey = h.e[1], ez = h.e[2];

    // the field's box in the buffer, and the state at the face's first layer
    // at tangential cell 0
    Real* const B = buf + (face_offset(h, a, b, c, face) * h.wsum + (long long)h.wpre[f] * area);
    const int ci = axis == 0 && high ? (a + 1) * ex - w : a * ex;
    const int cj = axis == 1 && high ? (b + 1) * ey - w : b * ey;
    const int ck = axis == 2 && high ? (c + 1) * ez - w : c * ez;
    Real* const Q = q + (f * fs + cell_off(d, ci, cj, ck));
    // steps of the layers, and of the tangential cells (ta, tb): (j, k) on i
    // faces, (i, k) on j faces, (i, j) on k faces; the box is in (k, j, i)
    // order, i fastest
    const int ne = axis == 0 ? ey : ex;
    const int lq = axis == 0 ? 1 : (axis == 1 ? d.sy : d.sz), lb = axis == 0 ? 1 : (axis == 1 ? ex : area);
    const int qa = axis == 0 ? d.sy : 1, qb = axis == 2 ? d.sy : d.sz;
    const int ba = axis == 0 ? w : 1, bb = axis == 2 ? ex : ne * w;
    // two layers of an i face move as one pair where the address allows
    auto pairs = [&](const Real* p) { return axis == 0 && w == 2 && (reinterpret_cast<uintptr_t>(p) % sizeof(R2)) == 0; };
    // rows of the state start at even elements and boxes hold pairs, so that
    // one answer holds for all cells
    const bool qpair = pairs(Q), bpair = pairs(B);

    int oq[HALO_ROWS], ob[HALO_ROWS];
    bool ok[HALO_ROWS];
    Real v[HALO_ROWS][2];
#pragma unroll
    for (int r = 0; r < HALO_ROWS; ++r) {
        const int t = fblk * (HALO_THREADS * HALO_ROWS) + r * HALO_THREADS + threadIdx.x;
        ok[r] = t < area;
        const int tb = t / ne, ta = t - tb * ne;
        oq[r] = ok[r] ? tb * qb + ta * qa : 0;
        ob[r] = ok[r] ? tb * bb + ta * ba : 0;
    }
    auto get = [&](const Real* P, const int* o, int l, bool pair) __attribute__((always_inline)) {
        if (pair) {
#pragma unroll
            for (int r = 0; r < HALO_ROWS; ++r) {
                const R2 x = *reinterpret_cast<const R2*>(P + o[r]);
                v[r][0] = x.x;
                v[r][1] = x.y;
            }
        } else {
#pragma unroll
            for (int r = 0; r < HALO_ROWS; ++r) {
                v[r][0] = P[o[r]];
                if (w > 1) v[r][1] = P[o[r] + l];
            }
        }
    };
    auto put = [&](Real* P, const int* o, int l, bool pair) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < HALO_ROWS; ++r) {
            if (!ok[r]) continue;
            if (pair) {
                R2 x;
                x.x = v[r][0];
                x.y = v[r][1];
                *reinterpret_cast<R2*>(P + o[r]) = x;
            } else {
                P[o[r]] = v[r][0];
                if (w > 1) P[o[r] + l] = v[r][1];
            }
        }
    };
    if (MODE == HALO_UNPACK) get(B, ob, lb, bpair);
    else get(Q, oq, lq, qpair);
    if (MODE != HALO_UNPACK) put(B, ob, lb, bpair);
    if (MODE != HALO_PACK) put(Q, oq, lq, qpair);
}

template <typename Real>
hipError_t launch_halo(const Dims& d, const HaloGeom& h, StateT<Real> q, Real* buf, HaloMode mode, hipStream_t s)
{
    const int nb = h.blk_end[2];
    if (nb <= 0) return hipSuccess;
    // A step with its exchange, all fields against one field a thread, by the
    // elements exchanged: 0.2 M (64^3 2x2x2) 21.5 against 15.9 us, 0.5 M (96^3)
    // 34.4 against 28.3, 0.66 M (96^3 4x2x1) 36.9 against 34.0, 0.88 M (126x128x128
    // 3x2x1) 41.3 against 45.6, 1.2 M (FP32 128^3 4x2x1) 34.6 against 36.9, 2.7 M
    // (FP32 224^3 2x2x2) 134 against 139: there the first has its loads in flight
    // with fewer threads to start.
    const double elems = ((double)h.nface[0] * h.area[0] + (double)h.nface[1] * h.area[1] + (double)h.nface[2] * h.area[2]) * h.wsum;
    auto go = [&](auto m) {
        constexpr HaloMode MODE = decltype(m)::value;
        if (elems <= 700000)
            halo_field_kernel<Real, MODE><<<nb * NF, HALO_THREADS, 0, s>>>(d, h, q.f[1] - q.f[0], q.f[0], buf);
        else
            halo_kernel<Real, MODE><<<nb, HALO_THREADS, 0, s>>>(d, h, q, buf);
    };
    if (mode == HALO_PACK) go(std::integral_constant<HaloMode, HALO_PACK>{});
    else if (mode == HALO_UNPACK) go(std::integral_constant<HaloMode, HALO_UNPACK>{});
    else go(std::integral_constant<HaloMode, HALO_EXCHANGE>{});
    return hipGetLastError();
}
template hipError_t launch_halo<double>(const Dims&, const HaloGeom&, StateT<double>, double*, HaloMode, hipStream_t);
template hipError_t launch_halo<float>(const Dims&, const HaloGeom&, StateT<float>, float*, HaloMode, hipStream_t);

}  // namespace cav
