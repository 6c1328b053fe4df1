// Bands of whole grid rows: what the kernels of a batch and of one large
// face-coefficient system share.  A block of kBf2Lanes threads owns a band of
// rows [y0, y1) over a range of planes [k0, k1) and marches it in z, two
// points a lane.
#pragma once

#include "bands.h"
#include "basis_f2.h"

namespace sstep {

// Two neighbouring points of a lane, loaded and stored together: an 8-byte
// access per lane takes the L1 as long as a 16-byte one.
template <typename T>
struct Two {
    T a, b;
};
__device__ __forceinline__ Two<double> buf_load2(double, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(Two<double>, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ Two<float> buf_load2(float, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(Two<float>, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
typedef unsigned int U32x4 __attribute__((ext_vector_type(4)));
// CACHED: the next launch finds the values in the last-level cache.
template <bool CACHED = false>
__device__ __forceinline__ void buf_store2(Two<double> v, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U32x4, v), r, off, 0, CACHED ? 0 : kNonTemporal);
}
template <bool CACHED = false>
__device__ __forceinline__ void buf_store2(Two<float> v, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U32x2, v), r, off, 0, 0);
}

// A lane's two points of a band: slots 2t and 2t + 1 of the block's rows
// [ye0, ye1) laid end to end, so that the second may be the first point of
// the next row (turn).
struct BandLane {
    int i0, i1;               // x positions
    bool dom0, dom1;          // the points exist
    bool int0, int1;          // ... and belong to the band
    bool hs0, hs1, hn0, hn1;  // the row below / above is in the block
    bool turn;
    uint32_t pl;              // index of the first point within a plane
    // LDS slots of the neighbours (of the pairs below and above), or a zero slot
    int iw, ie, is, in;
};
constexpr int kBf2Lanes = kBf2Threads / 2;
// LDS slots of a plane: two zeros, the points, and zeros that the pair of the
// last point can reach.
constexpr int kBf2Front = 2, kBf2Slots = kBf2Front + kBf2Threads + 2;
__device__ __forceinline__ BandLane band_lane(int nx, int y0, int y1, int ye0, int ye1)
{
    BandLane l;
    const int t0 = 2 * static_cast<int>(threadIdx.x);
    const int er = t0 / nx;
    l.i0 = t0 - er * nx;
    l.turn = l.i0 + 1 == nx;
    l.i1 = l.turn ? 0 : l.i0 + 1;
    const int e0 = ye0 + er, e1 = l.turn ? e0 + 1 : e0;
    l.dom0 = e0 < ye1, l.dom1 = e1 < ye1;
    l.int0 = l.dom0 && e0 >= y0 && e0 < y1, l.int1 = l.dom1 && e1 >= y0 && e1 < y1;
    l.hs0 = l.dom0 && e0 > ye0, l.hs1 = l.dom1 && e1 > ye0;
    l.hn0 = l.dom0 && e0 + 1 < ye1, l.hn1 = l.dom1 && e1 + 1 < ye1;
    l.pl = l.dom0 ? static_cast<uint32_t>(ye0 * nx + t0) : 0u;
    const int s0 = kBf2Front + t0;
    l.iw = l.dom0 && l.i0 > 0 ? s0 - 1 : 0;
    l.ie = l.dom1 && l.i1 + 1 < nx ? s0 + 2 : 0;
    l.is = l.hs0 || l.hs1 ? s0 - nx : 0;
    l.in = l.hn0 || l.hn1 ? s0 + nx : 0;
    return l;
}

// One vector and operator of band_pair.
template <typename T>
struct BandArgs {
    int nx, ny, nz, precond;
    T theta, sigma;
    const T *kx, *ky, *kz;  // faces (null: the constant operator)
    const T *pj, *pprev;    // p_j and p_{j-1}
    T *q, *p2;              // p_{j+1} and p_{j+2}
};

// Two basis steps for one vector per block (Sec. 2, Definition, taken twice):
//   q       = p_{j+1} from p_j and p_{j-1} (from p_0 alone when j = 0)
//   p_{j+2} = 2 theta (M^{-1} A q - sigma q) - p_j
// with every value formed by the operations, in the order, of k_bbasis, so
// the pair equals two single steps bit for bit.  A block owns a band of whole
// grid rows [y0, y1) of one system and a range of planes [k0, k1), and forms
// q on the band and on the row below and the row above it (when the grid has
// them), so that the second step finds every in-plane neighbour in the
// block; it marches the range in z with the current plane of p_j and of q in
// LDS and the planes above and below in registers, as the single-system pair
// kernel does.  Face coefficients are read once per point and plane (the
// bottom face is the top face of the plane below); the Jacobi weight is
// formed from them by the single step's expression.
//
// What bounds it: vector memory instructions through the L1, about 20 cycles
// each, whether a lane takes 8 or 16 bytes, then the latency of loads that
// wait behind stores in the same counter.  So a lane holds two neighbouring
// points, the Jacobi weight is not loaded, waves without ring rows skip those
// loads, and a plane's loads go out before the step's stores (20 systems of
// 32^3 to 96^3, 8 right-hand sides, FP64: 690 us a launch with one point per
// lane, 577 with two, 502 with the loads ahead of the stores; the weight
// loaded adds 40 us, three planes in flight instead of two change nothing).
// The points of the block's rows lie end to end, so the second of a lane may
// be the first of the next row: its x-faces are then one entry further, and
// the lane's two points are no x-neighbours.  Steps are unrolled so that the
// slots of the loads in flight, the LDS buffers and the planes in registers
// change names instead of places.
//
// The loop body has no branch but the waves' with ring rows: a neighbour that
// does not exist is read from a zero slot of the LDS plane (or, across the
// block's first and last rows, taken from the register loaded from global
// memory), and every value is formed and then selected.  Every memory access
// is a buffer access at a per-lane base plus a block-uniform plane offset;
// either is kMark when the point or the plane does not exist, and since every
// window stays below 1 GiB = kMark, such a sum lies outside it (the load
// returns 0, the store is dropped).
//
// MOM (moments Gram kind): the block also sums, over the points it stores,
// <q, M p_j>, <q, M q>, <p_{j+2}, M q>, <p_{j+2}, M p_{j+2}> (and
// <p_0, M p_0> first when FIRST), M the face diagonal with Jacobi (1 for the
// constant operator, whose diagonal the FGS kernel applies), and writes them
// to out, stride apart.
template <typename T, bool FACES, bool FIRST, int D, bool MOM, bool CACHED>
__device__ __forceinline__ void band_pair(const BandArgs<T> &a, int y0, int y1, int k0, int k1, double *out,
                                          int64_t stride)
{
    constexpr uint32_t ES = sizeof(T);
    using V = Two<T>;
    __shared__ T ps[2][kBf2Slots];
    __shared__ T qs[2][kBf2Slots];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const uint32_t nxy = static_cast<uint32_t>(nx) * static_cast<uint32_t>(ny);
    const int tid = threadIdx.x;
    if (tid < 2 * (kBf2Slots - kBf2Threads)) {
        const int z = tid / 2 < kBf2Front ? tid / 2 : kBf2Threads + tid / 2;
        ps[tid & 1][z] = T(0);
        qs[tid & 1][z] = T(0);
    }
    // The first plane step reads the other plane of q before any was stored: what
    // it forms is not stored, but its products are summed with weight 0, and what
    // an earlier block left in the LDS may be NaN.
    qs[1][kBf2Front + 2 * tid] = qs[1][kBf2Front + 2 * tid + 1] = T(0);
    // rows of the block: the band and the row on each side of it
    const int ye0 = y0 > 0 ? y0 - 1 : 0;
    const int ye1 = y1 < ny ? y1 + 1 : ny;
    const BandLane l = band_lane(nx, y0, y1, ye0, ye1);
    const int own = kBf2Front + 2 * tid;  // LDS slot of the first point
    // A point of the first or last row of the block reads its one neighbour
    // outside the block from global memory (0 where the grid ends there).
    const bool rs0 = l.dom0 && !l.hs0 && ye0 > 0, rs1 = l.dom1 && !l.hs1 && ye0 > 0;
    const bool rn0 = l.dom0 && !l.hn0 && ye1 < ny, rn1 = l.dom1 && !l.hn1 && ye1 < ny;
    const bool ring_wave = __ballot(rs0 || rs1 || rn0 || rn1) != 0;  // the others issue no ring loads
    const uint32_t b_pt = l.dom0 ? l.pl * ES : kMark;  // the points
    const uint32_t b_in = l.int0 && l.int1 ? l.pl * ES : kMark;  // the points, stored by this block
    // points stored alone: the other of the lane is in a ring row or past the rows
    const bool lone = l.int0 != l.int1;
    const bool lone_wave = __ballot(lone) != 0;
    const uint32_t b_ln = lone ? (l.int0 ? l.pl : l.pl + 1) * ES : kMark;
    const uint32_t b_r0 = rs0 ? (l.pl - nx) * ES : rn0 ? (l.pl + nx) * ES : kMark;
    const uint32_t b_r1 = rs1 ? (l.pl + 1 - nx) * ES : rn1 ? (l.pl + 1 + nx) * ES : kMark;
    const uint32_t pbytes = nxy * ES;
    const uint32_t cbytes = nxy * static_cast<uint32_t>(nz) * ES;
    const __amdgpu_buffer_rsrc_t rj = make_window(a.pj, cbytes);
    const __amdgpu_buffer_rsrc_t rv = make_window(FIRST ? a.pj : a.pprev, cbytes);
    const __amdgpu_buffer_rsrc_t rq = make_window(a.q, cbytes);
    const __amdgpu_buffer_rsrc_t r2 = make_window(a.p2, cbytes);
    // faces: x-faces (nx + 1 per grid row), y-faces (ny + 1 rows of nx per
    // plane), z-faces (nz + 1 planes)
    const uint32_t xrow = static_cast<uint32_t>(nx + 1);
    const uint32_t xplane = static_cast<uint32_t>(ny) * xrow * ES, yplane = static_cast<uint32_t>(ny + 1) * nx * ES;
    const __amdgpu_buffer_rsrc_t rfx = make_window(a.kx, static_cast<uint32_t>(nz) * xplane);
    const __amdgpu_buffer_rsrc_t rfy = make_window(a.ky, static_cast<uint32_t>(nz) * yplane);
    const __amdgpu_buffer_rsrc_t rfz = make_window(a.kz, (static_cast<uint32_t>(nz) + 1) * pbytes);
    const uint32_t b_fx = l.dom0 ? (l.pl + l.pl / static_cast<uint32_t>(nx)) * ES : kMark;
    const T theta = a.theta, sigma = a.sigma;
    const T two_theta = T(2) * theta;
    const T minv_c = a.precond ? T(1) / T(6) : T(1);
    // slot u holds, for plane kq = k0 - 1 + u (mod D): p_j on plane kq + 1,
    // p_{j-1}, the ring neighbours and the faces of plane kq
    V pjs[D], pps[D], rgs[D];
    V fxa[FACES ? D : 1], fxb[FACES ? D : 1], fss[FACES ? D : 1], fns[FACES ? D : 1], fts[FACES ? D : 1];
    // a slot filled for plane kn; past the range and below the grid at kMark
    // (no memory is read).  Plane kn = nz lies past the windows.
    auto refill = [&](int u, int kn) {
        const bool more = kn >= 0 && kn <= k1;
        const uint32_t o = more ? static_cast<uint32_t>(kn) * pbytes : kMark;
        const uint32_t up = b_pt + (kn <= k1 ? static_cast<uint32_t>(kn + 1) * pbytes : kMark);
        pjs[u] = buf_load2(T(), rj, up);
        if constexpr (!FIRST)
            pps[u] = buf_load2(T(), rv, b_pt + o);
        if constexpr (FACES) {
            const uint32_t ox = b_fx + (more ? static_cast<uint32_t>(kn) * xplane : kMark);
            const uint32_t oy = b_pt + (more ? static_cast<uint32_t>(kn) * yplane : kMark);
            fxa[u] = buf_load2(T(), rfx, ox);
            fxb[u] = buf_load2(T(), rfx, ox + 2 * ES);
            fss[u] = buf_load2(T(), rfy, oy);
            fns[u] = buf_load2(T(), rfy, oy + static_cast<uint32_t>(nx) * ES);
            fts[u] = buf_load2(T(), rfz, up);
        }
        if (ring_wave) {
            rgs[u].a = buf_load(T(), rj, b_r0 + o);
            rgs[u].b = buf_load(T(), rj, b_r1 + o);
        }
    };
    auto in_rows = [&](V v) -> V { return {v.a, l.dom1 ? v.b : T(0)}; };  // the second point may lie past the rows
    auto plane = [&](int k) -> uint32_t { return k >= 0 ? static_cast<uint32_t>(k) * pbytes : kMark; };
    V pm = in_rows(buf_load2(T(), rj, b_pt + plane(k0 - 2)));  // p_j one plane below the current one
    V p0 = in_rows(buf_load2(T(), rj, b_pt + plane(k0 - 1)));  // p_j on the current plane
    V qb{T(0), T(0)}, qc{T(0), T(0)};  // q two planes and one plane below the current one
    V fb{T(0), T(0)};                  // bottom faces of the current plane
    if constexpr (FACES)
        fb = buf_load2(T(), rfz, b_pt + plane(k0 - 1));
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0, m4 = 0.0;  // products (MOM)
    // coefficients, Jacobi weights and diagonal of the plane below (the second step's plane)
    V gw{}, ge{}, gs{}, gn{}, gb{}, gt{}, gd{}, gm{};
#pragma unroll
    for (int u = 0; u < D; ++u) {
        pps[u] = rgs[u] = V{T(0), T(0)};
        refill(u, k0 - 1 + u);
    }
    // planes k0 - 1 .. k1
    constexpr int kU = 6;
    static_assert(kU % D == 0 && kU % 2 == 0, "slots and LDS buffers alternate within the unrolled steps");
    const double wd = a.precond ? 1.0 : 0.0, wc = a.precond ? 0.0 : 1.0;
    uint32_t so2 = kMark;  // offset of the plane below, kMark outside the range
    for (int kq = k0 - 1;;) {
#pragma unroll
        for (int v = 0; v < kU; ++v) {
            const int u = v % D, buf = v & 1;
            const V pp = in_rows(pjs[u]), pv = pps[u], rg = rgs[u];
            const uint32_t so = static_cast<uint32_t>(kq - k0) < static_cast<uint32_t>(k1 - k0)
                                    ? static_cast<uint32_t>(kq) * pbytes
                                    : kMark;
            const bool act = kq >= 0 && kq < nz;  // block-uniform
            V fw{}, fe{}, fs{}, fn{}, ft{}, d{T(1), T(1)}, dinv{minv_c, minv_c};
            ps[buf][own] = p0.a, ps[buf][own + 1] = p0.b;
            lds_barrier();
            if constexpr (FACES) {
                fw = {fxa[u].a, l.turn ? fxb[u].a : fxa[u].b};
                fe = {fxa[u].b, l.turn ? fxb[u].b : fxb[u].a};
                fs = fss[u], fn = fns[u], ft = fts[u];
                d.a = ((((fw.a + fe.a) + fs.a) + fn.a) + fb.a) + ft.a;
                d.b = ((((fw.b + fe.b) + fs.b) + fn.b) + fb.b) + ft.b;
                // off the grid q = 0
                // the condition chooses what is divided by: chosen behind the
                // divisions it becomes a branch, and the loads below wait for it
                const V den{a.precond ? d.a : T(1), a.precond ? d.b : T(1)};
                dinv = {T(1) / den.a, T(1) / den.b};
                dinv = {l.dom0 && act ? dinv.a : T(0), l.dom1 && act ? dinv.b : T(0)};
            }
            V q;
            {
                const T *pl = ps[buf];
                const T w0 = pl[l.iw], e1 = pl[l.ie];
                const T e0 = l.turn ? T(0) : p0.b, w1 = l.turn ? T(0) : p0.a;
                const T sl0 = pl[l.is], sl1 = pl[l.is + 1], nl0 = pl[l.in], nl1 = pl[l.in + 1];
                const T s0 = l.hs0 ? sl0 : rg.a, s1 = l.hs1 ? sl1 : rg.b;
                const T n0 = l.hn0 ? nl0 : rg.a, n1 = l.hn1 ? nl1 : rg.b;
                V y;
                if constexpr (FACES) {
                    y.a = face_sum(fw.a, p0.a - w0, fe.a, p0.a - e0, fs.a, p0.a - s0, fn.a, p0.a - n0, fb.a,
                                   p0.a - pm.a, ft.a, p0.a - pp.a);
                    y.b = face_sum(fw.b, p0.b - w1, fe.b, p0.b - e1, fs.b, p0.b - s1, fn.b, p0.b - n1, fb.b,
                                   p0.b - pm.b, ft.b, p0.b - pp.b);
                } else {
                    y.a = T(6) * p0.a - (((((w0 + e0) + s0) + n0) + pm.a) + pp.a);
                    y.b = T(6) * p0.b - (((((w1 + e1) + s1) + n1) + pm.b) + pp.b);
                }
                if constexpr (FIRST) {
                    q.a = theta * (dinv.a * y.a - sigma * p0.a);
                    q.b = theta * (dinv.b * y.b - sigma * p0.b);
                } else {
                    q.a = two_theta * (dinv.a * y.a - sigma * p0.a) - pv.a;
                    q.b = two_theta * (dinv.b * y.b - sigma * p0.b) - pv.b;
                }
                if constexpr (!FACES) {
                    q.a = l.dom0 && act ? q.a : T(0);
                    q.b = act ? q.b : T(0);
                }
                q.b = l.dom1 ? q.b : T(0);
            }
            refill(u, kq + D);
            buf_store2<CACHED>(q, rq, b_in + so);
            if (lone_wave)
                buf_store_out(l.int0 ? q.a : q.b, rq, b_ln + so);
            qs[buf][own] = q.a, qs[buf][own + 1] = q.b;
            // the second step on the plane below: q there is in qs[buf ^ 1]
            // (stored before this plane's barrier), q below it in qb, above in q
            {
                const T *ql = qs[buf ^ 1];
                const T w0 = ql[l.iw], e1 = ql[l.ie];
                const T e0 = l.turn ? T(0) : qc.b, w1 = l.turn ? T(0) : qc.a;
                const T s0 = ql[l.is], s1 = ql[l.is + 1], n0 = ql[l.in], n1 = ql[l.in + 1];
                V y;
                if constexpr (FACES) {
                    y.a = face_sum(gw.a, qc.a - w0, ge.a, qc.a - e0, gs.a, qc.a - s0, gn.a, qc.a - n0, gb.a,
                                   qc.a - qb.a, gt.a, qc.a - q.a);
                    y.b = face_sum(gw.b, qc.b - w1, ge.b, qc.b - e1, gs.b, qc.b - s1, gn.b, qc.b - n1, gb.b,
                                   qc.b - qb.b, gt.b, qc.b - q.b);
                } else {
                    y.a = T(6) * qc.a - (((((w0 + e0) + s0) + n0) + qb.a) + q.a);
                    y.b = T(6) * qc.b - (((((w1 + e1) + s1) + n1) + qb.b) + q.b);
                }
                V p2;
                p2.a = two_theta * ((FACES ? gd.a : minv_c) * y.a - sigma * qc.a) - pm.a;
                p2.b = two_theta * ((FACES ? gd.b : minv_c) * y.b - sigma * qc.b) - pm.b;
                buf_store2<CACHED>(p2, r2, b_in + so2);
                if (lone_wave)
                    buf_store_out(l.int0 ? p2.a : p2.b, r2, b_ln + so2);
                if constexpr (MOM) {
                    // the plane just stored: p_j, q and p_{j+2} of plane kq - 1
                    const bool stored = so2 != kMark;
                    auto sum = [&](bool in, T diag, T pa, T qa, T p2a) {
                        double w = 1.0;
                        if constexpr (FACES)
                            w = __builtin_elementwise_fma(static_cast<double>(diag), wd, wc);
                        w = in && stored ? w : 0.0;
                        const double a = static_cast<double>(pa), b = static_cast<double>(qa);
                        const double c = static_cast<double>(p2a);
                        if constexpr (FIRST)
                            m0 += w * a * a;
                        m1 += w * b * a;
                        m2 += w * b * b;
                        m3 += w * c * b;
                        m4 += w * c * c;
                    };
                    sum(l.int0, gm.a, pm.a, qc.a, p2.a);
                    sum(l.int1, gm.b, pm.b, qc.b, p2.b);
                }
            }
            qb = qc;
            qc = q;
            pm = p0;
            p0 = pp;
            if constexpr (FACES) {
                gw = fw, ge = fe, gs = fs, gn = fn, gb = fb, gt = ft, gd = dinv, gm = d;
                fb = ft;
            }
            so2 = so;
            if (kq++ == k1)
                goto done;
        }
    }
done:
    if constexpr (MOM && FIRST) {
        const double v[5] = {m0, m1, m2, m3, m4};
        block_partials<5, kBf2Lanes>(v, out, stride);
    } else if constexpr (MOM) {
        const double v[4] = {m1, m2, m3, m4};
        block_partials<4, kBf2Lanes>(v, out, stride);
    }
}

}  // namespace sstep
