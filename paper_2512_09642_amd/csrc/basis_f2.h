// Two steps of the Chebyshev basis recurrence (Sec. 2, Definition) in one pass
// over memory, for the constant-coefficient 7- and 27-point operators with a
// constant Jacobi weight (Sec. 8 model problems):
//   q       = p_{j+1} = 2 theta (M^{-1} A p_j - sigma p_j) - p_{j-1}
//                       (theta (M^{-1} A p_0 - sigma p_0) when j = 0)
//   p_{j+2}           = 2 theta (M^{-1} A q - sigma q) - p_j
// Each value is formed with the same operations, in the same order, as by one
// single step (OpPoisson7 and OpPoisson27, common.h), so the pair equals two
// single steps bit for bit.
//
// HBM traffic per point: p_{j-1} and p_j read, q and p_{j+2} written, 4
// vectors for two columns against 6 for two single steps.
//
// Layout of the work.  A block of 16 waves owns an in-plane tile and a range
// of planes, which it marches in z.  A wave holds two grid rows, a lane one
// x-position of both, so the extended tile is 64 x 32 points: the interior
// plus two points on each side (one where the grid ends inside the tile).
// All of it loads p_j; q is formed everywhere, and is right one point inside
// the extended tile; p_{j+2} is stored on the interior.  No value is read
// from outside the extended tile, so a plane step has no edge cases: a
// missing neighbour in the grid reads as 0 because the loads of points
// outside it return 0 and q is selected to 0 there.  Two rows per lane share
// the offsets, the plane's masks, the barrier and the row between them.
// Planes of p_j and q sit in LDS, double-buffered with one barrier per plane;
// the planes above and below come from registers.
//
// What bounds it: instruction issue and HBM together.  A plane step is 145
// instructions for the 7-point operator (FP64 with products) over two points
// per lane, against 165 and eight branches for one point per lane in the form
// that read each neighbour under a condition: 224^3, average of the 8 launches
// of s = 16, 91 -> 76.6 us (3.8 -> 4.55 TB/s algorithmic); FP32 at 187 x 173 x
// 191, 47 -> 25 us.  27-point, 230^3: 2 x 194 us as single steps of 27 loads
// per point -> 94 us per pair (sums of rows, then planes, each formed once).
// Measured slower at 224^3: blocks of 8 waves (82.1 us), 4 planes of loads in
// flight (80.1), cached stores (81.8), non-temporal loads of p_{j-1} (78.0).
// Marching every other launch downward, to meet the planes last written, is
// worth 0-5% and would double the instantiations.
#pragma once

#include "common.h"

namespace sstep {

constexpr int kF2Lanes = 64;                   // extended tile width: one wave holds whole tile rows
constexpr int kF2Waves = 16;
constexpr int kF2Threads = kF2Lanes * kF2Waves;
constexpr int kF2Ext = 2 * kF2Waves;           // extended tile rows
constexpr int kF2Cus = 256;                    // blocks that run at a time: one per CU
constexpr int kF2MaxPlanes = 512;              // longest range tried

// Planes a block marches beyond its range: q needs one plane on each side;
// the 27-point sums of p_j two below and, p_{j+2} being formed two planes
// behind, one more above.
constexpr int f2_extra(bool box) { return box ? 5 : 2; }

struct F2Plan {
    uint32_t tiles_x, tiles_y, ranges;  // tiles along x / along y, z-ranges
    int txi, tyi;                       // interior points of a tile along x / y
    int xoff, yoff;                     // ring points before the interior
    int kz;                             // planes per range
    uint32_t nbl, per;                  // logical blocks, logical blocks per XCD
};

// Tiles of one axis: one tile (the grid ends inside it, one ring point) when
// the axis fits, else equal tiles with two ring points on each side.
inline void f2_axis(int n, int ext, uint32_t *tiles, int *ti, int *off)
{
    if (n <= ext - 2) {
        *tiles = 1, *ti = n, *off = 1;
        return;
    }
    *tiles = static_cast<uint32_t>((n + ext - 5) / (ext - 4));
    *ti = (n + static_cast<int>(*tiles) - 1) / static_cast<int>(*tiles);
    *off = 2;
}

// Byte window one block addresses: its planes, two below and two above.
inline int64_t f2_window_bytes(const Grid3 &g, int kz, int elem)
{
    return static_cast<int64_t>(kz + 4) * g.nxy * elem;
}

// Largest window of a block (kMark below).
constexpr int64_t kF2MaxWindow = (int64_t(1) << 30) - 1;

// Planes per range: the smallest number of plane steps the busiest CU makes,
// rounds * (kz + extra + start-up), the start-up (first loads, reductions)
// counted as two steps; 224^3: 28 planes, one block on each CU.
inline F2Plan plan_f2(const Grid3 &g, bool box, int elem)
{
    F2Plan p;
    f2_axis(g.nx, kF2Lanes, &p.tiles_x, &p.txi, &p.xoff);
    f2_axis(g.ny, kF2Ext, &p.tiles_y, &p.tyi, &p.yoff);
    const int64_t tiles = static_cast<int64_t>(p.tiles_x) * p.tiles_y;
    int64_t best = INT64_MAX;
    p.kz = 1;
    for (int kz = 2; kz <= kF2MaxPlanes && (kz == 2 || kz <= g.nz); ++kz) {
        if (kz > 2 && f2_window_bytes(g, kz, elem) > kF2MaxWindow)
            break;
        const int64_t nbl = tiles * ((g.nz + kz - 1) / kz);
        const int64_t cost = (nbl + kF2Cus - 1) / kF2Cus * (kz + f2_extra(box) + 2);
        if (cost < best)
            best = cost, p.kz = kz;
    }
    p.ranges = static_cast<uint32_t>((g.nz + p.kz - 1) / p.kz);
    p.nbl = static_cast<uint32_t>(tiles) * p.ranges;
    p.per = (p.nbl + kNumXcd - 1) / kNumXcd;
    return p;
}

// Barrier for LDS traffic only: its fences order LDS accesses, so global
// loads issued before it stay in flight (the fence of __syncthreads makes
// every wave wait for all of its outstanding global loads at each barrier).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Raw buffer access through a resource that covers one window of a vector:
// an offset at or beyond the window's size reads 0 and drops a store, so the
// kernel predicates its memory accesses on the offset alone and every load
// and store is issued unconditionally (no branch around a memory access, and
// no select on a loaded value, which the compiler would turn back into a
// branch): the compiler can then count the loads in flight and keeps them
// in flight across the barriers.
//
// Offsets are a per-lane base plus a block-uniform plane offset; either is
// kMark when the point or the plane does not exist.  Every window stays below
// 1 GiB = kMark, so such a sum lies outside it.
constexpr uint32_t kMark = 0x40000000u;
constexpr int32_t kRsrcWord3 = 0x00020000;  // raw buffer, 32-bit data format (gfx9 family)
constexpr int kNonTemporal = 2;             // cache-policy bit of a buffer access: non-temporal
typedef unsigned int U32x2 __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_window(const T *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(base), 0, static_cast<int>(bytes), kRsrcWord3);
}

__device__ __forceinline__ double buf_load(double, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ float buf_load(float, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
// A value read once.
__device__ __forceinline__ double buf_load_once(double, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kNonTemporal));
}
__device__ __forceinline__ float buf_load_once(float, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kNonTemporal));
}
// FP64 results are stored non-temporally, FP32 ones through the caches: the
// 248-byte FP32 row pieces end mid-line, and L2 merges such partial lines
// only for cached stores (FP32 pair 47 us cached against 62 us
// non-temporal, FP64 84 us non-temporal against 87 us cached, in the
// solve's setting at 224^3).
__device__ __forceinline__ void buf_store_out(double v, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U32x2, v), r, off, 0, kNonTemporal);
}
__device__ __forceinline__ void buf_store_out(float v, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, 0);
}

// D: planes by which the global loads run ahead of their use (a ring of D
// register slots per loaded stream, the loop unrolled by D so that every
// slot index is a constant).
// BOX: the 27-point operator, else the 7-point one.
// MOM (moments Gram kind): the block also sums, over the points it stores,
// <q, p_j>, <q, q>, <p_{j+2}, q>, <p_{j+2}, p_{j+2}> (and <p_0, p_0> first
// when FIRST), unweighted (the constant diagonal is applied afterwards), and
// writes them to consecutive slots of mpart, stride mstride, at its logical
// block index.
template <typename T, bool BOX, bool FIRST, int D, bool MOM>
__global__ __launch_bounds__(kF2Threads, kF2Waves / 4) void k_basis_f2(
    const DevState *__restrict__ st, Grid3 g, T minv, const T *__restrict__ pprev, const T *__restrict__ pj,
    T *__restrict__ qout, T *__restrict__ p2out, T theta, T sigma, F2Plan plan, double *__restrict__ mpart,
    int64_t mstride)
{
    constexpr uint32_t ES = sizeof(T);
    constexpr int W = kF2Lanes;
    constexpr int PAD = W + 8;  // reads beside the extended tile's edge stay inside the array
    __shared__ T ps[2][kF2Ext * W + 2 * PAD];
    __shared__ T qs[2][kF2Ext * W + 2 * PAD];
    if (st->done)
        return;
    const uint32_t lb = xcd_block(blockIdx.x, plan.per);
    if (lb >= plan.nbl)
        return;  // whole block: no barrier is skipped by part of it
    const uint32_t ntile = plan.tiles_x * plan.tiles_y;
    const uint32_t zr = lb / ntile, tile = lb - zr * ntile;
    const uint32_t ty = tile / plan.tiles_x, tx = tile - ty * plan.tiles_x;
    const int lane = threadIdx.x % W, wave = threadIdx.x / W;
    const int gi = static_cast<int>(tx) * plan.txi - plan.xoff + lane;
    const int gj = static_cast<int>(ty) * plan.tyi - plan.yoff + 2 * wave;  // rows gj and gj + 1
    const int li = lane - plan.xoff, lj = 2 * wave - plan.yoff;             // position in the interior
    const bool dx = gi >= 0 && gi < g.nx;
    const bool dom0 = dx && gj >= 0 && gj < g.ny, dom1 = dx && gj + 1 >= 0 && gj + 1 < g.ny;
    const bool ix = li >= 0 && li < plan.txi;
    const bool int0 = dom0 && ix && lj >= 0 && lj < plan.tyi;
    const bool int1 = dom1 && ix && lj + 1 >= 0 && lj + 1 < plan.tyi;
    // q (and with it p_{j-1}) is needed on the interior and one point around it
    const bool rx = li >= -1 && li <= plan.txi;
    const bool rq0 = dom0 && rx && lj >= -1 && lj <= plan.tyi;
    const bool rq1 = dom1 && rx && lj + 1 >= -1 && lj + 1 <= plan.tyi;
    const int k0 = static_cast<int>(zr) * plan.kz;
    const int k1 = k0 + plan.kz < g.nz ? k0 + plan.kz : g.nz;
    // the block's window: planes kb .. ke - 1 of every vector (p_j is read
    // from two planes below the range to one plane above it)
    const int kb = k0 - 2 > 0 ? k0 - 2 : 0;
    const int ke = k1 + 2 < g.nz ? k1 + 2 : g.nz;
    const uint32_t plane = static_cast<uint32_t>(g.nxy) * ES;
    const uint32_t wbytes = static_cast<uint32_t>(ke - kb) * plane;
    const int64_t wbase = static_cast<int64_t>(kb) * g.nxy;
    const __amdgpu_buffer_rsrc_t rj = make_window(pj + wbase, wbytes);
    const __amdgpu_buffer_rsrc_t rv = make_window(FIRST ? pj + wbase : pprev + wbase, wbytes);
    const __amdgpu_buffer_rsrc_t rq = make_window(qout + wbase, wbytes);
    const __amdgpu_buffer_rsrc_t r2 = make_window(p2out + wbase, wbytes);
    const uint32_t pl0 = static_cast<uint32_t>(gj * g.nx + gi) * ES, pl1 = pl0 + static_cast<uint32_t>(g.nx) * ES;
    const uint32_t bj0 = dom0 ? pl0 : kMark, bj1 = dom1 ? pl1 : kMark;  // p_j
    const uint32_t bv0 = rq0 ? pl0 : kMark, bv1 = rq1 ? pl1 : kMark;    // p_{j-1}
    const uint32_t bs0 = int0 ? pl0 : kMark, bs1 = int1 ? pl1 : kMark;  // stored points
    // block-uniform plane offset, kMark outside [klo, khi]
    auto po = [&](int k, int klo, int khi) -> uint32_t {
        return k >= klo && k <= khi ? static_cast<uint32_t>(k - kb) * plane : kMark;
    };
    const int kj_hi = k1 + 1 < g.nz ? k1 + 1 : g.nz - 1;  // last plane of p_j the range reads
    const int kq_lo = k0 > 0 ? k0 - 1 : 0;                // planes q is formed on
    const int kq_hi = k1 < g.nz ? k1 : g.nz - 1;
    const T two_theta = T(2) * theta;
    const int i0 = PAD + 2 * wave * W + lane;  // LDS slot of the first row's point; the second is W further
    // first plane step; the 27-point sums of p_j start two planes earlier
    const int kfirst = BOX ? k0 - 3 : k0 - 1;
    const int nstep = (k1 - k0 + f2_extra(BOX) + D - 1) / D * D;
    // p_j on the current plane kq, and below it
    T c0 = T(0), c1 = T(0), m0 = T(0), m1 = T(0), l0 = T(0), l1 = T(0);
    if constexpr (!BOX) {
        m0 = buf_load(T(), rj, bj0 + po(k0 - 2, 0, kj_hi)), m1 = buf_load(T(), rj, bj1 + po(k0 - 2, 0, kj_hi));
        c0 = buf_load(T(), rj, bj0 + po(k0 - 1, 0, kj_hi)), c1 = buf_load(T(), rj, bj1 + po(k0 - 1, 0, kj_hi));
    }
    T qc0 = T(0), qc1 = T(0), qb0 = T(0), qb1 = T(0);  // q one and two planes below the current one
    // in-plane 3 x 3 sums (BOX): of p_j on planes kq - 1 and kq, of q on kq - 3 and kq - 2
    T pm0 = T(0), pm1 = T(0), pc0 = T(0), pc1 = T(0), um0 = T(0), um1 = T(0), uc0 = T(0), uc1 = T(0);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0, s4 = 0.0;  // products (MOM)
    // slot u holds, for plane kq = kfirst + u (mod D): p_j on plane kq + 1
    // and p_{j-1} on plane kq
    T pjs[D][2], pvs[D][2];
    auto fill = [&](int u, int kq) {
        const uint32_t oj = po(kq + 1, 0, kj_hi);
        pjs[u][0] = buf_load(T(), rj, bj0 + oj);
        pjs[u][1] = buf_load(T(), rj, bj1 + oj);
        if constexpr (!FIRST) {
            const uint32_t ov = po(kq, kq_lo, kq_hi);
            pvs[u][0] = buf_load(T(), rv, bv0 + ov);
            pvs[u][1] = buf_load(T(), rv, bv1 + ov);
        }
    };
#pragma unroll
    for (int u = 0; u < D; ++u)
        fill(u, kfirst + u);
    // steps past the last plane load nothing (their offsets lie outside the
    // window) and store nothing
    for (int base = kfirst; base < kfirst + nstep; base += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int kq = base + u;
            T *const P = ps[u & 1], *const Q = qs[u & 1];
            static_assert(D % 2 == 0, "the LDS buffers alternate with the slot");
            const T t0 = pjs[u][0], t1 = pjs[u][1];  // p_j on plane kq + 1
            T v0 = T(0), v1 = T(0);
            if constexpr (!FIRST)
                v0 = pvs[u][0], v1 = pvs[u][1];
            T y0, y1, z0, z1;  // A p_j on plane kq; A q on the second step's plane
            T q0, q1;
            const bool act = kq >= kq_lo && kq <= kq_hi;  // block-uniform
            auto first_step = [&](T y, T c, T v) -> T {
                if constexpr (FIRST)
                    return theta * (minv * y - sigma * c);
                else
                    return two_theta * (minv * y - sigma * c) - v;
            };
            if constexpr (BOX) {
                P[i0] = t0, P[i0 + W] = t1;
                Q[i0] = qc0, Q[i0 + W] = qc1;
                lds_barrier();
                // 3 x 3 sums of the plane just exchanged: rows south of the
                // first, first, second, north of the second, each centre,
                // west, east
                auto sums = [&](const T *a, T x0, T x1, T &r0, T &r1) {
                    const T rs = (a[i0 - W] + a[i0 - W - 1]) + a[i0 - W + 1];
                    const T ra = (x0 + a[i0 - 1]) + a[i0 + 1];
                    const T rb = (x1 + a[i0 + W - 1]) + a[i0 + W + 1];
                    const T rn = (a[i0 + 2 * W] + a[i0 + 2 * W - 1]) + a[i0 + 2 * W + 1];
                    r0 = (rs + ra) + rb;
                    r1 = (ra + rb) + rn;
                };
                T pt0, pt1, ut0, ut1;
                sums(P, t0, t1, pt0, pt1);
                sums(Q, qc0, qc1, ut0, ut1);
                y0 = T(27) * c0 - ((pm0 + pc0) + pt0);
                y1 = T(27) * c1 - ((pm1 + pc1) + pt1);
                z0 = T(27) * qb0 - ((um0 + uc0) + ut0);
                z1 = T(27) * qb1 - ((um1 + uc1) + ut1);
                pm0 = pc0, pm1 = pc1, pc0 = pt0, pc1 = pt1;
                um0 = uc0, um1 = uc1, uc0 = ut0, uc1 = ut1;
                q0 = first_step(y0, c0, v0);
                q1 = first_step(y1, c1, v1);
                q0 = dom0 && act ? q0 : T(0);
                q1 = dom1 && act ? q1 : T(0);
            } else {
                P[i0] = c0, P[i0 + W] = c1;
                lds_barrier();
                y0 = T(6) * c0 - (((((P[i0 - 1] + P[i0 + 1]) + P[i0 - W]) + c1) + m0) + t0);
                y1 = T(6) * c1 - (((((P[i0 + W - 1] + P[i0 + W + 1]) + c0) + P[i0 + 2 * W]) + m1) + t1);
                q0 = first_step(y0, c0, v0);
                q1 = first_step(y1, c1, v1);
                q0 = dom0 && act ? q0 : T(0);
                q1 = dom1 && act ? q1 : T(0);
                // q on the plane below was stored before this plane's barrier
                const T *R = qs[(u & 1) ^ 1];
                z0 = T(6) * qc0 - (((((R[i0 - 1] + R[i0 + 1]) + R[i0 - W]) + qc1) + qb0) + q0);
                z1 = T(6) * qc1 - (((((R[i0 + W - 1] + R[i0 + W + 1]) + qc0) + R[i0 + 2 * W]) + qb1) + q1);
                Q[i0] = q0, Q[i0 + W] = q1;
            }
            {
                const uint32_t oq = po(kq, k0, k1 - 1);
                buf_store_out(q0, rq, bs0 + oq);
                buf_store_out(q1, rq, bs1 + oq);
            }
            // second step, on plane kq - 1 (BOX: kq - 2)
            const int k2 = BOX ? kq - 2 : kq - 1;
            const T a0 = BOX ? l0 : m0, a1 = BOX ? l1 : m1;       // p_j there
            const T b0 = BOX ? qb0 : qc0, b1 = BOX ? qb1 : qc1;   // q there
            const T w0 = two_theta * (minv * z0 - sigma * b0) - a0;
            const T w1 = two_theta * (minv * z1 - sigma * b1) - a1;
            {
                const uint32_t o2 = po(k2, k0, k1 - 1);
                buf_store_out(w0, r2, bs0 + o2);
                buf_store_out(w1, r2, bs1 + o2);
            }
            if constexpr (MOM) {
                // the points just stored; a product with q or p_{j+2}
                // selected to 0 elsewhere adds 0
                const bool in = k2 >= k0 && k2 < k1;  // block-uniform
                const bool own0 = int0 && in, own1 = int1 && in;
                const double e0 = own0 ? static_cast<double>(b0) : 0.0, e1 = own1 ? static_cast<double>(b1) : 0.0;
                const double f0 = own0 ? static_cast<double>(w0) : 0.0, f1 = own1 ? static_cast<double>(w1) : 0.0;
                const double d0 = static_cast<double>(a0), d1 = static_cast<double>(a1);
                if constexpr (FIRST) {
                    s0 += (own0 ? d0 : 0.0) * d0;
                    s0 += (own1 ? d1 : 0.0) * d1;
                }
                s1 += e0 * d0, s1 += e1 * d1;
                s2 += e0 * e0, s2 += e1 * e1;
                s3 += f0 * e0, s3 += f1 * e1;
                s4 += f0 * f0, s4 += f1 * f1;
            }
            qb0 = qc0, qb1 = qc1, qc0 = q0, qc1 = q1;
            if constexpr (BOX)
                l0 = m0, l1 = m1;
            m0 = c0, m1 = c1, c0 = t0, c1 = t1;
            // refill the slot for plane kq + D once its values are used, so
            // that the load writes the slot's own registers
            fill(u, kq + D);
        }
    }
    if constexpr (MOM) {
        double *out = mpart + lb;
        if constexpr (FIRST) {
            const double v[5] = {s0, s1, s2, s3, s4};
            block_partials<5, kF2Threads>(v, out, mstride);
        } else {
            const double v[4] = {s1, s2, s3, s4};
            block_partials<4, kF2Threads>(v, out, mstride);
        }
    }
}

}  // namespace sstep
