// One application of a constant-coefficient operator (7- or 27-point) to a
// vector in one pass over memory, with what the outer iteration does with it:
// the residual and basis start (Sec. 2), or one step of the Chebyshev
// recurrence (Sec. 2, Definition).
//
// The layout is that of the two-step basis (basis_f2.h) with a ring of one
// point: a block of 16 waves owns an in-plane tile of at most 62 x 30 points
// of its 64 x 32 extended tile and marches a range of planes; a wave holds
// two grid rows, a lane one x-position of both.  Planes of the vector sit in
// LDS, double-buffered with one barrier per plane, and each is read from
// memory once per range; the 27-point operator sums rows, then planes, each
// sum formed once per point instead of 27 loads per point.  Values are formed
// with the operations of OpPoisson7 / OpPoisson27 (common.h), in their order.
//
// What bounds it: HBM at large grids (27-point residual at 230^3 in a solve 371 -> 58
// us, 5.1 TB/s algorithmic; 7-point at 224^3 62.5 -> 50 us, stopping test
// included), the chain of planes at small ones, where a thread per point is
// kept.
#pragma once

#include "basis_f2.h"
#include "march_rule.h"

namespace sstep {

// Blocks that run at a time: the kernels below stay within 64 registers.
constexpr int kMarchCus = 2 * kF2Cus;
static_assert(kMarchLanes == kF2Lanes && kMarchRows == kF2Ext, "the rule counts the lanes of these tiles");

// Planes per range by the same cost as plan_f2 (one plane below and one above
// the range; the 27-point sums start one step earlier).
inline F2Plan plan_march(const Grid3 &g, bool box, int elem)
{
    F2Plan p;
    auto axis = [](int n, int ext, uint32_t *tiles, int *ti) {
        *tiles = static_cast<uint32_t>((n + ext - 3) / (ext - 2));
        *ti = (n + static_cast<int>(*tiles) - 1) / static_cast<int>(*tiles);
    };
    axis(g.nx, kF2Lanes, &p.tiles_x, &p.txi);
    axis(g.ny, kF2Ext, &p.tiles_y, &p.tyi);
    p.xoff = p.yoff = 1;
    const int64_t tiles = static_cast<int64_t>(p.tiles_x) * p.tiles_y;
    int64_t best = INT64_MAX;
    p.kz = 1;
    for (int kz = 2; kz <= kF2MaxPlanes && (kz == 2 || kz <= g.nz); ++kz) {
        if (kz > 2 && f2_window_bytes(g, kz, elem) > kF2MaxWindow)
            break;
        const int64_t nbl = tiles * ((g.nz + kz - 1) / kz);
        const int64_t cost = (nbl + kMarchCus - 1) / kMarchCus * (kz + (box ? 2 : 0) + 3);
        if (cost < best)
            best = cost, p.kz = kz;
    }
    p.ranges = static_cast<uint32_t>((g.nz + p.kz - 1) / p.kz);
    p.nbl = static_cast<uint32_t>(tiles) * p.ranges;
    p.per = (p.nbl + kNumXcd - 1) / kNumXcd;
    return p;
}

// Marches y = A u over the block's range and calls f(point, plane, centre u,
// y, second stream's value) for the two points of the lane on each plane of
// the range; point 0 / 1, called by every lane (values outside the tile are
// not A u).  v: the second stream, read on the interior (none when !SECOND).
// sh: 2 (32 x 64 + 144) elements of LDS.
template <typename T, bool BOX, int D, bool SECOND, class F>
__device__ __forceinline__ void march(const F2Plan &plan, const Grid3 &g, const T *__restrict__ u,
                                      const T *__restrict__ v, uint32_t lb, T (*sh)[kF2Ext * kF2Lanes + 144], F &&f)
{
    constexpr uint32_t ES = sizeof(T);
    constexpr int W = kF2Lanes;
    constexpr int PAD = W + 8;
    const uint32_t ntile = plan.tiles_x * plan.tiles_y;
    const uint32_t zr = lb / ntile, tile = lb - zr * ntile;
    const uint32_t ty = tile / plan.tiles_x, tx = tile - ty * plan.tiles_x;
    const int lane = threadIdx.x % W, wave = threadIdx.x / W;
    const int gi = static_cast<int>(tx) * plan.txi - 1 + lane;
    const int gj = static_cast<int>(ty) * plan.tyi - 1 + 2 * wave;
    const bool dx = gi >= 0 && gi < g.nx && lane <= plan.txi + 1;
    const bool dom0 = dx && gj >= 0 && gj < g.ny, dom1 = dx && gj + 1 >= 0 && gj + 1 < g.ny;
    const bool ix = lane >= 1 && lane <= plan.txi;
    const int lj = 2 * wave - 1;
    const bool int0 = dom0 && ix && lj >= 0 && lj < plan.tyi;
    const bool int1 = dom1 && ix && lj + 1 >= 0 && lj + 1 < plan.tyi;
    const int k0 = static_cast<int>(zr) * plan.kz;
    const int k1 = k0 + plan.kz < g.nz ? k0 + plan.kz : g.nz;
    const int kb = k0 - 1 > 0 ? k0 - 1 : 0;
    const int ke = k1 + 1 < g.nz ? k1 + 1 : g.nz;
    const uint32_t plane = static_cast<uint32_t>(g.nxy) * ES;
    const uint32_t wbytes = static_cast<uint32_t>(ke - kb) * plane;
    const int64_t wbase = static_cast<int64_t>(kb) * g.nxy;
    const __amdgpu_buffer_rsrc_t ru = make_window(u + wbase, wbytes);
    const __amdgpu_buffer_rsrc_t rv = make_window(SECOND ? v + wbase : u + wbase, wbytes);
    const uint32_t pl0 = static_cast<uint32_t>(gj * g.nx + gi) * ES, pl1 = pl0 + static_cast<uint32_t>(g.nx) * ES;
    const uint32_t bu0 = dom0 ? pl0 : kMark, bu1 = dom1 ? pl1 : kMark;
    const uint32_t bv0 = int0 ? pl0 : kMark, bv1 = int1 ? pl1 : kMark;
    auto po = [&](int k, int klo, int khi) -> uint32_t {
        return k >= klo && k <= khi ? static_cast<uint32_t>(k - kb) * plane : kMark;
    };
    const int i0 = PAD + 2 * wave * W + lane;
    const int kfirst = BOX ? k0 - 2 : k0;  // the 27-point sums start one plane below the range
    const int nstep = (k1 - kfirst + D - 1) / D * D;
    T c0 = T(0), c1 = T(0), m0 = T(0), m1 = T(0);  // u on planes kq and kq - 1
    if constexpr (!BOX) {
        m0 = buf_load(T(), ru, bu0 + po(k0 - 1, 0, ke - 1)), m1 = buf_load(T(), ru, bu1 + po(k0 - 1, 0, ke - 1));
        c0 = buf_load(T(), ru, bu0 + po(k0, 0, ke - 1)), c1 = buf_load(T(), ru, bu1 + po(k0, 0, ke - 1));
    }
    T pm0 = T(0), pm1 = T(0), pc0 = T(0), pc1 = T(0);  // 3 x 3 sums on planes kq - 1 and kq (BOX)
    T us[D][2], vs[D][2];
    auto fill = [&](int s, int kq) {
        const uint32_t ou = po(kq + 1, 0, ke - 1);
        us[s][0] = buf_load(T(), ru, bu0 + ou);
        us[s][1] = buf_load(T(), ru, bu1 + ou);
        if constexpr (SECOND) {
            const uint32_t ov = po(kq, k0, k1 - 1);
            vs[s][0] = buf_load_once(T(), rv, bv0 + ov);
            vs[s][1] = buf_load_once(T(), rv, bv1 + ov);
        }
    };
#pragma unroll
    for (int s = 0; s < D; ++s)
        fill(s, kfirst + s);
    for (int base = kfirst; base < kfirst + nstep; base += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            static_assert(D % 2 == 0, "the LDS buffers alternate with the slot");
            const int kq = base + s;
            T *const P = sh[s & 1];
            const T t0 = us[s][0], t1 = us[s][1];
            T v0 = T(0), v1 = T(0);
            if constexpr (SECOND)
                v0 = vs[s][0], v1 = vs[s][1];
            T y0, y1;
            if constexpr (BOX) {
                P[i0] = t0, P[i0 + W] = t1;
                lds_barrier();
                const T rs = (P[i0 - W] + P[i0 - W - 1]) + P[i0 - W + 1];
                const T ra = (t0 + P[i0 - 1]) + P[i0 + 1];
                const T rb = (t1 + P[i0 + W - 1]) + P[i0 + W + 1];
                const T rn = (P[i0 + 2 * W] + P[i0 + 2 * W - 1]) + P[i0 + 2 * W + 1];
                const T pt0 = (rs + ra) + rb, pt1 = (ra + rb) + rn;
                y0 = T(27) * c0 - ((pm0 + pc0) + pt0);
                y1 = T(27) * c1 - ((pm1 + pc1) + pt1);
                pm0 = pc0, pm1 = pc1, pc0 = pt0, pc1 = pt1;
            } else {
                P[i0] = c0, P[i0 + W] = c1;
                lds_barrier();
                y0 = T(6) * c0 - (((((P[i0 - 1] + P[i0 + 1]) + P[i0 - W]) + c1) + m0) + t0);
                y1 = T(6) * c1 - (((((P[i0 + W - 1] + P[i0 + W + 1]) + c0) + P[i0 + 2 * W]) + m1) + t1);
            }
            // the offset of the points in a window of the same planes, kMark
            // outside the interior and the range
            const uint32_t o = po(kq, k0, k1 - 1);
            const bool in = kq >= k0 && kq < k1;
            f(bv0 + o, int0 && in, c0, y0, v0);
            f(bv1 + o, int1 && in, c1, y1, v1);
            m0 = c0, m1 = c1, c0 = t0, c1 = t1;
            fill(s, kq + D);
        }
    }
}

// r = b - A x in FP64, the block's partial of ||r||^2 at its logical block,
// and p_0 = p0scale (M^{-1} r or r) as column 0 of P (k_residual).  A marched
// plane of x is read once per range; b is read once.
template <typename TP, bool BOX>
__global__ __launch_bounds__(kF2Threads, 8) void k_residual_m(const DevState *__restrict__ st, Grid3 g, double minv,
                                                             TP *__restrict__ p0, double *__restrict__ rpart,
                                                             int p0_mode, int write_p0, F2Plan plan)
{
    __shared__ double sh[2][kF2Ext * kF2Lanes + 144];
    if (st->done)
        return;
    const uint32_t lb = xcd_block(blockIdx.x, plan.per);
    if (lb >= plan.nbl)
        return;
    const double scale = st->p0scale;
    const double wr = p0_mode ? 1.0 : minv;
    const uint32_t ntile = plan.tiles_x * plan.tiles_y;
    const int k0 = static_cast<int>(lb / ntile) * plan.kz;
    const int k1 = k0 + plan.kz < g.nz ? k0 + plan.kz : g.nz;
    const int kb = k0 - 1 > 0 ? k0 - 1 : 0, ke = k1 + 1 < g.nz ? k1 + 1 : g.nz;
    const __amdgpu_buffer_rsrc_t rp =
        make_window(p0 + static_cast<int64_t>(kb) * g.nxy,
                    write_p0 ? static_cast<uint32_t>(ke - kb) * static_cast<uint32_t>(g.nxy * sizeof(TP)) : 0u);
    double acc = 0.0;
    march<double, BOX, 2, true>(plan, g, st->x, st->b, lb, sh,
                                [&](uint32_t off, bool own, double, double y, double b) {
                                    const double r = own ? b - y : 0.0;
                                    acc += r * r;
                                    // the offset counts bytes of an FP64 window: halved (and still outside
                                    // when marked) for FP32
                                    const TP v = static_cast<TP>(scale * (wr * r));
                                    buf_store_out(v, rp, sizeof(TP) == 8 ? off : own ? off / 2 : kMark);
                                });
    const double v[1] = {acc};
    block_partials<1, kF2Threads>(v, rpart + lb, 1);
}

// One step of the Chebyshev recurrence (k_basis, k_basis_mom): p_{j+1} from
// p_j (STEP 0) or from p_j and p_{j-1} (STEP 1), A p_j into apj when it is
// kept, and with MOM the block's products <p_{j+1}, p_j>, <p_{j+1}, p_{j+1}>
// (<p_0, p_0> first with STEP 0), unweighted: the constant diagonal is
// applied afterwards.
template <typename T, bool BOX, int STEP, bool MOM>
__global__ __launch_bounds__(kF2Threads, 8) void k_basis_m(const DevState *__restrict__ st, Grid3 g, T minv,
                                                          const T *__restrict__ pj, const T *__restrict__ pprev,
                                                          T *__restrict__ apj, T *__restrict__ pnext, T theta,
                                                          T sigma, F2Plan plan, double *__restrict__ mpart,
                                                          int64_t mstride)
{
    static_assert(STEP == 0 || STEP == 1, "every launch forms a column");
    __shared__ T sh[2][kF2Ext * kF2Lanes + 144];
    if (st->done)
        return;
    const uint32_t lb = xcd_block(blockIdx.x, plan.per);
    if (lb >= plan.nbl)
        return;
    const uint32_t ntile = plan.tiles_x * plan.tiles_y;
    const int k0 = static_cast<int>(lb / ntile) * plan.kz;
    const int k1 = k0 + plan.kz < g.nz ? k0 + plan.kz : g.nz;
    const int kb = k0 - 1 > 0 ? k0 - 1 : 0, ke = k1 + 1 < g.nz ? k1 + 1 : g.nz;
    const int64_t wbase = static_cast<int64_t>(kb) * g.nxy;
    const uint32_t wbytes = static_cast<uint32_t>(ke - kb) * static_cast<uint32_t>(g.nxy * sizeof(T));
    const __amdgpu_buffer_rsrc_t rn = make_window(pnext + wbase, wbytes);
    const __amdgpu_buffer_rsrc_t ra = make_window(apj ? apj + wbase : pnext, apj ? wbytes : 0u);
    const T two_theta = T(2) * theta;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    march<T, BOX, 2, STEP == 1>(plan, g, pj, pprev, lb, sh, [&](uint32_t off, bool own, T c, T y, T v) {
        T pn;
        if constexpr (STEP == 0)
            pn = theta * (minv * y - sigma * c);
        else
            pn = two_theta * (minv * y - sigma * c) - v;
        if constexpr (!MOM)
            buf_store_out(y, ra, off);
        buf_store_out(pn, rn, off);
        if constexpr (MOM) {
            const double a = own ? static_cast<double>(pn) : 0.0, b = static_cast<double>(c);
            if constexpr (STEP == 0)
                s0 += (own ? b : 0.0) * b;
            s1 += a * b;
            s2 += a * a;
        }
    });
    if constexpr (MOM) {
        if constexpr (STEP == 0) {
            const double v[3] = {s0, s1, s2};
            block_partials<3, kF2Threads>(v, mpart + lb, mstride);
        } else {
            const double v[2] = {s1, s2};
            block_partials<2, kF2Threads>(v, mpart + lb, mstride);
        }
    }
}

}  // namespace sstep
