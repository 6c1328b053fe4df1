// Two steps of the Chebyshev basis in one launch for small 7-point systems
// (constant or face coefficients) and for thin ones (constant):
//   q       = p_{j+1} from p_j and p_{j-1} (from p_0 alone when j = 0)
//   p_{j+2} = 2 theta (M^{-1} A q - sigma q) - p_j
// A block owns a brick of points, 8 x 8 x 8 in all but thin grids; each of its
// threads forms q at one point of it or of the ring around it, from memory (the caches, at these
// sizes), and after one exchange through LDS those of the brick form p_{j+2}
// from their own faces and the neighbours' q.  No march and no second load.
//
// What bounds it: the launch and one chain of loads, as a single step's, paid
// once for two columns; half of q is formed twice, which costs little while
// the chip is not filled (45^3, s = 16, face coefficients: 5.4 us for two
// columns, 6.4 in single steps; constant operator 4.6, 8.8 by the march).
#pragma once

#include "band_f2.h"
#include "launch.h"
#include "stop.h"

namespace sstep {

constexpr int kBrickThreads = 1024;  // points of a brick and its ring, at most

// A brick of w points along each axis and its extended form of e: two points
// more where the grid goes on (o = 1), none where the brick spans it (o = 0).
struct BrickAxis {
    int32_t w, e, o, cnt;
};
struct BrickPlan {
    BrickAxis x, y, z;
    uint32_t nbl, per;
    bool cube() const { return x.e == 10 && x.o && y.e == 10 && y.o && z.e == 10 && z.o; }
};
inline BrickAxis brick_axis(int n, int w)
{
    return w >= n ? BrickAxis{n, n, 0, 1} : BrickAxis{w, w + 2, 1, (n + w - 1) / w};
}
inline BrickPlan brick_plan(BrickAxis x, BrickAxis y, BrickAxis z)
{
    const uint32_t nbl = static_cast<uint32_t>(x.cnt) * static_cast<uint32_t>(y.cnt) * static_cast<uint32_t>(z.cnt);
    return {x, y, z, nbl, (nbl + kNumXcd - 1) / kNumXcd};
}
// Cubes of 8 points (10 with the ring), unless the grid is so thin that they
// would be mostly empty: then the shape with the fewest blocks.
inline BrickPlan plan_brick(const Grid3 &g)
{
    BrickPlan best = brick_plan(brick_axis(g.nx, 8), brick_axis(g.ny, 8), brick_axis(g.nz, 8));
    if (static_cast<int64_t>(best.nbl) * 512 <= 2 * g.nxy * g.nz)
        return best;
    best.nbl = 0;
    constexpr int kTry[] = {1022, 510, 254, 126, 62, 30, 14, 8, 6, 2, 1};
    for (int wx : kTry)
        for (int wy : kTry)
            for (int wz : kTry) {
                const BrickAxis x = brick_axis(g.nx, wx), y = brick_axis(g.ny, wy), z = brick_axis(g.nz, wz);
                if (static_cast<int64_t>(x.e) * y.e * z.e > kBrickThreads)
                    continue;
                const BrickPlan p = brick_plan(x, y, z);
                if (!best.nbl || p.nbl < best.nbl)
                    best = p;
                break;  // a shorter one of these takes no fewer blocks (planned for each launch of a solve without a graph)
            }
    return best;
}

// MOM: the product sums of the pair (band_pair), one partial per brick.
// STOP: the launch also makes the stopping test (small_chain, j = 0).
// CUBE: 8 points and a ring along every axis, known to the compiler.
template <typename T, bool FACES, bool FIRST, bool MOM, bool STOP, bool CUBE>
__global__ __launch_bounds__(kBrickThreads) void k_basis_brick(DevState *__restrict__ st, BandArgs<T> a,
                                                               BrickPlan plan, double *__restrict__ mpart,
                                                               int64_t mstride, StopArgs stop)
{
    __shared__ T qs[kBrickThreads];
    // with the test in this launch the flag may be set as the block starts: the
    // block leaves at the test's barrier
    const int done = wave_done(st);
    if (!STOP && done)
        return;
    const uint32_t lb = xcd_block(blockIdx.x, plan.per);
    if (lb >= plan.nbl)
        return;  // whole block
    double share = 0.0;
    if constexpr (STOP)
        if (!done)
            share = partial_share<kBrickThreads>(stop);
    const uint32_t cxy = static_cast<uint32_t>(plan.x.cnt) * plan.y.cnt;
    const int bz = static_cast<int>(lb / cxy), bxy = static_cast<int>(lb - bz * cxy);
    const int by = bxy / plan.x.cnt, bx = bxy - by * plan.x.cnt;
    const int tid = threadIdx.x;
    const int wx = CUBE ? 8 : plan.x.w, wy = CUBE ? 8 : plan.y.w, wz = CUBE ? 8 : plan.z.w;
    const int sx = CUBE ? 10 : plan.x.e, sxy = CUBE ? 100 : plan.x.e * plan.y.e, sz = CUBE ? 10 : plan.z.e;  // slots
    const int ox = CUBE ? 1 : plan.x.o, oy = CUBE ? 1 : plan.y.o, oz = CUBE ? 1 : plan.z.o;
    const int ez = tid / sxy, r = tid - ez * sxy;
    const int ey = r / sx, ex = r - ey * sx;
    const int i = bx * wx + ex - ox, j = by * wy + ey - oy, k = bz * wz + ez - oz;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t nxy = static_cast<int64_t>(nx) * ny;
    const bool dom = ez < sz && i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz;
    const bool own = dom && ex >= ox && ex < ox + wx && ey >= oy && ey < oy + wy && ez >= oz && ez < oz + wz;
    const int64_t c = dom ? (static_cast<int64_t>(k) * ny + j) * nx + i : 0;
    const T two_theta = T(2) * a.theta;
    T pc = T(0), q = T(0), dinv = a.precond ? T(1) / T(6) : T(1), d = T(1);
    T fw = T(0), fe = T(0), fs = T(0), fn = T(0), fb = T(0), ft = T(0);
    if (dom && !done) {
        const T *__restrict__ p = a.pj;
        pc = p[c];
        const T w = i > 0 ? p[c - 1] : T(0), e = i + 1 < nx ? p[c + 1] : T(0);
        const T s = j > 0 ? p[c - nx] : T(0), n = j + 1 < ny ? p[c + nx] : T(0);
        const T b = k > 0 ? p[c - nxy] : T(0), t = k + 1 < nz ? p[c + nxy] : T(0);
        T pv = T(0);
        if constexpr (!FIRST)
            pv = a.pprev[c];
        T y;
        if constexpr (FACES) {
            const int64_t row = static_cast<int64_t>(k) * ny + j;
            const int64_t fx = c + row, fy = c + static_cast<int64_t>(k) * nx;
            fw = a.kx[fx], fe = a.kx[fx + 1], fs = a.ky[fy], fn = a.ky[fy + nx], fb = a.kz[c], ft = a.kz[c + nxy];
            d = ((((fw + fe) + fs) + fn) + fb) + ft;
            dinv = a.precond ? T(1) / d : T(1);
            y = face_sum(fw, pc - w, fe, pc - e, fs, pc - s, fn, pc - n, fb, pc - b, ft, pc - t);
        } else {
            y = T(6) * pc - (((((w + e) + s) + n) + b) + t);
        }
        if constexpr (FIRST)
            q = a.theta * (dinv * y - a.sigma * pc);
        else
            q = two_theta * (dinv * y - a.sigma * pc) - pv;
    }
    qs[tid] = q;  // 0 off the grid
    if constexpr (STOP)
        if (stop_at_head<kBrickThreads>(st, done, stop, share, lb == 0))
            return;
    __syncthreads();
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0, m4 = 0.0;
    if (own) {
        // an own point's neighbours have slots wherever the grid goes on; a cube
        // has them beyond the grid too, where q = 0
        const T w = CUBE || i > 0 ? qs[tid - 1] : T(0), e = CUBE || i + 1 < nx ? qs[tid + 1] : T(0);
        const T s = CUBE || j > 0 ? qs[tid - sx] : T(0), n = CUBE || j + 1 < ny ? qs[tid + sx] : T(0);
        const T b = CUBE || k > 0 ? qs[tid - sxy] : T(0), t = CUBE || k + 1 < nz ? qs[tid + sxy] : T(0);
        T y;
        if constexpr (FACES)
            y = face_sum(fw, q - w, fe, q - e, fs, q - s, fn, q - n, fb, q - b, ft, q - t);
        else
            y = T(6) * q - (((((w + e) + s) + n) + b) + t);
        const T p2 = two_theta * (dinv * y - a.sigma * q) - pc;
        a.q[c] = q;
        a.p2[c] = p2;
        if constexpr (MOM) {
            const double wt = FACES && a.precond ? static_cast<double>(d) : 1.0;
            const double u0 = static_cast<double>(pc), u1 = static_cast<double>(q), u2 = static_cast<double>(p2);
            m0 = wt * u0 * u0, m1 = wt * u1 * u0, m2 = wt * u1 * u1, m3 = wt * u2 * u1, m4 = wt * u2 * u2;
        }
    }
    if constexpr (MOM && FIRST) {
        const double v[5] = {m0, m1, m2, m3, m4};
        block_partials<5, kBrickThreads>(v, mpart + lb, mstride);
    } else if constexpr (MOM) {
        const double v[4] = {m1, m2, m3, m4};
        block_partials<4, kBrickThreads>(v, mpart + lb, mstride);
    }
}

}  // namespace sstep
