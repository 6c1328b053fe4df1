// Two steps of the Chebyshev basis in one launch for small 7-point systems
// (constant or face coefficients):
//   q       = p_{j+1} from p_j and p_{j-1} (from p_0 alone when j = 0)
//   p_{j+2} = 2 theta (M^{-1} A q - sigma q) - p_j
// A block owns a brick of 8 x 8 x 8 points; each of its threads forms q at one
// point of the 10 x 10 x 10 around it, from memory (the caches, at these
// sizes), and after one exchange through LDS those of the brick form p_{j+2}
// from their own faces and the neighbours' q.  No march and no second load.
//
// What bounds it: the launch and one chain of loads, as a single step's, paid
// once for two columns; half of q is formed twice, which costs little while
// the chip is not filled (45^3, s = 16, face coefficients: 5.2 us for two
// columns, 6.4 in single steps; constant operator 4.4, 8.8 by the march).
#pragma once

#include "band_f2.h"
#include "launch.h"
#include "stop.h"

namespace sstep {

constexpr int kBrick = 8, kBrickExt = kBrick + 2, kBrickPoints = kBrickExt * kBrickExt * kBrickExt;
constexpr int kBrickThreads = 1024;

struct BrickPlan {
    uint32_t bx, by, nbl, per;
};
inline BrickPlan plan_brick(const Grid3 &g)
{
    auto cut = [](int n) { return static_cast<uint32_t>((n + kBrick - 1) / kBrick); };
    BrickPlan p;
    p.bx = cut(g.nx), p.by = cut(g.ny);
    p.nbl = p.bx * p.by * cut(g.nz);
    p.per = (p.nbl + kNumXcd - 1) / kNumXcd;
    return p;
}

// MOM: the product sums of the pair (band_pair), one partial per brick.
// STOP: the launch also makes the stopping test (small_chain, j = 0).
template <typename T, bool FACES, bool FIRST, bool MOM, bool STOP>
__global__ __launch_bounds__(kBrickThreads) void k_basis_brick(DevState *__restrict__ st, BandArgs<T> a,
                                                               BrickPlan plan, double *__restrict__ mpart,
                                                               int64_t mstride, StopArgs stop)
{
    __shared__ T qs[kBrickPoints];
    if (st->done)
        return;
    const uint32_t lb = xcd_block(blockIdx.x, plan.per);
    if (lb >= plan.nbl)
        return;  // whole block
    double share = 0.0;
    if constexpr (STOP)
        share = partial_share<kBrickThreads>(stop);
    const int bz = static_cast<int>(lb / (plan.bx * plan.by)), bxy = static_cast<int>(lb - bz * plan.bx * plan.by);
    const int by = bxy / static_cast<int>(plan.bx), bx = bxy - by * static_cast<int>(plan.bx);
    const int tid = threadIdx.x;
    const int ez = tid / (kBrickExt * kBrickExt), exy = tid - ez * kBrickExt * kBrickExt;
    const int ey = exy / kBrickExt, ex = exy - ey * kBrickExt;
    const int i = bx * kBrick + ex - 1, j = by * kBrick + ey - 1, k = bz * kBrick + ez - 1;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t nxy = static_cast<int64_t>(nx) * ny;
    const bool dom = tid < kBrickPoints && i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz;
    const bool own = dom && ex >= 1 && ex <= kBrick && ey >= 1 && ey <= kBrick && ez >= 1 && ez <= kBrick;
    const int64_t c = dom ? (static_cast<int64_t>(k) * ny + j) * nx + i : 0;
    const T two_theta = T(2) * a.theta;
    T pc = T(0), q = T(0), dinv = a.precond ? T(1) / T(6) : T(1), d = T(1);
    T fw = T(0), fe = T(0), fs = T(0), fn = T(0), fb = T(0), ft = T(0);
    if (dom) {
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
    if (tid < kBrickPoints)
        qs[tid] = q;  // 0 off the grid
    if constexpr (STOP)
        if (stop_at_head<kBrickThreads>(st, stop, share, lb == 0))
            return;
    __syncthreads();
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0, m4 = 0.0;
    if (own) {
        const T w = qs[tid - 1], e = qs[tid + 1], s = qs[tid - kBrickExt], n = qs[tid + kBrickExt];
        const T b = qs[tid - kBrickExt * kBrickExt], t = qs[tid + kBrickExt * kBrickExt];
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
