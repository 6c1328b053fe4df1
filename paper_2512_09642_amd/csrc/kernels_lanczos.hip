// Spectrum bounds for the Chebyshev basis by Lanczos (Sec. 8, setup of the
// experiments): a few Lanczos steps on M^{-1}A give Ritz values that
// approximate its extreme eigenvalues from inside.
//
// M^{-1}A is self-adjoint in the M-inner product <u, v>_M = u^T M v, so the
// recurrence runs on M-orthonormal vectors z_j (no reorthogonalisation):
//     z_0 = u / ||u||_M,  beta_0 = 0,
//     y = A z_j,  alpha_j = z_j^T y,
//     w = M^{-1} y - alpha_j z_j - beta_j z_{j-1},
//     beta_{j+1} = ||w||_M,  z_{j+1} = w / beta_{j+1},
// stopping early (m = j + 1 steps) when beta_{j+1} is not above
// 1e-13 max_{i<=j} |alpha_i| or not finite.  The Ritz values are the
// eigenvalues of the m x m tridiagonal T_m = tridiag(beta; alpha; beta),
// found on the device by sections on Sturm counts, one wave per eigenvalue.
//
// A step is two passes over row chunks, HBM- (or cache-) bound like the basis
// kernels, with one partial sum per block: the product and alpha, then w and
// beta.  No launch of its own sums the partials or divides by beta: every
// block of the next pass sums them in the same order (at most 1024, 8 KB from
// the L2), and the vectors stay w, divided where they are read, entry by entry: a
// factor common to the vector, the reciprocal of its norm, would carry one
// rounding error into every entry.
// 10 steps on a 128^3 faces operator, s = 16: 571 -> 447 us per call; the
// product 19.7 us and w 16.0 us at 5.1 and 5.3 TB/s out of the last-level
// cache (twice the blocks: 20.1 and 19.0), the Ritz values 43 -> 13.6 us.
#include "launch.h"
#include "opsel.h"
#include "stop.h"

namespace sstep {
namespace {

// M diagonal and its inverse at a point: constant (Poisson, or no
// preconditioner) or from the library's diagonal arrays.
struct Diag {
    const double *d;     // M diagonal, or null for the constant dconst
    const double *dinv;  // M^{-1} diagonal (CSR), or null: 1/d
    double dconst;

    __device__ __forceinline__ void at(int64_t c, double &dd, double &di) const
    {
        if (d) {
            dd = d[c];
            di = dinv ? dinv[c] : 1.0 / dd;
        } else {
            dd = dconst;
            di = 1.0 / dconst;
        }
    }
};

__device__ __forceinline__ void block_partial(double v, double *out)
{
    __shared__ double part[kBlock / kWave];
    v = wave_sum(v);
    if (threadIdx.x % kWave == 0)
        part[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double acc = part[0];
#pragma unroll
        for (int q = 1; q < kBlock / kWave; ++q)
            acc += part[q];
        *out = acc;
    }
}

// Partial sums of ||u||_M^2 = sum d u^2.
__global__ __launch_bounds__(kBlock) void k_lz_norm0(Diag dg, const double *__restrict__ u,
                                                     double *__restrict__ part, int64_t n, int64_t chunk)
{
    const int64_t beg = static_cast<int64_t>(blockIdx.x) * chunk;
    const int64_t end = beg + chunk < n ? beg + chunk : n;
    double acc = 0.0;
    for (int64_t c = beg + threadIdx.x; c < end; c += kBlock) {
        double d, di;
        dg.at(c, d, di);
        acc += d * u[c] * u[c];
    }
    block_partial(acc, part + blockIdx.x);
}

// Sum of the block partials by a block of kBlock threads, the same in every block
// and in every thread.
__device__ __forceinline__ double sum_partials(const double *__restrict__ part, int cnt)
{
    double v = 0.0;
    for (int q = threadIdx.x; q < cnt; q += kBlock)
        v += part[q];
    v = wave_sum(v);
    __shared__ double wsum[kBlock / kWave];
    if (threadIdx.x % kWave == 0)
        wsum[threadIdx.x / kWave] = v;
    __syncthreads();
    v = wsum[0];
#pragma unroll
    for (int q = 1; q < kBlock / kWave; ++q)
        v += wsum[q];
    return v;
}

// beta_{j} ends the recurrence: not above 1e-13 amax, or not finite.
__device__ __forceinline__ bool beta_stops(double beta, double amax)
{
    return !(beta > 1e-13 * amax) || !isfinite(beta);
}

// y = A z_j with z_j = w_j / scale, and partial sums of z_j^T y.  scale is
// the root of the last partials: ||u||_M (j = 0, w_0 = u) or beta_j; the
// first block records it and the end of the recurrence.
template <class Op>
__global__ __launch_bounds__(kBlock) void k_lz_apply(LzState *__restrict__ ls, const double *__restrict__ w,
                                                     double *__restrict__ y, const double *__restrict__ pin,
                                                     double *__restrict__ pout, double *__restrict__ ab, int j,
                                                     int steps, int cnt, uint32_t per, int64_t n, int64_t chunk,
                                                     Op op)
{
    const uint32_t lb = xcd_block(blockIdx.x, per);
    if (lb >= static_cast<uint32_t>(cnt))
        return;  // whole block
    // the first block may end the recurrence as this one starts: one thread
    // reads the flag, and the barrier of the sum hands it to all
    __shared__ int ended;
    if (threadIdx.x == 0)
        ended = ls->stopped;
    const double scale = sqrt(sum_partials(pin, cnt));
    if (ended)
        return;
    // j = 0: amax = 0, a zero or non-finite start
    const bool stop = beta_stops(scale, ls->amax);
    if (lb == 0 && threadIdx.x == 0) {
        if (j == 0)
            ls->scale = scale;
        else
            ab[steps + j - 1] = scale;
        ls->m = j;
        if (stop)
            ls->stopped = 1;
    }
    if (stop)
        return;
    const int64_t beg = static_cast<int64_t>(lb) * chunk;
    const int64_t end = beg + chunk < n ? beg + chunk : n;
    double acc = 0.0;
#pragma unroll 2
    for (int64_t c = beg + threadIdx.x; c < end; c += kBlock) {
        double pc, yy, dinv;
        op.apply(w, c, pc, yy, dinv);
        yy /= scale;
        y[c] = yy;
        acc += pc * yy;
    }
    block_partial(acc / scale, pout + lb);
}

// w_{j+1} = M^{-1} y - alpha_j z_j - beta_j z_{j-1} (in place of y) and
// partial sums of ||w_{j+1}||_M^2; alpha_j is the sum of the last partials,
// recorded by the first block.  wprev is null for j = 0.
__global__ __launch_bounds__(kBlock) void k_lz_orth(LzState *__restrict__ ls, Diag dg, double *__restrict__ y,
                                                    const double *__restrict__ w, const double *__restrict__ wprev,
                                                    const double *__restrict__ pin, double *__restrict__ pout,
                                                    double *__restrict__ ab, int j, int steps, int cnt,
                                                    uint32_t per, int64_t n, int64_t chunk)
{
    const uint32_t lb = xcd_block(blockIdx.x, per);
    if (ls->stopped || lb >= static_cast<uint32_t>(cnt))
        return;  // whole block
    const double alpha = sum_partials(pin, cnt);
    if (lb == 0 && threadIdx.x == 0) {
        ab[j] = alpha;
        ls->amax = fmax(ls->amax, fabs(alpha));
    }
    const double sj = j > 0 ? ab[steps + j - 1] : ls->scale;  // z_j = w_j / sj
    const double sp = j > 1 ? ab[steps + j - 2] : ls->scale;  // and z_{j-1} = w_{j-1} / sp, beta_j = sj
    const int64_t beg = static_cast<int64_t>(lb) * chunk;
    const int64_t end = beg + chunk < n ? beg + chunk : n;
    double acc = 0.0;
    auto point = [&](int64_t c, double zp) {
        double d, di;
        dg.at(c, d, di);
        const double v = di * y[c] - alpha * (w[c] / sj) - sj * zp;
        y[c] = v;
        acc += d * v * v;
    };
    if (j > 0)
#pragma unroll 4
        for (int64_t c = beg + threadIdx.x; c < end; c += kBlock)
            point(c, wprev[c] / sp);
    else
#pragma unroll 4
        for (int64_t c = beg + threadIdx.x; c < end; c += kBlock)
            point(c, 0.0);
    block_partial(acc, pout + lb);
}

// Number of eigenvalues of T_m below x (Sturm count: negative pivots of the
// LDL^T factorisation of T_m - x I).
__device__ int sturm_count(const double *al, const double *be, int m, double x, double pivmin)
{
    int cnt = 0;
    double d = al[0] - x;
    if (fabs(d) < pivmin)
        d = -pivmin;
    cnt += d < 0.0;
    for (int i = 1; i < m; ++i) {
        d = (al[i] - x) - be[i - 1] * be[i - 1] / d;
        if (fabs(d) < pivmin)
            d = -pivmin;
        cnt += d < 0.0;
    }
    return cnt;
}

// Ritz values of T_m, ascending: block k (one wave) narrows the Gershgorin
// interval of T_m to the k-th smallest eigenvalue until the interval can no
// longer be divided in FP64.  A section is 64 points, one a lane: 9 or 10
// chains of divisions instead of the 53 of a bisection.  The first block also
// records the last beta, summed like the others by all its waves: the digits
// of a step do not depend on how many follow.
__global__ __launch_bounds__(kBlock) void k_lz_ritz(LzState *__restrict__ ls, const double *__restrict__ pin, int cnt,
                                                   double *__restrict__ ab, int steps, double *__restrict__ ritz)
{
    __shared__ double al[kMaxLanczos], be[kMaxLanczos];
    const int lane = threadIdx.x, k = blockIdx.x;  // the first wave divides
    const int stopped = ls->stopped;
    const int m = stopped ? ls->m : steps;
    if (k == 0 && !stopped) {
        const double beta = sqrt(sum_partials(pin, cnt));
        if (lane == 0) {
            ab[2 * steps - 1] = beta;
            ls->m = steps;
        }
    }
    if (k >= m)
        return;
    if (lane < m) {
        al[lane] = ab[lane];
        be[lane] = lane + 1 < m ? ab[steps + lane] : 0.0;
    }
    __syncthreads();
    if (lane >= kWave)
        return;
    double lo = al[0], hi = al[0], tmax = 0.0;
    for (int i = 0; i < m; ++i) {
        const double r = (i > 0 ? fabs(be[i - 1]) : 0.0) + (i + 1 < m ? fabs(be[i]) : 0.0);
        lo = fmin(lo, al[i] - r);
        hi = fmax(hi, al[i] + r);
        tmax = fmax(tmax, fabs(al[i]) + r);
    }
    const double pivmin = 1e-300 + 4.0 * 2.2250738585072014e-308 * fmax(1.0, tmax * tmax);
    for (int it = 0; it < 64; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (!(mid > lo && mid < hi))
            break;
        // ascending; the middle lane takes the midpoint itself, so that every section divides the interval
        const double x = lane == kWave / 2 ? mid : lo + (hi - lo) * ((lane + 0.5) / (kWave + 1));
        const uint64_t above = __ballot(sturm_count(al, be, m, x, pivmin) > k);
        const int f = above ? __builtin_ctzll(above) : kWave;  // first point above the eigenvalue
        const double xl = __shfl(x, f > 0 ? f - 1 : 0), xh = __shfl(x, f < kWave ? f : 0);
        lo = f > 0 ? xl : lo;
        hi = f < kWave ? xh : hi;
    }
    if (lane == 0)
        ritz[k] = 0.5 * (lo + hi);
}

Diag diag_of(const OpDev &op)
{
    if (!op.precond)
        return Diag{nullptr, nullptr, 1.0};
    if (op.kind == kOpPoisson)
        return Diag{nullptr, nullptr, 6.0};
    if (op.kind == kOpPoisson27)
        return Diag{nullptr, nullptr, 26.0};
    if (op.kind == kOpFaces)
        return Diag{op.dvec, nullptr, 1.0};
    return Diag{op.dvec, op.invd, 1.0};
}

template <class Op>
hipError_t apply_step(const LzArgs &l, const Op &op, const double *w, double *y, int j, int steps, uint32_t per,
                      hipStream_t st)
{
    hipLaunchKernelGGL((k_lz_apply<Op>), dim3(per * kNumXcd), dim3(kBlock), 0, st, l.ls, w, y, l.part + l.nb, l.part,
                       l.ab, j, steps, l.nb, per, l.n, l.chunk, op);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_lanczos(const LzArgs &l, const OpDev &op, const double *u, int steps, hipStream_t st)
{
    const Diag dg = diag_of(op);
    const uint32_t per = (static_cast<uint32_t>(l.nb) + kNumXcd - 1) / kNumXcd;
    double *const pb = l.part + l.nb;  // partials of the norms; those of alpha are at l.part
    const double *wprev = nullptr, *w = u;
    hipLaunchKernelGGL(k_lz_norm0, dim3(l.nb), dim3(kBlock), 0, st, dg, u, pb, l.n, l.chunk);
    for (int j = 0; j < steps; ++j) {
        double *y = l.v[j % 3];  // w_{j-1} and w_j are in the other two, or u
        hipError_t e;
        if (op.kind == kOpPoisson)
            e = apply_step(l, make_poisson<double>(op), w, y, j, steps, per, st);
        else if (op.kind == kOpPoisson27)
            e = apply_step(l, make_poisson27<double>(op), w, y, j, steps, per, st);
        else if (op.kind == kOpFaces)
            e = apply_step(l, Ops<double>::faces(op), w, y, j, steps, per, st);
        else if (op.ell_slice && ell_keep(op, 8))
            e = apply_step(l, Ops<double>::ell<true>(op), w, y, j, steps, per, st);
        else if (op.ell_slice)
            e = apply_step(l, Ops<double>::ell<false>(op), w, y, j, steps, per, st);
        else
            e = apply_step(l, Ops<double>::csr(op), w, y, j, steps, per, st);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_lz_orth, dim3(per * kNumXcd), dim3(kBlock), 0, st, l.ls, dg, y, w, wprev, l.part, pb,
                           l.ab, j, steps, l.nb, per, l.n, l.chunk);
        wprev = w;
        w = y;
    }
    hipLaunchKernelGGL(k_lz_ritz, dim3(steps), dim3(kBlock), 0, st, l.ls, pb, l.nb, l.ab, steps, l.ab + 2 * steps);
    return hipGetLastError();
}

}  // namespace sstep
