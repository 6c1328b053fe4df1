// Stopping test of the outer iteration (Sec. 8: stop at the first k with
// ||r_k|| < tol ||r_0||, strict, on the true residual), run right after the
// residual kernel and before any basis or Gram work of iteration k.
#pragma once

#include "launch.h"

namespace sstep {

constexpr int kSumThreads = 256;

// What the test decides from rho2 = ||b - A x_k||^2 and the state, with first
// telling whether this is the first residual of a solve.
struct StopResult {
    double rho, rho0, relres;
    int stop, status;
};
__device__ __forceinline__ StopResult stop_decide(const DevState *st, double rho2, int first)
{
    StopResult r;
    r.rho = sqrt(rho2);
    r.rho0 = first ? r.rho : st->rho0;
    r.relres = 0.0;
    r.stop = r.status = 0;
    if (first && r.rho0 == 0.0) {
        r.stop = 1;
    } else if (!isfinite(r.rho)) {
        r.stop = 1;
        r.status = 6;  // SSTEP_E_NONFINITE
        r.relres = r.rho;
    } else {
        r.relres = r.rho / r.rho0;
        if (!st->no_stop) {
            if (r.rho < st->tol * r.rho0)
                r.stop = 1;
            else if (st->iter >= st->max_outer) {
                r.stop = 1;
                r.status = 5;  // SSTEP_E_NOCONV
            }
        }
    }
    return r;
}

// Writes the outcome into the state, rho_k to *dbg_rho (may be NULL) and
// rho_k / rho_0 to hist[k] when k < hist_cap.  One thread.
__device__ __forceinline__ void stop_record(DevState *st, const StopResult &r, double *dbg_rho, double *hist,
                                            int hist_cap)
{
    st->first = 0;
    st->rho0 = r.rho0;
    st->rho = r.rho;
    st->relres = r.relres;
    if (st->iter < hist_cap)
        hist[st->iter] = r.relres;
    if (dbg_rho)
        *dbg_rho = r.rho;
    if (r.stop) {
        st->status = r.status;
        st->done = 1;
    }
}

// One thread.  rho2 = ||b - A x_k||^2.  Records rho_0 on the first call of a
// solve, then stops the solve (done = 1) when rho_k < tol rho_0, at max_outer
// (SSTEP_E_NOCONV) or on a non-finite norm (SSTEP_E_NONFINITE).  A no_stop
// state (single-step and timing entry points) stops only on a zero initial
// or a non-finite norm.  Writes rho_k to *dbg_rho (may be NULL) and
// rho_k / rho_0 to hist[k] when k < hist_cap.  Returns 1 when the solve is
// (now) stopped.
__device__ inline int stop_test(DevState *__restrict__ st, double rho2, double *__restrict__ dbg_rho,
                                double *__restrict__ hist, int hist_cap)
{
    const StopResult r = stop_decide(st, rho2, st->first);
    stop_record(st, r, dbg_rho, hist, hist_cap);
    return r.stop;
}

// Sum of part[0..cnt) in a fixed order by the first kSumThreads threads of a
// block (thread t takes t, t + 256, ..., the waves combine by butterfly and
// the four wave sums are added in order).  Returns the total in thread 0
// (other threads: unspecified).  Every thread of the block must call it.
__device__ inline double fixed_order_sum(const double *part, int cnt)
{
    __shared__ double wsum[kSumThreads / kWave];
    double acc = 0.0;
    if (threadIdx.x < kSumThreads) {
#pragma unroll 4
        for (int q = threadIdx.x; q < cnt; q += kSumThreads)
            acc += part[q];
    }
    acc = wave_sum(acc);
    if (threadIdx.x < kSumThreads && threadIdx.x % kWave == 0)
        wsum[threadIdx.x / kWave] = acc;
    __syncthreads();
    double v = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < kSumThreads / kWave; ++w)
            v += wsum[w];
    return v;
}

// The same test at the head of a launch of NT-thread blocks, in place of one
// of its own: every block sums the partials in the same order and decides for
// itself; the block that record names writes the state.  The others read only
// what no test of this solve changes after the first residual, which is told
// by the iteration count, and st->done, which may be set while they start: done
// is what each wave read, and a block stops as a whole when any of its waves
// read it set (the recording block then takes the same decision).  part_sum: the
// thread's share of the partials (partial_share), of no meaning in a wave whose
// done is set.  Every thread of the block must call it; it returns the same to
// all of them.
struct StopArgs {
    const double *rpart;
    double *dbg_rho, *hist;
    int nbr, hist_cap;
};
// st->done as one value for the wave.
__device__ __forceinline__ int wave_done(const DevState *st) { return __builtin_amdgcn_readfirstlane(st->done); }
template <int NT>
__device__ __forceinline__ double partial_share(const StopArgs &a)
{
    double acc = 0.0;
    for (int q = threadIdx.x; q < a.nbr; q += NT)
        acc += a.rpart[q];
    return acc;
}
template <int NT>
__device__ __forceinline__ int stop_at_head(DevState *st, int done, const StopArgs &a, double part_sum, bool record)
{
    double rho2 = wave_sum(part_sum);
    if constexpr (NT > kWave) {
        __shared__ double wsum[NT / kWave];
        __shared__ int wdone[NT / kWave];
        if (threadIdx.x % kWave == 0) {
            wsum[threadIdx.x / kWave] = rho2;
            wdone[threadIdx.x / kWave] = done;
        }
        __syncthreads();
        rho2 = 0.0;
        for (int w = 0; w < NT / kWave; ++w) {
            rho2 += wsum[w];
            done |= wdone[w];
        }
    }
    if (done)
        return 1;
    const StopResult r = stop_decide(st, rho2, st->iter == 0);
    if (record && threadIdx.x == 0)
        stop_record(st, r, a.dbg_rho, a.hist, a.hist_cap);
    return r.stop;
}

// A pair of a batch has stopped: counted once, by one thread.
__device__ __forceinline__ void pair_stopped(BGlob *gl, const BSys &Q)
{
    atomicAdd(&gl->ndone, 1);
    atomicAdd(&gl->bdone, Q.nbl);
}

}  // namespace sstep
