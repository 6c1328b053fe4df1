// Batched outer iteration over many stencil systems and right-hand sides:
// residual + basis start, basis step, update and the FP32 scaling pre-pass.
// The residual over chunk tiles, the single basis step and the Gram reduction are
// persistent, a fixed grid walking a table of tiles; the two-step basis and its
// residual take a block per band and right-hand side, the update one per 256 points
// of a pair.  The work of pairs whose solve has stopped is skipped.  The Gram and
// FGS kernels of the batched iteration live with the single-system ones
// (batched_impl.h).
#include "band_f2.h"
#include "grid_limits.h"
#include "launch.h"

namespace sstep {
namespace {

// Stencil at one point of one system, its face coefficients loaded once and
// reused for every right-hand side.
template <typename T, bool FACES>
struct PointStencil {
    int64_t c, nx, nxy;
    bool hw, he, hs, hn, hb, ht;
    T fw, fe, fs, fn, fb, ft, dinv;

    __device__ __forceinline__ void init(const BSys &S, int64_t cc, int precond, const T *kx, const T *ky,
                                         const T *kz)
    {
        c = cc;
        nx = S.g.nx;
        nxy = S.g.nxy;
        const uint32_t q = fdiv(static_cast<uint32_t>(c), S.g.dx);
        const uint32_t i = static_cast<uint32_t>(c) - q * S.g.nx;
        const uint32_t k = fdiv(q, S.g.dy);
        const uint32_t j = q - k * S.g.ny;
        hw = i > 0, he = i + 1 < static_cast<uint32_t>(S.g.nx);
        hs = j > 0, hn = j + 1 < static_cast<uint32_t>(S.g.ny);
        hb = k > 0, ht = k + 1 < static_cast<uint32_t>(S.g.nz);
        if constexpr (FACES) {
            const int64_t fx = c + q, fy = c + static_cast<int64_t>(k) * S.g.nx;
            fw = kx[fx], fe = kx[fx + 1], fs = ky[fy], fn = ky[fy + S.g.nx], fb = kz[c], ft = kz[c + S.g.nxy];
            dinv = precond ? T(1) / (((((fw + fe) + fs) + fn) + fb) + ft) : T(1);
        } else {
            dinv = precond ? T(1) / T(6) : T(1);
        }
    }

    __device__ __forceinline__ T apply(const T *__restrict__ p, T &pc) const
    {
        pc = p[c];
        const T w = hw ? p[c - 1] : T(0), e = he ? p[c + 1] : T(0);
        const T s = hs ? p[c - nx] : T(0), n = hn ? p[c + nx] : T(0);
        const T b = hb ? p[c - nxy] : T(0), t = ht ? p[c + nxy] : T(0);
        if constexpr (FACES)
            return face_sum(fw, pc - w, fe, pc - e, fs, pc - s, fn, pc - n, fb, pc - b, ft, pc - t);
        else
            return T(6) * pc - (((((w + e) + s) + n) + b) + t);
    }
};

template <typename T>
__device__ __forceinline__ T block_sum(T v)
{
    __shared__ T part[kBlock / kWave];
    v = wave_sum(v);
    if (threadIdx.x % kWave == 0)
        part[threadIdx.x / kWave] = v;
    __syncthreads();
    T acc = part[0];
#pragma unroll
    for (int q = 1; q < kBlock / kWave; ++q)
        acc += part[q];
    __syncthreads();
    return acc;
}

// r = b - A x (FP64) per pair over a chunk, ||r||^2 partial per (pair, chunk),
// p_0 = p0scale * (M^{-1} r or r) as column 0 of the pair's basis.  The
// right-hand sides go in groups of kRhsGroup: a point's coefficients are
// loaded once for the group, and each pair's partial is summed in the same
// order as one pair at a time would.
constexpr int kRhsGroup = 8;
template <typename TP, bool FACES>
__global__ __launch_bounds__(kBlock) void k_bresidual(const BGlob *__restrict__ gl, const BSys *__restrict__ sys,
                                                      const BTile *__restrict__ tiles, int ntiles,
                                                      const DevState *__restrict__ pairs, int nrhs, int precond,
                                                      int p0_mode, int write_p0, TP *__restrict__ P,
                                                      double *__restrict__ rpart)
{
    if (gl->ndone == gl->npairs)
        return;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const BTile tl = tiles[t];
        const BSys &S = sys[tl.q];
        const int64_t beg = static_cast<int64_t>(tl.chunk) * S.gchunk;
        const int64_t end = beg + S.gchunk < S.n ? beg + S.gchunk : S.n;
        for (int r0 = 0; r0 < nrhs; r0 += kRhsGroup) {
            bool act[kRhsGroup];
            bool any = false;
#pragma unroll
            for (int u = 0; u < kRhsGroup; ++u) {
                act[u] = r0 + u < nrhs && !pairs[S.pair0 + r0 + u].done;
                any = any || act[u];
            }
            if (!any)
                continue;  // the same for the whole block
            double acc[kRhsGroup];
#pragma unroll
            for (int u = 0; u < kRhsGroup; ++u)
                acc[u] = 0.0;
            for (int64_t c = beg + threadIdx.x; c < end; c += kBlock) {
                PointStencil<double, FACES> op;
                op.init(S, c, precond, S.kx, S.ky, S.kz);
#pragma unroll
                for (int u = 0; u < kRhsGroup; ++u) {
                    if (!act[u])
                        continue;
                    const DevState &ps = pairs[S.pair0 + r0 + u];
                    double pc;
                    const double rr = ps.b[c] - op.apply(ps.x, pc);
                    acc[u] += rr * rr;
                    if (write_p0)
                        P[S.pofs + static_cast<int64_t>(r0 + u) * S.ld + c] =
                            static_cast<TP>(ps.p0scale * (p0_mode ? rr : op.dinv * rr));
                }
            }
#pragma unroll
            for (int u = 0; u < kRhsGroup; ++u) {
                if (!act[u])
                    continue;  // act is the same in every thread
                const double sum = block_sum(acc[u]);
                if (threadIdx.x == 0)
                    rpart[S.rofs + static_cast<int64_t>(r0 + u) * S.nch + tl.chunk] = sum;
            }
        }
    }
}

// FP32+IR pre-pass: p0scale of each pair from its residual partials.
__global__ __launch_bounds__(kBlock) void k_bp0scale(const BSys *__restrict__ sys, DevState *__restrict__ pairs,
                                                     int npairs, int nrhs, const double *__restrict__ rpart)
{
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= npairs || pairs[p].done)
        return;
    const BSys &S = sys[p / nrhs];
    const int r = p % nrhs;
    double acc = 0.0;
    for (int q = 0; q < S.nch; ++q)
        acc += rpart[S.rofs + static_cast<int64_t>(r) * S.nch + q];
    const double rms = sqrt(acc) * S.inv_sqrt_n;
    pairs[p].p0scale = (rms > 0.0 && isfinite(rms)) ? ldexp(1.0, -ilogb(rms)) : 1.0;
}

// Basis step j for every active pair (Sec. 2, Definition): y = A p_j -> AP
// (when AP is kept), p_{j+1} from the three-term recurrence.
template <typename T, bool FACES, int STEP>
__global__ __launch_bounds__(kBlock) void k_bbasis(const BGlob *__restrict__ gl, const BSys *__restrict__ sys,
                                                   const PTile *__restrict__ tiles, int ntiles,
                                                   const DevState *__restrict__ pairs, int nrhs, int precond, int j,
                                                   T *__restrict__ P, T *__restrict__ AP)
{
    if (gl->ndone == gl->npairs)
        return;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const PTile tl = tiles[t];
        const BSys &S = sys[tl.q];
        const int64_t c = static_cast<int64_t>(tl.blk) * kBlock + threadIdx.x;
        if (c >= S.n)
            continue;
        const T *kx = nullptr, *ky = nullptr, *kz = nullptr;
        if constexpr (FACES) {
            if constexpr (sizeof(T) == 8)
                kx = reinterpret_cast<const T *>(S.kx), ky = reinterpret_cast<const T *>(S.ky),
                kz = reinterpret_cast<const T *>(S.kz);
            else
                kx = reinterpret_cast<const T *>(S.kx32), ky = reinterpret_cast<const T *>(S.ky32),
                kz = reinterpret_cast<const T *>(S.kz32);
        }
        PointStencil<T, FACES> op;
        op.init(S, c, precond, kx, ky, kz);
        const T theta = static_cast<T>(S.theta), sigma = static_cast<T>(S.sigma);
        const int64_t step = static_cast<int64_t>(nrhs) * S.ld;
        // Right-hand sides in groups of kRg: every load of a group is issued
        // before its stores (P is read and written through one pointer, so
        // the compiler keeps loads after earlier stores).
        constexpr int kRg = 4;
        for (int r0 = 0; r0 < nrhs; r0 += kRg) {
            T y[kRg], pc[kRg], pp[kRg];
            bool act[kRg];
#pragma unroll
            for (int u = 0; u < kRg; ++u) {
                const int r = r0 + u;
                act[u] = r < nrhs && !pairs[S.pair0 + r].done;
                y[u] = pc[u] = pp[u] = T(0);
                if (act[u]) {
                    const int64_t col = S.pofs + (static_cast<int64_t>(j) * nrhs + r) * S.ld;
                    y[u] = op.apply(P + col, pc[u]);
                    if constexpr (STEP == 1)
                        pp[u] = P[col - step + c];
                }
            }
#pragma unroll
            for (int u = 0; u < kRg; ++u) {
                if (!act[u])
                    continue;
                const int64_t col = S.pofs + (static_cast<int64_t>(j) * nrhs + r0 + u) * S.ld;
                if (AP)  // not kept by the recurrence Gram kind
                    __builtin_nontemporal_store(y[u], AP + col + c);
                if constexpr (STEP == 0) {
                    P[col + step + c] = theta * (op.dinv * y[u] - sigma * pc[u]);
                } else if constexpr (STEP == 1) {
                    const T two_theta = T(2) * theta;
                    P[col + step + c] = two_theta * (op.dinv * y[u] - sigma * pc[u]) - pp[u];
                }
            }
        }
    }
}

// Two basis steps (band_pair) for one pair per block.  Logical blocks take the
// right-hand sides of one band fastest, so the blocks that read the same
// coefficients run together on one XCD and share them through its L2.
// MOM: the products go to the pair's slots from slot 2j + 1 (0 when FIRST),
// one partial per band (BSys::mofs).
template <typename T, bool FACES, bool FIRST, int D, bool MOM>
__global__ __launch_bounds__(kBf2Lanes) void k_bbasis_f2(const BGlob *__restrict__ gl, const BSys *__restrict__ sys,
                                                         const BF2Tile *__restrict__ tiles, uint32_t nbl,
                                                         const uint32_t *__restrict__ map,
                                                         const DevState *__restrict__ pairs, int nrhs, int precond,
                                                         int j, T *__restrict__ P, double *__restrict__ mpart, int s)
{
    if (gl->ndone == gl->npairs)
        return;
    const uint32_t lb = map[blockIdx.x];
    if (lb >= nbl)
        return;  // whole block: no barrier is skipped by part of it
    const BF2Tile tl = tiles[lb / static_cast<uint32_t>(nrhs)];
    const int r = static_cast<int>(lb % static_cast<uint32_t>(nrhs));
    const BSys &S = sys[tl.q];
    if (pairs[S.pair0 + r].done)
        return;
    const int64_t step = static_cast<int64_t>(nrhs) * S.ld;
    T *const col = P + S.pofs + static_cast<int64_t>(r) * S.ld + static_cast<int64_t>(j) * step;
    BandArgs<T> a{S.g.nx, S.g.ny, S.g.nz, precond, static_cast<T>(S.theta), static_cast<T>(S.sigma),
                  nullptr, nullptr, nullptr, col, FIRST ? col : col - step, col + step, col + 2 * step};
    if constexpr (FACES && sizeof(T) == 8)
        a.kx = reinterpret_cast<const T *>(S.kx), a.ky = reinterpret_cast<const T *>(S.ky),
        a.kz = reinterpret_cast<const T *>(S.kz);
    else if constexpr (FACES)
        a.kx = reinterpret_cast<const T *>(S.kx32), a.ky = reinterpret_cast<const T *>(S.ky32),
        a.kz = reinterpret_cast<const T *>(S.kz32);
    double *out = nullptr;
    if constexpr (MOM)
        out = mpart + S.mofs + (static_cast<int64_t>(r) * bmom_slots(s) + (FIRST ? 0 : 2 * j + 1)) * S.nf2q +
              (static_cast<int32_t>(lb / static_cast<uint32_t>(nrhs)) - S.f2first);
    band_pair<T, FACES, FIRST, D, MOM, false>(a, tl.y0, tl.y1, tl.k0, tl.k1, out, S.nf2q);
}

// Residual over the two-step basis's band table (FP64 arithmetic; p_0 stored
// in TP): on the band's rows of one right-hand side, r = b - A x, p_0 =
// p0scale M^{-1} r (p0scale r with p0_mode 1), and the band's partial of
// ||r||^2 in slot `slot` of the pair's `slots` band partials.  The block
// marches its range of planes as the two-step basis does, two points a lane:
// x of the current plane (the band's rows and the row on each side) sits in
// LDS, double-buffered with one barrier per plane, the planes below and above
// in registers, so each range reads x once (plus one plane on each side), and
// the loads of a plane run two planes ahead.  The operator expression and the
// Jacobi weight are PointStencil's, as in k_bresidual.  A buffer window is one
// plane, empty where the plane does not exist (the FP64 vectors of an FP32
// batch may exceed the basis's 1 GiB).
//
// 20 systems of 32^3 to 96^3, 8 right-hand sides, FP64: 520 -> 361 us a launch
// (1.25 GB of vectors, 3.5 TB/s); 12 systems of 9^3 to 33^3, 3 right-hand
// sides, FP32+IR: 25.6 -> 16.0.
constexpr uint32_t kNoPoint = 0xF0000000u;  // past every window of a plane
template <typename TP, bool FACES>
__global__ __launch_bounds__(kBf2Lanes, 4) void k_bres_f2(const BGlob *__restrict__ gl, const BSys *__restrict__ sys,
                                                       const BF2Tile *__restrict__ tiles, uint32_t nbl,
                                                       const uint32_t *__restrict__ map,
                                                       const DevState *__restrict__ pairs, int nrhs, int precond,
                                                       int p0_mode, TP *__restrict__ P, double *__restrict__ mpart,
                                                       int slots, int slot)
{
    using V = Two<double>;
    constexpr uint32_t ES = sizeof(double);
    __shared__ double xs[2][kBf2Slots];
    if (gl->ndone == gl->npairs)
        return;
    const uint32_t lb = map[blockIdx.x];
    if (lb >= nbl)
        return;  // whole block: no barrier is skipped by part of it
    const BF2Tile tl = tiles[lb / static_cast<uint32_t>(nrhs)];
    const int r = static_cast<int>(lb % static_cast<uint32_t>(nrhs));
    const BSys &S = sys[tl.q];
    const DevState &st = pairs[S.pair0 + r];
    if (st.done)
        return;
    const int nx = S.g.nx, ny = S.g.ny, nz = S.g.nz;
    const int64_t nxy = S.g.nxy;
    const int tid = threadIdx.x;
    if (tid < 2 * (kBf2Slots - kBf2Threads))
        xs[tid & 1][tid / 2 < kBf2Front ? tid / 2 : kBf2Threads + tid / 2] = 0.0;
    const int ye0 = tl.y0 > 0 ? tl.y0 - 1 : 0;
    const int ye1 = tl.y1 < ny ? tl.y1 + 1 : ny;
    const BandLane l = band_lane(nx, tl.y0, tl.y1, ye0, ye1);
    const int own = kBf2Front + 2 * tid;  // LDS slot of the first point
    const bool lone = l.int0 != l.int1;   // one point of the lane is stored
    const bool lone_wave = __ballot(lone) != 0;
    const uint32_t o_pt = l.dom0 ? l.pl * ES : kNoPoint, o_fx = l.dom0 ? (l.pl + l.pl / nx) * ES : kNoPoint;
    const uint32_t o_fn = l.dom0 ? (l.pl + nx) * ES : kNoPoint;
    const uint32_t o_in = l.int0 && l.int1 ? l.pl * sizeof(TP) : kNoPoint;
    const uint32_t o_ln = lone ? (l.int0 ? l.pl : l.pl + 1) * sizeof(TP) : kNoPoint;
    const double *__restrict__ x = st.x;
    const double *__restrict__ b = st.b;
    const double scale = st.p0scale;
    TP *__restrict__ p0 = P + S.pofs + static_cast<int64_t>(r) * S.ld;
    const double dconst = precond ? 1.0 / 6.0 : 1.0;
    const int k0 = tl.k0, k1 = tl.k1;
    // plane k of an array with w entries per plane; no entries when !in
    auto win = [](const auto *base, int64_t w, int k, bool in) {
        return make_window(base + static_cast<int64_t>(k) * w, in ? static_cast<uint32_t>(w * sizeof(*base)) : 0u);
    };
    auto in_rows = [&](V v) -> V { return {v.a, l.dom1 ? v.b : 0.0}; };  // the second point may lie past the rows
    auto load_x = [&](int k) -> V { return in_rows(buf_load2(0.0, win(x, nxy, k, k >= 0 && k < nz), o_pt)); };
    // slot u holds, for plane k = k0 + u (mod D): x on plane k + 1, b and the faces of plane k
    constexpr int D = 2, kU = 6;
    V xt[D], bc[D], fxa[D], fxb[D], fss[D], fns[D], fts[D];
    auto refill = [&](int u, int k) {
        const bool in = k < k1;
        xt[u] = buf_load2(0.0, win(x, nxy, k + 1, in && k + 1 < nz), o_pt);
        bc[u] = buf_load2(0.0, win(b, nxy, k, in), o_pt);
        if constexpr (FACES) {
            const __amdgpu_buffer_rsrc_t rx = win(S.kx, static_cast<int64_t>(ny) * (nx + 1), k, in);
            const __amdgpu_buffer_rsrc_t ry = win(S.ky, static_cast<int64_t>(ny + 1) * nx, k, in);
            fxa[u] = buf_load2(0.0, rx, o_fx);
            fxb[u] = buf_load2(0.0, rx, o_fx + 2 * ES);
            fss[u] = buf_load2(0.0, ry, o_pt);
            fns[u] = buf_load2(0.0, ry, o_fn);
            fts[u] = buf_load2(0.0, win(S.kz, nxy, k + 1, in), o_pt);
        }
    };
    V xb = load_x(k0 - 1), xc = load_x(k0);
    V fb{0.0, 0.0};
    if constexpr (FACES)
        fb = buf_load2(0.0, win(S.kz, nxy, k0, true), o_pt);
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < D; ++u)
        refill(u, k0 + u);
    for (int k = k0;;) {
#pragma unroll
        for (int v = 0; v < kU; ++v) {
            const int u = v % D;
            double *buf = xs[v & 1];
            const V xa = in_rows(xt[u]), bb = bc[u];
            V fw{}, fe{}, fs{}, fn{}, ft{};
            if constexpr (FACES) {
                fw = {fxa[u].a, l.turn ? fxb[u].a : fxa[u].b};
                fe = {fxa[u].b, l.turn ? fxb[u].b : fxb[u].a};
                fs = fss[u], fn = fns[u], ft = fts[u];
            }
            buf[own] = xc.a, buf[own + 1] = xc.b;
            lds_barrier();
            const double w0 = buf[l.iw], e1 = buf[l.ie];
            const double e0 = l.turn ? 0.0 : xc.b, w1 = l.turn ? 0.0 : xc.a;
            const double s0 = buf[l.is], s1 = buf[l.is + 1], n0 = buf[l.in], n1 = buf[l.in + 1];
            refill(u, k + D);
            V ax, d{dconst, dconst};
            if constexpr (FACES) {
                ax.a = face_sum(fw.a, xc.a - w0, fe.a, xc.a - e0, fs.a, xc.a - s0, fn.a, xc.a - n0, fb.a,
                                xc.a - xb.a, ft.a, xc.a - xa.a);
                ax.b = face_sum(fw.b, xc.b - w1, fe.b, xc.b - e1, fs.b, xc.b - s1, fn.b, xc.b - n1, fb.b,
                                xc.b - xb.b, ft.b, xc.b - xa.b);
                d.a = ((((fw.a + fe.a) + fs.a) + fn.a) + fb.a) + ft.a;
                d.b = ((((fw.b + fe.b) + fs.b) + fn.b) + fb.b) + ft.b;
                d = {precond ? d.a : 1.0, precond ? d.b : 1.0};
                d = {1.0 / d.a, 1.0 / d.b};
            } else {
                ax.a = 6.0 * xc.a - (((((w0 + e0) + s0) + n0) + xb.a) + xa.a);
                ax.b = 6.0 * xc.b - (((((w1 + e1) + s1) + n1) + xb.b) + xa.b);
            }
            V rr{bb.a - ax.a, bb.b - ax.b};
            const TP pa = static_cast<TP>(scale * (p0_mode ? rr.a : d.a * rr.a));
            const TP pb = static_cast<TP>(scale * (p0_mode ? rr.b : d.b * rr.b));
            const __amdgpu_buffer_rsrc_t rp = win(p0, nxy, k, true);
            buf_store2(Two<TP>{pa, pb}, rp, o_in);
            if (lone_wave)
                buf_store_out(l.int0 ? pa : pb, rp, o_ln);
            rr = {l.int0 ? rr.a : 0.0, l.int1 ? rr.b : 0.0};
            acc += rr.a * rr.a;
            acc += rr.b * rr.b;
            xb = xc;
            xc = xa;
            fb = ft;
            if (++k == k1)
                goto done;
        }
    }
done:
    const double v[1] = {acc};
    block_partials<1, kBf2Lanes>(v,
                                 mpart + S.mofs + (static_cast<int64_t>(r) * slots + slot) * S.nf2q +
                                     (static_cast<int32_t>(lb / static_cast<uint32_t>(nrhs)) - S.f2first),
                                 S.nf2q);
}

// acc = sum_i alpha_i p_i at one point: P is read once, non-temporal loads,
// eight columns in flight at a time, summed in column order.
template <typename T>
__device__ __forceinline__ double basis_sum(const T *__restrict__ Pr, int64_t step, int64_t c, int s,
                                            const double *__restrict__ alpha)
{
    double acc = 0.0;
    int i = 0;
    for (; i + 8 <= s; i += 8) {
        T v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = __builtin_nontemporal_load(Pr + (i + u) * step + c);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            acc += static_cast<double>(v[u]) * alpha[i + u];
    }
    for (; i < s; ++i)
        acc += static_cast<double>(__builtin_nontemporal_load(Pr + i * step + c)) * alpha[i];
    return acc;
}

// x += P alpha for every pair whose solve continues: a block per kBlock points
// of one pair, right-hand side after right-hand side, from block first on (a batch
// of more than kBlocksPerLaunch takes several launches).  HBM-bound: 20 systems of
// 32^3 to 96^3, 8 right-hand sides, s = 16, FP64: 1440 us with chunk tiles of
// 2048 rows or more that walk the right-hand sides, 1370 (5.6 TB/s) with these;
// 12 systems of 9^3 to 33^3, 3 right-hand sides, FP32+IR, whose 70 tiles left
// most CUs idle: 25.3 -> 6.2 us.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_bupdate(const BGlob *__restrict__ gl, const BSys *__restrict__ sys,
                                                    const PTile *__restrict__ tiles, uint32_t ntiles,
                                                    const DevState *__restrict__ pairs, int nrhs, int s,
                                                    const T *__restrict__ P, uint32_t first)
{
    if (gl->ndone == gl->npairs)
        return;
    const uint32_t lb = first + blockIdx.x, r = lb / ntiles;
    const PTile tl = tiles[lb - r * ntiles];
    const BSys &S = sys[tl.q];
    const DevState &ps = pairs[S.pair0 + r];
    const int64_t c = static_cast<int64_t>(tl.blk) * kBlock + threadIdx.x;
    if (ps.done || c >= S.n)
        return;
    ps.x[c] += basis_sum(P + S.pofs + static_cast<int64_t>(r) * S.ld, static_cast<int64_t>(nrhs) * S.ld, c, s,
                         ps.alpha);
}

}  // namespace

hipError_t launch_bresidual(const BatchArgs &a, hipStream_t st, bool write_p0)
{
    const int w = write_p0 ? 1 : 0;
    if (a.fp32) {
        if (a.faces)
            hipLaunchKernelGGL((k_bresidual<float, true>), dim3(a.grid_bt), dim3(kBlock), 0, st, a.gl, a.sys,
                               a.btiles, a.nbt, a.pairs, a.nrhs, a.precond, a.p0_mode, w,
                               static_cast<float *>(a.P), a.rpart);
        else
            hipLaunchKernelGGL((k_bresidual<float, false>), dim3(a.grid_bt), dim3(kBlock), 0, st, a.gl, a.sys,
                               a.btiles, a.nbt, a.pairs, a.nrhs, a.precond, a.p0_mode, w,
                               static_cast<float *>(a.P), a.rpart);
    } else {
        if (a.faces)
            hipLaunchKernelGGL((k_bresidual<double, true>), dim3(a.grid_bt), dim3(kBlock), 0, st, a.gl, a.sys,
                               a.btiles, a.nbt, a.pairs, a.nrhs, a.precond, a.p0_mode, w,
                               static_cast<double *>(a.P), a.rpart);
        else
            hipLaunchKernelGGL((k_bresidual<double, false>), dim3(a.grid_bt), dim3(kBlock), 0, st, a.gl, a.sys,
                               a.btiles, a.nbt, a.pairs, a.nrhs, a.precond, a.p0_mode, w,
                               static_cast<double *>(a.P), a.rpart);
    }
    return hipGetLastError();
}

hipError_t launch_bp0scale(const BatchArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(k_bp0scale, dim3((a.npairs + kBlock - 1) / kBlock), dim3(kBlock), 0, st, a.sys, a.pairs,
                       a.npairs, a.nrhs, a.rpart);
    return hipGetLastError();
}

namespace {
template <typename T, bool FACES>
hipError_t bbasis_t(const BatchArgs &a, int j, hipStream_t st)
{
    T *P = static_cast<T *>(a.P), *AP = static_cast<T *>(a.AP);
    if (j + 1 >= a.s && !a.rec)  // the last step forms A p_{s-1} only, unless p_s is kept
        hipLaunchKernelGGL((k_bbasis<T, FACES, 2>), dim3(a.grid_pt), dim3(kBlock), 0, st, a.gl, a.sys, a.ptiles,
                           a.npt, a.pairs, a.nrhs, a.precond, j, P, AP);
    else if (j == 0)
        hipLaunchKernelGGL((k_bbasis<T, FACES, 0>), dim3(a.grid_pt), dim3(kBlock), 0, st, a.gl, a.sys, a.ptiles,
                           a.npt, a.pairs, a.nrhs, a.precond, j, P, AP);
    else
        hipLaunchKernelGGL((k_bbasis<T, FACES, 1>), dim3(a.grid_pt), dim3(kBlock), 0, st, a.gl, a.sys, a.ptiles,
                           a.npt, a.pairs, a.nrhs, a.precond, j, P, AP);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_bbasis(const BatchArgs &a, int j, hipStream_t st)
{
    if (a.fp32)
        return a.faces ? bbasis_t<float, true>(a, j, st) : bbasis_t<float, false>(a, j, st);
    return a.faces ? bbasis_t<double, true>(a, j, st) : bbasis_t<double, false>(a, j, st);
}

namespace {
template <typename T, bool FACES, int D, bool MOM>
hipError_t bbasis_pair_v(const BatchArgs &a, int j, hipStream_t st)
{
    const dim3 grid(a.f2grid);
    const uint32_t nbl = static_cast<uint32_t>(a.nf2) * static_cast<uint32_t>(a.nrhs);
    T *P = static_cast<T *>(a.P);
    if (j == 0)
        hipLaunchKernelGGL((k_bbasis_f2<T, FACES, true, D, MOM>), grid, dim3(kBf2Lanes), 0, st, a.gl, a.sys,
                           a.f2tiles, nbl, a.f2map, a.pairs, a.nrhs, a.precond, j, P, a.mpart, a.s);
    else
        hipLaunchKernelGGL((k_bbasis_f2<T, FACES, false, D, MOM>), grid, dim3(kBf2Lanes), 0, st, a.gl, a.sys,
                           a.f2tiles, nbl, a.f2map, a.pairs, a.nrhs, a.precond, j, P, a.mpart, a.s);
    return hipGetLastError();
}
// D: planes of loads in flight.
template <typename T, bool FACES>
hipError_t bbasis_pair_t(const BatchArgs &a, int j, hipStream_t st)
{
    constexpr int D = 2;
    return a.mom ? bbasis_pair_v<T, FACES, D, true>(a, j, st) : bbasis_pair_v<T, FACES, D, false>(a, j, st);
}
}  // namespace

namespace {
template <typename TP, bool FACES>
hipError_t bres_f2_t(const BatchArgs &a, hipStream_t st)
{
    const uint32_t nbl = static_cast<uint32_t>(a.nf2) * static_cast<uint32_t>(a.nrhs);
    hipLaunchKernelGGL((k_bres_f2<TP, FACES>), dim3(a.f2grid), dim3(kBf2Lanes), 0, st, a.gl, a.sys, a.f2tiles,
                       nbl, a.f2map, a.pairs, a.nrhs, a.precond, a.p0_mode, static_cast<TP *>(a.P), a.mpart,
                       a.bres_slots, a.bres_slot);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_bres_f2(const BatchArgs &a, hipStream_t st)
{
    if (!a.f2 || !a.bres)
        return hipErrorInvalidValue;  // only over a band table with its partial slots
    if (a.fp32)
        return a.faces ? bres_f2_t<float, true>(a, st) : bres_f2_t<float, false>(a, st);
    return a.faces ? bres_f2_t<double, true>(a, st) : bres_f2_t<double, false>(a, st);
}

// Steps j and j + 1 of every active pair's basis (recurrence Gram kind, the
// band table built on the host).
hipError_t launch_bbasis_pair(const BatchArgs &a, int j, hipStream_t st)
{
    if (!a.f2 || j < 0 || j + 2 > a.s)
        return hipErrorInvalidValue;
    if (a.fp32)
        return a.faces ? bbasis_pair_t<float, true>(a, j, st) : bbasis_pair_t<float, false>(a, j, st);
    return a.faces ? bbasis_pair_t<double, true>(a, j, st) : bbasis_pair_t<double, false>(a, j, st);
}

hipError_t launch_bupdate(const BatchArgs &a, hipStream_t st)
{
    const uint32_t npt = static_cast<uint32_t>(a.npt);
    auto part = [&](uint64_t first, uint32_t blocks) -> hipError_t {
        const uint32_t f = static_cast<uint32_t>(first);
        if (a.fp32)
            hipLaunchKernelGGL(k_bupdate<float>, dim3(blocks), dim3(kBlock), 0, st, a.gl, a.sys, a.ptiles, npt,
                               a.pairs, a.nrhs, a.s, static_cast<const float *>(a.P), f);
        else
            hipLaunchKernelGGL(k_bupdate<double>, dim3(blocks), dim3(kBlock), 0, st, a.gl, a.sys, a.ptiles, npt,
                               a.pairs, a.nrhs, a.s, static_cast<const double *>(a.P), f);
        return hipGetLastError();
    };
    return in_launches(static_cast<uint64_t>(npt) * static_cast<uint64_t>(a.nrhs), hipSuccess, part);
}

}  // namespace sstep
