// Batched outer iteration over many stencil systems and right-hand sides:
// residual + basis start, basis step, update and the FP32 scaling pre-pass.
// Each kernel is persistent: a fixed grid walks a table of tiles, and the work
// of pairs whose solve has stopped is skipped.  The Gram and FGS kernels of
// the batched iteration live with the single-system ones (batched_impl.h).
#include "basis_f2.h"
#include "launch.h"

namespace sstep {
namespace {

// (A p)_c of the face operator from the differences of p_c to its neighbours.
// The fused multiply-adds are written out: the single and the two-step basis
// give the same bits whatever else surrounds the expression.
template <typename T>
__device__ __forceinline__ T face_sum(T fw, T dw, T fe, T de, T fs, T ds, T fn, T dn, T fb, T db, T ft, T dt)
{
    T y = __builtin_elementwise_fma(fw, dw, fe * de);
    y = __builtin_elementwise_fma(fs, ds, y);
    y = __builtin_elementwise_fma(fn, dn, y);
    y = __builtin_elementwise_fma(fb, db, y);
    return __builtin_elementwise_fma(ft, dt, y);
}

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
__device__ __forceinline__ void buf_store2(Two<double> v, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U32x4, v), r, off, 0, kNonTemporal);
}
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
__device__ __forceinline__ BandLane band_lane(const BF2Tile &tl, int nx, int ny, int ye0, int ye1)
{
    BandLane l;
    const int t0 = 2 * static_cast<int>(threadIdx.x);
    const int er = t0 / nx;
    l.i0 = t0 - er * nx;
    l.turn = l.i0 + 1 == nx;
    l.i1 = l.turn ? 0 : l.i0 + 1;
    const int e0 = ye0 + er, e1 = l.turn ? e0 + 1 : e0;
    l.dom0 = e0 < ye1, l.dom1 = e1 < ye1;
    l.int0 = l.dom0 && e0 >= tl.y0 && e0 < tl.y1, l.int1 = l.dom1 && e1 >= tl.y0 && e1 < tl.y1;
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

// Two basis steps for one pair per block (Sec. 2, Definition, taken twice):
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
// formed from them by the single step's expression.  Logical blocks take the
// right-hand sides of one band fastest, so the blocks that read the same
// coefficients run together on one XCD and share them through its L2.
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
// to the pair's product slots from slot 2j + 1 (0 when FIRST), one partial
// per band (BSys::mofs).
template <typename T, bool FACES, bool FIRST, int D, bool MOM>
__global__ __launch_bounds__(kBf2Lanes) void k_bbasis_f2(const BGlob *__restrict__ gl, const BSys *__restrict__ sys,
                                                         const BF2Tile *__restrict__ tiles, uint32_t nbl,
                                                         const uint32_t *__restrict__ map,
                                                         const DevState *__restrict__ pairs, int nrhs, int precond,
                                                         int j, T *__restrict__ P, double *__restrict__ mpart, int s)
{
    constexpr uint32_t ES = sizeof(T);
    using V = Two<T>;
    __shared__ T ps[2][kBf2Slots];
    __shared__ T qs[2][kBf2Slots];
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
    const int nx = S.g.nx, ny = S.g.ny, nz = S.g.nz;
    const uint32_t nxy = static_cast<uint32_t>(S.g.nxy);
    const int tid = threadIdx.x;
    if (tid < 2 * (kBf2Slots - kBf2Threads)) {
        const int z = tid / 2 < kBf2Front ? tid / 2 : kBf2Threads + tid / 2;
        ps[tid & 1][z] = T(0);
        qs[tid & 1][z] = T(0);
    }
    // rows of the block: the band and the row on each side of it
    const int ye0 = tl.y0 > 0 ? tl.y0 - 1 : 0;
    const int ye1 = tl.y1 < ny ? tl.y1 + 1 : ny;
    const BandLane l = band_lane(tl, nx, ny, ye0, ye1);
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
    const int k0 = tl.k0, k1 = tl.k1;
    const uint32_t pbytes = nxy * ES;
    const int64_t step = static_cast<int64_t>(nrhs) * S.ld;
    T *const col = P + S.pofs + static_cast<int64_t>(r) * S.ld + static_cast<int64_t>(j) * step;
    const uint32_t cbytes = static_cast<uint32_t>(S.n) * ES;
    const __amdgpu_buffer_rsrc_t rj = make_window(col, cbytes);
    const __amdgpu_buffer_rsrc_t rv = make_window(FIRST ? col : col - step, cbytes);
    const __amdgpu_buffer_rsrc_t rq = make_window(col + step, cbytes);
    const __amdgpu_buffer_rsrc_t r2 = make_window(col + 2 * step, cbytes);
    const T *kxp = nullptr, *kyp = nullptr, *kzp = nullptr;
    if constexpr (FACES) {
        if constexpr (sizeof(T) == 8)
            kxp = reinterpret_cast<const T *>(S.kx), kyp = reinterpret_cast<const T *>(S.ky),
            kzp = reinterpret_cast<const T *>(S.kz);
        else
            kxp = reinterpret_cast<const T *>(S.kx32), kyp = reinterpret_cast<const T *>(S.ky32),
            kzp = reinterpret_cast<const T *>(S.kz32);
    }
    // faces: x-faces (nx + 1 per grid row), y-faces (ny + 1 rows of nx per
    // plane), z-faces (nz + 1 planes)
    const uint32_t xrow = static_cast<uint32_t>(nx + 1);
    const uint32_t xplane = static_cast<uint32_t>(ny) * xrow * ES, yplane = static_cast<uint32_t>(ny + 1) * nx * ES;
    const __amdgpu_buffer_rsrc_t rfx = make_window(kxp, static_cast<uint32_t>(nz) * xplane);
    const __amdgpu_buffer_rsrc_t rfy = make_window(kyp, static_cast<uint32_t>(nz) * yplane);
    const __amdgpu_buffer_rsrc_t rfz = make_window(kzp, (static_cast<uint32_t>(nz) + 1) * pbytes);
    const uint32_t b_fx = l.dom0 ? (l.pl + l.pl / static_cast<uint32_t>(nx)) * ES : kMark;
    const T theta = static_cast<T>(S.theta), sigma = static_cast<T>(S.sigma);
    const T two_theta = T(2) * theta;
    const T minv_c = precond ? T(1) / T(6) : T(1);
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
    const double wd = precond ? 1.0 : 0.0, wc = precond ? 0.0 : 1.0;
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
                const T ra = T(1) / d.a, rb = T(1) / d.b;
                dinv.a = l.dom0 && act ? (precond ? ra : T(1)) : T(0);
                dinv.b = l.dom1 && act ? (precond ? rb : T(1)) : T(0);
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
            buf_store2(q, rq, b_in + so);
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
                buf_store2(p2, r2, b_in + so2);
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
    if constexpr (MOM) {
        const int ns = bmom_slots(s);
        double *out = mpart + S.mofs + (static_cast<int64_t>(r) * ns + (FIRST ? 0 : 2 * j + 1)) * S.nf2q +
                      (static_cast<int32_t>(lb / static_cast<uint32_t>(nrhs)) - S.f2first);
        if constexpr (FIRST) {
            const double v[5] = {m0, m1, m2, m3, m4};
            block_partials<5, kBf2Lanes>(v, out, S.nf2q);
        } else {
            const double v[4] = {m1, m2, m3, m4};
            block_partials<4, kBf2Lanes>(v, out, S.nf2q);
        }
    }
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
    const BandLane l = band_lane(tl, nx, ny, ye0, ye1);
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
                d.a = 1.0 / (((((fw.a + fe.a) + fs.a) + fn.a) + fb.a) + ft.a);
                d.b = 1.0 / (((((fw.b + fe.b) + fs.b) + fn.b) + fb.b) + ft.b);
                d = {precond ? d.a : 1.0, precond ? d.b : 1.0};
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

// x += P alpha for every pair whose solve continues.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_bupdate(const BGlob *__restrict__ gl, const BSys *__restrict__ sys,
                                                    const BTile *__restrict__ tiles, int ntiles,
                                                    const DevState *__restrict__ pairs, int nrhs, int s,
                                                    const T *__restrict__ P)
{
    if (gl->ndone == gl->npairs)
        return;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const BTile tl = tiles[t];
        const BSys &S = sys[tl.q];
        const int64_t beg = static_cast<int64_t>(tl.chunk) * S.gchunk;
        const int64_t end = beg + S.gchunk < S.n ? beg + S.gchunk : S.n;
        for (int r = 0; r < nrhs; ++r) {
            const DevState &ps = pairs[S.pair0 + r];
            if (ps.done)
                continue;
            double *__restrict__ x = ps.x;
            const T *Pr = P + S.pofs + static_cast<int64_t>(r) * S.ld;
            const int64_t step = static_cast<int64_t>(nrhs) * S.ld;
            for (int64_t c = beg + threadIdx.x; c < end; c += kBlock) {
                // P is read once: non-temporal loads, eight columns in flight
                // at a time, summed in column order
                double acc = 0.0;
                int i = 0;
                for (; i + 8 <= s; i += 8) {
                    T v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        v[u] = __builtin_nontemporal_load(Pr + (i + u) * step + c);
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        acc += static_cast<double>(v[u]) * ps.alpha[i + u];
                }
                for (; i < s; ++i)
                    acc += static_cast<double>(__builtin_nontemporal_load(Pr + i * step + c)) * ps.alpha[i];
                x[c] += acc;
            }
        }
    }
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
    if (a.fp32)
        hipLaunchKernelGGL(k_bupdate<float>, dim3(a.grid_bt), dim3(kBlock), 0, st, a.gl, a.sys, a.btiles, a.nbt,
                           a.pairs, a.nrhs, a.s, static_cast<const float *>(a.P));
    else
        hipLaunchKernelGGL(k_bupdate<double>, dim3(a.grid_bt), dim3(kBlock), 0, st, a.gl, a.sys, a.btiles, a.nbt,
                           a.pairs, a.nrhs, a.s, static_cast<const double *>(a.P));
    return hipGetLastError();
}

}  // namespace sstep
