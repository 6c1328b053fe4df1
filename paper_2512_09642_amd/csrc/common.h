// Shared device-side definitions of the s-step CG library (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sstep {

constexpr int kMaxS = 32;             // largest basis width
constexpr int kMaxE = kMaxS * (kMaxS + 1) / 2 + kMaxS;  // Gram lower triangle + right-hand side
constexpr int kBlock = 256;           // threads per block of the streaming kernels
constexpr int kWave = 64;
constexpr unsigned kNumXcd = 8;       // MI355X: 8 XCDs, each with its own L2

// State of one solve, resident in device memory.  Every kernel of the outer
// iteration reads `done` first and returns at once when it is set, so graph
// replays issued after convergence do no work.
struct DevState {
    const double *b;   // right-hand side of the current solve
    double *x;         // iterate, updated in place
    double tol;        // relative residual tolerance
    double rho0;       // ||b - A x_0||
    double rho;        // ||b - A x_k|| of the last residual
    double relres;     // rho / rho0
    double p0scale;    // power-of-two factor applied to p_0 (FP32+IR); 1 in FP64
    double delta;      // ||ctil - G atil|| / ||ctil|| of the last Gram solve
    double lnorm;      // ||L||_F, L the strictly lower part of the last scaled Gram matrix
    int32_t done;      // 1 once the solve has stopped
    int32_t status;    // sstep_status value
    int32_t iter;      // completed outer updates
    int32_t max_outer;
    int32_t first;     // 1 until rho0 has been recorded
    int32_t no_stop;   // 1 = never stop (single-step and timing entry points)
    int32_t hist_cap;  // capacity of the device history (0 = off)
    int32_t pad;
    double alpha[kMaxS];  // coefficients of the unscaled basis, x += P alpha
};

// Division of 32-bit unsigned n < 2^31 by an invariant divisor d >= 1 with a
// multiply-high and a shift (Granlund & Montgomery, PLDI 1994, round-up
// variant): l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1,
// n / d = (n + mulhi(m, n)) >> l.
struct FastDiv {
    uint32_t d, m, l;
};

inline FastDiv make_fastdiv(uint32_t d)
{
    uint32_t l = 0;
    while ((1ull << l) < d)
        ++l;
    const uint64_t m = ((1ull << 32) * ((1ull << l) - d)) / d + 1;
    return FastDiv{d, static_cast<uint32_t>(m), l};
}

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv &f)
{
    const uint32_t t = __umulhi(f.m, n);
    return static_cast<uint32_t>((static_cast<uint64_t>(t) + n) >> f.l);
}

// Grid of a 3D stencil operator, x fastest.
struct Grid3 {
    int32_t nx, ny, nz;
    int64_t nxy;
    FastDiv dx, dy;
};

// Logical block index that gives each XCD a contiguous range of blocks:
// hardware block b runs on XCD b % 8, so XCD x processes logical blocks
// [x * per, (x + 1) * per) in ascending order and the stencil neighbours of a
// block (one plane away) are mostly resident in that XCD's own L2.
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t per)
{
    return (b % kNumXcd) * per + b / kNumXcd;
}

// A 32-bit register moved between lanes on the vector ALU.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;        // quad_perm 1,0,3,2 / 2,3,0,1
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128;      // rotations within a row of 16 lanes
constexpr int kDppRowNewBcast = 0x150;                 // + l: lane l of each row to its whole row

template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    return __hiloint2double(static_cast<int>(dpp_mov<CTRL>(static_cast<uint32_t>(__double2hiint(v)))),
                            static_cast<int>(dpp_mov<CTRL>(static_cast<uint32_t>(__double2loint(v)))));
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __uint_as_float(dpp_mov<CTRL>(__float_as_uint(v)));
}

// v + its value ROWS / 16 rows of 16 lanes away (ROWS 32: the other half of
// the wave; 16: the other row of the half), in every lane.
template <int ROWS>
__device__ __forceinline__ void swap_rows(uint32_t &a, uint32_t &b)
{
    static_assert(ROWS == 16 || ROWS == 32, "rows exchanged by one instruction");
    const auto r = ROWS == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                              : __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0], b = r[1];
}
// The same for two values at once: a's sums in the first half of the wave (row
// of the half), b's in the second.
template <int ROWS>
__device__ __forceinline__ double add_rows(double a, double b)
{
    uint32_t l0 = static_cast<uint32_t>(__double2loint(a)), l1 = static_cast<uint32_t>(__double2loint(b));
    uint32_t h0 = static_cast<uint32_t>(__double2hiint(a)), h1 = static_cast<uint32_t>(__double2hiint(b));
    swap_rows<ROWS>(l0, l1);
    swap_rows<ROWS>(h0, h1);
    return __hiloint2double(static_cast<int>(h0), static_cast<int>(l0)) +
           __hiloint2double(static_cast<int>(h1), static_cast<int>(l1));
}
template <int ROWS>
__device__ __forceinline__ double add_rows(double v)
{
    return add_rows<ROWS>(v, v);
}
template <int ROWS>
__device__ __forceinline__ float add_rows(float v)
{
    uint32_t a = __float_as_uint(v), b = a;
    swap_rows<ROWS>(a, b);
    return __uint_as_float(a) + __uint_as_float(b);
}

// Butterfly sum over the 64 lanes of a wave (lanes 32 apart, then 16, 8, 4, 2,
// 1); every lane gets the total and the order of the additions is fixed, so
// the result is reproducible.  Formed by lane moves on the vector ALU: the
// same six exchanges through the LDS permute unit take some 600 cycles, which
// a kernel of a few microseconds shows at its end.  (After the step over 8
// lanes a row repeats itself, so a rotation by 4 meets the lane 4 apart.)
template <typename T>
__device__ __forceinline__ T row_sum(T v)
{
    v += dpp<kDppRor8>(v);
    v += dpp<kDppRor4>(v);
    v += dpp<kDppXor2>(v);
    v += dpp<kDppXor1>(v);
    return v;
}
template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
    v = add_rows<32>(v);
    v = add_rows<16>(v);
    return row_sum(v);
}

// Block sums of NV per-thread values in a fixed order (each wave by
// butterfly, then the waves in order); value u goes to out[u * stride].
// Every thread of the block must call it.
template <int NV, int NT>
__device__ __forceinline__ void block_partials(const double (&v)[NV], double *__restrict__ out, int64_t stride)
{
    constexpr int NW = NT / kWave;
    __shared__ double part[NW][NV];
    // up to four values share the steps of the butterfly, a row of lanes each
    // (four values of four waves on a SIMD: 28 additions instead of 96)
    const int lane = threadIdx.x % kWave, row = lane / 16;
#pragma unroll
    for (int u = 0; u < NV; u += 4) {
        double t;
        int at = u;  // the value in the lane's row
        if (NV - u == 1) {
            t = wave_sum(v[u]);
        } else if (NV - u == 2) {
            t = row_sum(add_rows<16>(add_rows<32>(v[u], v[u + 1 < NV ? u + 1 : u])));
            at += row / 2;
        } else {
            const double ab = add_rows<32>(v[u], v[u + 1 < NV ? u + 1 : u]);
            const double c = v[u + 2 < NV ? u + 2 : u];
            const double cd = NV - u > 3 ? add_rows<32>(c, v[u + 3 < NV ? u + 3 : u]) : add_rows<32>(c);
            t = row_sum(add_rows<16>(ab, cd));
            at += row / 2 + row % 2 * 2;  // rows: a, c, b, d
        }
        const bool first = NV - u == 1 ? lane == 0 : NV - u == 2 ? lane % 32 == 0 : lane % 16 == 0;
        if (first && at < NV)
            part[threadIdx.x / kWave][at] = t;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double acc = 0.0;
        for (int w = 0; w < NW; ++w)
            acc += part[w][threadIdx.x];
        out[threadIdx.x * stride] = acc;
    }
}

// ---------------------------------------------------------------------------
// Operators.  apply() returns the centre value p_c, y = (A p)_c and the
// Jacobi factor M^{-1}_cc (1 without preconditioning); apply_w() also the
// weight of the M inner product at c: the diagonal a_cc with Jacobi, 1
// without, and 1 for the constant-coefficient stencils, whose constant
// diagonal the caller applies afterwards.
// ---------------------------------------------------------------------------

// Constant-coefficient 7-point Poisson operator: diagonal 6, off-diagonal -1.
template <typename T>
struct OpPoisson7 {
    Grid3 g;
    T minv;  // 1/6 with Jacobi, 1 without

    __device__ __forceinline__ void apply_w(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv, T &wt) const
    {
        apply(p, c, pc, y, dinv);
        wt = T(1);
    }
    __device__ __forceinline__ void apply(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv) const
    {
        const uint32_t q = fdiv(static_cast<uint32_t>(c), g.dx);  // j + ny*k
        const uint32_t i = static_cast<uint32_t>(c) - q * g.nx;
        const uint32_t k = fdiv(q, g.dy);
        const uint32_t j = q - k * g.ny;
        pc = p[c];
        const T w = i > 0 ? p[c - 1] : T(0);
        const T e = i + 1 < static_cast<uint32_t>(g.nx) ? p[c + 1] : T(0);
        const T s = j > 0 ? p[c - g.nx] : T(0);
        const T n = j + 1 < static_cast<uint32_t>(g.ny) ? p[c + g.nx] : T(0);
        const T b = k > 0 ? p[c - g.nxy] : T(0);
        const T t = k + 1 < static_cast<uint32_t>(g.nz) ? p[c + g.nxy] : T(0);
        y = T(6) * pc - (((((w + e) + s) + n) + b) + t);
        dinv = minv;
    }
};

// Constant-coefficient 27-point operator (Sec. 8): diagonal 26, -1 on the 26
// other points of the 3 x 3 x 3 box, so (A p)_c = 27 p_c - (sum of p over the
// box); neighbours outside the grid are 0.
template <typename T>
struct OpPoisson27 {
    Grid3 g;
    T minv;  // 1/26 with Jacobi, 1 without

    __device__ __forceinline__ void apply_w(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv, T &wt) const
    {
        apply(p, c, pc, y, dinv);
        wt = T(1);
    }
    __device__ __forceinline__ void apply(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv) const
    {
        const uint32_t q = fdiv(static_cast<uint32_t>(c), g.dx);
        const uint32_t i = static_cast<uint32_t>(c) - q * g.nx;
        const uint32_t k = fdiv(q, g.dy);
        const uint32_t j = q - k * g.ny;
        const bool has_w = i > 0, has_e = i + 1 < static_cast<uint32_t>(g.nx);
        const bool has_s = j > 0, has_n = j + 1 < static_cast<uint32_t>(g.ny);
        const bool has_b = k > 0, has_t = k + 1 < static_cast<uint32_t>(g.nz);
        pc = p[c];
        T box = T(0);
#pragma unroll
        for (int dk = -1; dk <= 1; ++dk) {
            if ((dk < 0 && !has_b) || (dk > 0 && !has_t))
                continue;
            T plane = T(0);
#pragma unroll
            for (int dj = -1; dj <= 1; ++dj) {
                if ((dj < 0 && !has_s) || (dj > 0 && !has_n))
                    continue;
                const int64_t r = c + dj * static_cast<int64_t>(g.nx) + dk * g.nxy;
                T row = p[r];
                if (has_w)
                    row += p[r - 1];
                if (has_e)
                    row += p[r + 1];
                plane += row;
            }
            box += plane;
        }
        y = T(27) * pc - box;
        dinv = minv;
    }
};

// (A p)_c of the face operator from the differences of p_c to its neighbours.
// The fused multiply-adds are written out: every kernel gives the same bits,
// whatever else surrounds the expression, the single basis step those of the
// two-step kernels among them.
template <typename T>
__device__ __forceinline__ T face_sum(T fw, T dw, T fe, T de, T fs, T ds, T fn, T dn, T fb, T db, T ft, T dt)
{
    T y = __builtin_elementwise_fma(fw, dw, fe * de);
    y = __builtin_elementwise_fma(fs, ds, y);
    y = __builtin_elementwise_fma(fn, dn, y);
    y = __builtin_elementwise_fma(fb, db, y);
    return __builtin_elementwise_fma(ft, dt, y);
}

// Variable-coefficient 7-point operator from face coefficients (boundary
// faces included): (A p)_c = sum_f k_f (p_c - p_q), p_q = 0 outside.
template <typename T>
struct OpFaces7 {
    Grid3 g;
    const T *__restrict__ kx;
    const T *__restrict__ ky;
    const T *__restrict__ kz;
    int precond;

    __device__ __forceinline__ void apply(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv) const
    {
        T wt;
        apply_w(p, c, pc, y, dinv, wt);
    }
    __device__ __forceinline__ void apply_w(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv, T &wt) const
    {
        const uint32_t q = fdiv(static_cast<uint32_t>(c), g.dx);
        const uint32_t i = static_cast<uint32_t>(c) - q * g.nx;
        const uint32_t k = fdiv(q, g.dy);
        const uint32_t j = q - k * g.ny;
        const int64_t fx = c + q;                          // (k*ny + j)*(nx+1) + i
        const int64_t fy = c + static_cast<int64_t>(k) * g.nx;  // (k*(ny+1) + j)*nx + i
        const T fw = kx[fx], fe = kx[fx + 1];
        const T fs = ky[fy], fn = ky[fy + g.nx];
        const T fb = kz[c], ft = kz[c + g.nxy];
        pc = p[c];
        const T w = i > 0 ? p[c - 1] : T(0);
        const T e = i + 1 < static_cast<uint32_t>(g.nx) ? p[c + 1] : T(0);
        const T s = j > 0 ? p[c - g.nx] : T(0);
        const T n = j + 1 < static_cast<uint32_t>(g.ny) ? p[c + g.nx] : T(0);
        const T b = k > 0 ? p[c - g.nxy] : T(0);
        const T t = k + 1 < static_cast<uint32_t>(g.nz) ? p[c + g.nxy] : T(0);
        y = face_sum(fw, pc - w, fe, pc - e, fs, pc - s, fn, pc - n, fb, pc - b, ft, pc - t);
        const T d = ((((fw + fe) + fs) + fn) + fb) + ft;
        dinv = precond ? T(1) / d : T(1);
        wt = precond ? d : T(1);
    }
};

// General CSR matrix, one row per thread.
template <typename T>
struct OpCsr {
    const int32_t *__restrict__ rp;
    const int32_t *__restrict__ ci;
    const T *__restrict__ val;
    const T *__restrict__ invd;  // M^{-1} diagonal (all ones without preconditioning)

    __device__ __forceinline__ void apply_w(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv, T &wt) const
    {
        apply(p, c, pc, y, dinv);
        wt = T(1) / dinv;
    }
    __device__ __forceinline__ void apply(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv) const
    {
        const int32_t k0 = rp[c], k1 = rp[c + 1];
        T acc = T(0);
        for (int32_t k = k0; k < k1; ++k)
            acc += val[k] * p[ci[k]];
        pc = p[c];
        y = acc;
        dinv = invd[c];
    }
};

// The same CSR operator stored in slices of kEllSlice consecutive rows, one
// wave a slice, values column-major inside the slice, so the lanes of a wave
// read each entry index with one coalesced load.  A row keeps its CSR entries
// in their order, so the sum is formed with the same operations in the same
// order as by OpCsr.  A slice comes in one of two forms:
//  * listed (EllSlice::diag 0): as many entries per row as the longest row of
//    the slice has, each with its column; the padding has column -1 and is
//    skipped;
//  * by offsets (diag 1): the distinct values of column - row in the slice,
//    ascending, each with the bit mask of the rows that have such an entry;
//    no column is stored or read (8 bytes an entry instead of 12), and the
//    addresses of the vector do not wait for a column.  Matrices from grids
//    have few offsets.  Chosen per slice where the offsets times 7 are at
//    most the longest row times 10 (the bytes of both forms are then equal in
//    FP64; rows missing an offset hold a zero there that is not used).
constexpr int kEllSlice = 64;
constexpr int kEllGroup = 8;  // offsets of a slice are padded to a multiple of this

struct EllSlice {
    int64_t val;   // first value (w times kEllSlice follow)
    int64_t pat;   // first column (listed) or first offset and mask
    int32_t w;     // entries per row (listed) or offsets
    int32_t diag;
};

// In FP64 the Jacobi weight is formed from the row's own diagonal entry,
// precond ? 1 / a_cc : 1 (the value the M^{-1} vector holds, to the bit),
// which saves reading that vector; FP32 reads its rounded copy.
//
// Called by the lanes of a wave with consecutive c from a multiple of
// kEllSlice on; a lane past the last row may repeat the last row, and then
// gets a value of no meaning.
template <typename T, bool KEEP>
struct OpEll {
    const EllSlice *__restrict__ slice;
    const int32_t *__restrict__ col;
    const T *__restrict__ val;
    const int32_t *__restrict__ dofs;
    const uint64_t *__restrict__ dmask;
    const T *__restrict__ invd;  // M^{-1} diagonal (all ones without preconditioning); FP32 only
    int32_t n;
    int precond;

    __device__ __forceinline__ void apply(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv) const
    {
        T wt;
        apply_w(p, c, pc, y, dinv, wt);
    }
    // A matrix entry: through the caches (KEEP) or, read once per product,
    // non-temporal.
    template <typename V>
    static __device__ __forceinline__ V entry(const V *q)
    {
        if constexpr (KEEP)
            return *q;
        else
            return __builtin_nontemporal_load(q);
    }
    __device__ __forceinline__ void apply_w(const T *__restrict__ p, int64_t c, T &pc, T &y, T &dinv, T &wt) const
    {
        const int32_t row = static_cast<int32_t>(c);
        const int32_t q = __builtin_amdgcn_readfirstlane(row / kEllSlice);
        const EllSlice S = slice[q];
        const T *__restrict__ v = val + S.val + (row - q * kEllSlice);
        T acc = T(0), diag = T(1);
        constexpr int U = kEllGroup;  // entries whose loads are issued together
        if (S.diag) {
            const int32_t *__restrict__ off = dofs + S.pat;
            const uint64_t *__restrict__ mask = dmask + S.pat;
            // offsets and masks are padded to a multiple of U (mask 0); the
            // values of the padding repeat the last ones
            for (int k0 = 0; k0 < S.w; k0 += U) {
                T a[U], x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int k = k0 + u < S.w ? k0 + u : S.w - 1;
                    a[u] = entry(v + int64_t(k) * kEllSlice);
                    const int32_t j = row + off[k0 + u];
                    x[u] = p[j < 0 ? 0 : (j < n ? j : n - 1)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint64_t m = mask[k0 + u];
                    acc += a[u] * (__builtin_amdgcn_inverse_ballot_w64(m) ? x[u] : T(0));
                    diag = __builtin_amdgcn_inverse_ballot_w64(off[k0 + u] == 0 ? m : 0) ? a[u] : diag;
                }
            }
        } else {
            const int32_t *__restrict__ cp = col + S.pat + (row - q * kEllSlice);
            // the columns and values of the next U entries are in flight while
            // the vector's entries of these are (30011 random rows of 46: 18.8
            // -> 15 us; 16 entries at a time take registers from the other form)
            int32_t j[U];
            T a[U];
            auto fetch = [&](int k0, int32_t(&jj)[U], T(&aa)[U]) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    jj[u] = -1;
                    aa[u] = T(0);
                    if (k0 + u < S.w) {
                        jj[u] = entry(cp + int64_t(k0 + u) * kEllSlice);
                        aa[u] = entry(v + int64_t(k0 + u) * kEllSlice);
                    }
                }
            };
            fetch(0, j, a);
            for (int k0 = 0; k0 < S.w; k0 += U) {
                T x[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    x[u] = p[j[u] >= 0 ? j[u] : row];
                int32_t jn[U];
                T an[U];
                fetch(k0 + U, jn, an);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    acc = j[u] >= 0 ? acc + a[u] * x[u] : acc;
                    diag = j[u] == row ? a[u] : diag;
                    j[u] = jn[u], a[u] = an[u];
                }
            }
        }
        pc = p[c];
        y = acc;
        if constexpr (sizeof(T) == 8)
            dinv = precond ? T(1) / diag : T(1);
        else
            dinv = invd[c];
        wt = precond ? diag : T(1);
    }
};

}  // namespace sstep
