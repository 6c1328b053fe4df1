// Where one basis step of a constant operator is marched (k_basis_m, march.h):
// host code without HIP dependency, used by the dispatch and by a host test.
#pragma once

#include <cstdint>

namespace sstep {

// Tiles of the marched kernels: 64 x 32 lanes with a ring of one point.
constexpr int kMarchLanes = 64, kMarchRows = 32;

// Share of the lanes of its tiles that a plane of nx x ny points fills.
inline double march_fill(int64_t nx, int64_t ny)
{
    const int64_t tx = (nx + kMarchLanes - 3) / (kMarchLanes - 2), ty = (ny + kMarchRows - 3) / (kMarchRows - 2);
    return static_cast<double>(nx * ny) / static_cast<double>(tx * ty * kMarchLanes * kMarchRows);
}

// The alternative is a thread per point (7-point FP64 without products and even
// nx: k_basis_p2).  What a march costs grows with its lanes, filled or not, and a
// short one leaves the chip idle, so it is taken from some fill on and from some
// filled unknowns on, n times the fill.  us a step, marched / not:
//  * 27-point: from 4 MiB a column, fill 1/4, and 7 2^15 filled in FP64 (20 x 20 x
//    1500, 0.12 M: 14.0 / 11.3; 24 x 24 x 1500, 0.24 M: 14.4 / 15.8; 100 x 100 x 60,
//    0.37 M: 7.7 / 12.2), 9 2^16 in FP32 (30 x 200 x 200, 0.51 M: 10.7 / 9.6; 42 x
//    42 x 1000, 0.76 M: 10.9 / 13.0).
//  * 7-point with the products: from 24 MiB, fill 0.3.  The march is the faster
//    step only from 5 M filled unknowns on (187^3 34.6 / 32.3, 200^3 38.4 / 39.7,
//    224^3 45.8 / 56.8), but leaves a partial per block instead of one per 256
//    points: solves of 3 iterations with s = 9, 147^3 731 / 774, 187^3 1209 / 1321,
//    40 x 40 x 6000 (fill 0.39) 1759 / 1900.
//  * 7-point FP64 without them: fill 0.5, odd nx from 19 2^18 filled (187^3, 4.0 M:
//    35.2 / 30.8; 601 x 601 x 20, 6.1 M: 35.7 / 38.1), even nx, where k_basis_p2 is
//    the other way, from 9 2^20 (200^3, 5.6 M: 38.3 / 35.6; 1024 x 1024 x 8, 7.2 M:
//    41.1 / 35.6; 256^3, 11.9 M: 72.5 / 91.2; above the line 1024 x 1024 x 64 alone
//    376 / 346).
//  * 7-point FP32: from 24 MiB, fill 0.5 (64 x 200 x 700, fill 0.45: 28.2 / 25.9;
//    300^3 67.5 / 79.7; solves with s = 9, 187^3 916 / 933, 256^3 2354 / 2406).
//  * 7-point with A p stored: not marched (FP64 187^3 45 / 35, 225^3 75 / 67, FP32
//    224^3 40 / 33, 256^3 64 / 49; the other way 300^3 154 / 179 and 87 / 89).
inline bool march_step_pays(int64_t nx, int64_t ny, int64_t nz, bool box, int elem, bool products, bool stored_ap)
{
    const int64_t n = nx * ny * nz, bytes = n * elem;
    const double fill = march_fill(nx, ny), filled = fill * static_cast<double>(n);
    const bool fp64 = elem == 8;
    if (nz < 2)
        return false;
    if (box)
        return bytes >= (int64_t(4) << 20) && fill >= 0.25 && filled >= (fp64 ? 7 << 15 : 9 << 16);
    if (stored_ap || bytes < (int64_t(24) << 20))
        return false;
    if (products)
        return fill >= 0.3;
    return fill >= 0.5 && (!fp64 || filled >= (nx % 2 ? 19 << 18 : 9 << 20));
}

}  // namespace sstep
