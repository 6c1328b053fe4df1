// Whether the entries of a sliced CSR matrix (OpEll, common.h) go through the
// caches: host code without HIP dependency, used by the dispatch and by a host test.
#pragma once

#include <cstdint>

namespace sstep {

// Matrix values of at most this many bytes go through the caches, which hold
// them between products: basis step of a 7-point matrix, FP64, cached against
// non-temporal: 101^3 15.2 / 17.5 us, 128^3 (134 MB with padding) 28.4 / 35.7,
// 160^3 (257 MB) 65.3 / 65.4, 192^3 126 / 109.
constexpr int64_t kEllKeepBytes = int64_t(192) << 20;
// ... unless the entries of the vector that the listed slices read reach over more
// bytes than this, from a slice's first column to its last: then the matrix takes
// the place of the vector in the L2 (4 MB of each XCD).  Random columns, 7 a row,
// basis step cached / non-temporal: FP64 500000 rows 31.3 / 34.7 us, 600000 (4.8 MB)
// 41.4 / 42.0, 750000 52.5 / 49.3, 1000000 86.5 / 81.3; FP32 1000000 (4 MB) 47.7 /
// 54.1, 1500000 49.3 / 48.5; a grid's columns permuted among 512 rows, 2000376 rows
// (0.3 MB) FP64 32.8 / 44.8.
constexpr int64_t kEllKeepSpan = int64_t(11) << 19;

// values: entries of the slices, padding included; span: the mean over them of
// the rows between a slice's first and last column, 0 for a slice kept by offsets.
inline bool ell_keep_pays(int64_t values, int64_t span, int elem)
{
    return values * elem <= kEllKeepBytes && span * elem <= kEllKeepSpan;
}

}  // namespace sstep
