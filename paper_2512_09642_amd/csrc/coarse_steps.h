// The launches of the overlapped coarse sweeps (kernels_coarse.hip; host code
// without HIP dependency).
#pragma once

#include <algorithm>
#include <cstdint>

namespace sstep {

constexpr int64_t kCoarseRows = 65535;  // block rows of a launch

// Dependent steps of nu >= 1 sweeps over nwf wavefronts: sweep l takes wavefront t
// at step t + 8 l.
inline int64_t coarse_steps(int64_t nwf, int64_t nu) { return nwf + 8 * (nu - 1); }

// The sweeps first .. last of a step.
struct StepSweeps {
    int64_t first, last;
};
inline StepSweeps step_sweeps(int64_t step, int64_t nwf, int64_t nu)
{
    return {step < nwf ? 0 : (step - nwf) / 8 + 1, std::min<int64_t>(step / 8, nu - 1)};
}

// f(t, rows) for each launch of a step: block row y takes wavefront t - 8 y.
// The rows of a step are independent, so a step of more than kCoarseRows goes in
// several launches.
template <class F>
inline void step_launches(int64_t step, int64_t nwf, int64_t nu, F &&f)
{
    const StepSweeps s = step_sweeps(step, nwf, nu);
    for (int64_t l = s.first; l <= s.last; l += kCoarseRows)
        f(static_cast<int>(step - 8 * l), static_cast<uint32_t>(std::min(s.last - l + 1, kCoarseRows)));
}

// The steps one after the other, for a block that walks them itself.  The sweeps of
// a step stand at the wavefronts oldest(), oldest() - 8, ..., newest(); steps without
// any (between sweeps over fewer than 8 wavefronts) are left out.
struct StepWalk {
    int nwf, phase, active, left;  // phase: steps since the newest sweep began; left: sweeps not begun

    constexpr StepWalk(int fronts, int nu) : nwf(fronts), phase(0), active(1), left(nu - 1) {}
    constexpr bool more() const { return active > 0; }
    constexpr int newest() const { return phase; }
    constexpr int oldest() const { return phase + 8 * (active - 1); }
    constexpr void next()
    {
        ++phase;
        if (oldest() == nwf)
            --active;
        if (left > 0 && (phase == 8 || active == 0))
            --left, ++active, phase = 0;
    }
};

}  // namespace sstep
