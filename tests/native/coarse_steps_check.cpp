// The launches of coarse_steps.h for "nwf nu" given as arguments: every sweep takes
// every wavefront once, at step t + 8 l, in launches of at most kCoarseRows rows;
// prints the steps, launches and the most rows of one.  The walk of one block
// (StepWalk) takes the same steps.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "coarse_steps.h"

int main(int argc, char **argv)
{
    if (argc != 4)
        return 2;
    const int64_t nwf = std::atol(argv[1]), nu = std::atol(argv[2]), every = std::atol(argv[3]);
    std::vector<int64_t> sweeps(size_t(nwf), 0);  // sweeps that have taken the wavefront
    int64_t launches = 0, most = 0;
    const int64_t steps = sstep::coarse_steps(nwf, nu);
    for (int64_t step = 0; step < steps; step += every) {
        std::vector<char> seen(every > 1 ? size_t(nwf) : 0, 0);
        sstep::step_launches(step, nwf, nu, [&](int t0, uint32_t rows) {
            ++launches;
            most = std::max<int64_t>(most, rows);
            for (int64_t y = 0; y < rows; ++y) {
                const int64_t t = t0 - 8 * y, l = (step - t) / 8;
                if (t < 0 || t >= nwf || (step - t) % 8 || l < 0 || l >= nu)
                    std::exit(1);
                if (every > 1) {
                    if (seen[size_t(t)]++)
                        std::exit(3);
                } else if (sweeps[size_t(t)]++ != l) {
                    std::exit(4);
                }
            }
        });
    }
    if (every == 1)
        for (int64_t v : sweeps)
            if (v != nu)
                return 5;
    if (most > 65535)
        return 6;
    if (every == 1) {  // the same walked by one block
        std::vector<int64_t> walked(size_t(nwf), 0);
        int64_t ended = 0, held = 0;
        for (sstep::StepWalk w{static_cast<int>(nwf), static_cast<int>(nu)}; w.more(); w.next()) {
            ++held;
            int64_t l = ended;
            for (int t = w.oldest(); t >= w.newest(); t -= 8, ++l) {
                if (t < 0 || t >= nwf || walked[size_t(t)]++ != l)
                    return 7;
                ended += t == nwf - 1;
            }
        }
        for (int64_t v : walked)
            if (v != nu)
                return 8;
        if (held != (nwf < 8 ? nwf * nu : steps))
            return 9;
    }
    std::printf("%ld %ld %ld\n", long(steps), long(launches), long(most));
    return 0;
}
