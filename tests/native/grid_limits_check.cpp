// in_launches (grid_limits.h) over the block counts given as arguments: prints
// "blocks launches covered" for each, and fails when a launch does not fit, leaves a
// block out or takes one twice.
#include <cstdio>
#include <cstdlib>

#include "grid_limits.h"

int main(int argc, char **argv)
{
    for (int k = 1; k < argc; ++k) {
        const uint64_t blocks = std::strtoull(argv[k], nullptr, 10);
        uint64_t next = 0, launches = 0;
        const int e = sstep::in_launches(blocks, 0, [&](uint64_t first, uint32_t count) -> int {
            ++launches;
            if (first != next || count == 0 || !sstep::launch_fits(count, 1024))
                return 1;
            next = first + count;
            return 0;
        });
        if (e != 0 || next != blocks)
            return 1;
        std::printf("%llu %llu\n", (unsigned long long)blocks, (unsigned long long)launches);
    }
    const int e = sstep::in_launches(uint64_t(1) << 23, 0, [](uint64_t first, uint32_t) { return first ? 7 : 0; });
    if (e != 7)
        return 1;
    std::printf("%d %d\n", int(sstep::launch_fits((1u << 24) - 1, 256)), int(sstep::launch_fits(1u << 24, 256)));
    return 0;
}
