// Runs a solve loop's queue (replay.h) over the expectations given as a string of
// 0 and 1 (1: the replay in flight is expected to be the last), one per read-back,
// until the replays are used up; prints the replays in flight at each wait.
#include <cstdio>
#include <cstdlib>
#include <string>

#include "replay.h"

int main(int argc, char **argv)
{
    if (argc != 3)
        return 2;
    const long bound = std::atol(argv[1]);
    const std::string last = argv[2];
    int64_t launched = 0, checked = 0;
    bool expect = false;
    while (checked < bound) {
        while (sstep::queue_replay(launched, checked, bound, expect))
            ++launched;
        if (launched == checked) {
            std::printf("stuck\n");
            return 1;
        }
        std::printf("%ld ", long(launched - checked));
        ++checked;
        expect = size_t(checked) <= last.size() && last[size_t(checked) - 1] == '1';
    }
    std::printf("%ld\n", long(launched));
    return 0;
}
