// Which graph replays of a solve are queued ahead (host code without HIP
// dependency, used by the solve loops and by a host test).
#pragma once

#include <cstdint>

namespace sstep {

// launched replays have been queued and checked of them read back; a solve takes
// at most bound.  One replay stays queued behind the one being waited for, so that
// the device does not wait for the host, unless the one in flight is expected to be
// the last: a replay after the stop still starts every kernel.  The loop queues
// while this holds, then waits: after an expectation that was wrong, too, the next
// wait has a replay behind it again.
inline bool queue_replay(int64_t launched, int64_t checked, int64_t bound, bool last)
{
    return launched < bound && launched - checked < (last ? 1 : 2);
}

}  // namespace sstep
