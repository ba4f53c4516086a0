// How a wave of bound_scan_kernel queues what passes of a group's 16 result registers, and how long the queue is.
#pragma once

namespace psc {

// The registers that are queued between two drains at the most.  A wave that holds eight groups has room for a whole
// group's; one that holds four (its centroids take twice the LDS, and two workgroups are to fit a compute unit) drains
// after register 8 too.  A drain leaves up to 63 entries, and a register brings up to 64.
template <int GROUPS>
constexpr int kQueuedRegisters = GROUPS == 8 ? 16 : 9;
template <int GROUPS>
constexpr int kQueuePlaces = 64 * (kQueuedRegisters<GROUPS> + 1);

// some(t): whether anything passes in registers 3 t .. 3 t + 2 (t < 5); check(r) queues what passes in register r; drain()
// leaves at most 63 entries.  The drain in the middle does not depend on what passes in the registers before it.
template <int GROUPS, class Some, class Check, class Drain>
__attribute__((always_inline)) constexpr void queue_group(Some &&some, Check &&check, Drain &&drain)
{
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        if (some(t)) {
#pragma unroll
            for (int r = 3 * t; r < 3 * t + 3; ++r) check(r);
        }
        if (kQueuedRegisters<GROUPS> == 9 && t == 2) drain();
    }
    check(15);
    drain();
}

}  // namespace psc
