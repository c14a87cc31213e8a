// meet.h — the workgroups of a launch agree on whether to run together (bq_cluster.hip).
//
// Word 0 of `mem` counts arrivals and carries the one decision, made once by a compare and swap:
// go, by the last to arrive and if every XCD has enough workgroups, or abort, by the same one
// if not or by anyone who waited too long.  All return that decision, so none runs unless all
// are resident, and none leaves a run that others began.  Words 2 to 9 count the workgroups of
// an XCD; a workgroup's count is performed before its arrival (arrive() releases it), so the
// last arrival finds the counts complete.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbit {

constexpr int kXcds = 8;
constexpr uint32_t kMeetGo = 0x40000000u, kMeetAbort = 0x80000000u;

// slot: the workgroup's number on its XCD (no member's if the XCD is none of the eight).  Mem:
// add(word, v) and read(word) unordered, arrive() adds 1 to word 0 in order (acquire and
// release), swap(seen, v) replaces word 0, late() the wait limit has passed, pause().
template <class Mem>
__host__ __device__ inline bool meet(Mem &mem, uint32_t groups, uint32_t members, uint32_t xcc, uint32_t &slot)
{
    slot = xcc < (uint32_t)kXcds ? mem.add(2 + xcc, 1u) : ~0u;
    uint32_t seen = mem.arrive() + 1u;
    if (seen == groups) {
        bool enough = true;
        for (int k = 0; k < kXcds; ++k) enough = enough && mem.read(2 + k) >= members;
        const uint32_t decision = seen | (enough ? kMeetGo : kMeetAbort);
        if (mem.swap(seen, decision)) seen = decision;
    }
    while (!(seen & (kMeetGo | kMeetAbort))) {
        if (mem.late()) {
            const uint32_t decision = seen | kMeetAbort;
            if (mem.swap(seen, decision)) seen = decision;
        } else {
            mem.pause();
            seen = mem.read(0);
        }
    }
    return (seen & kMeetGo) != 0u;
}

}  // namespace pbit
