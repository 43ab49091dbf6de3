// The order in which one launch does several passes over the same units of work (workgroup numbers), where a unit may depend on
// units of the pass before.  Its workgroups need not all fit on the device at once: a stream may be confined to a few compute
// units, and other kernels may hold the rest.  No HIP in here: the host tests run it with threads.
//
// Workgroups take tickets from one counter; a ticket is a slice of one pass, and the passes' tickets follow each other.  A unit
// whose layer is still in an earlier pass waits for it, that is for units of smaller tickets.  A ticket is only ever taken by a
// workgroup that runs, so the smallest ticket not done waits for nothing, and however few workgroups run, all tickets get done.
#pragma once

#include <stdint.h>

namespace rgc {

struct TicketOrder {
  uint32_t units;
  uint32_t slices, passes;      // tickets of a pass, passes
};

// Passes of at most `wanted` tickets each.  A ticket's units lie `slices` apart: those of one layer, which may be the only one with
// anything to do, go to as many tickets as it has units.
constexpr TicketOrder ticket_order(uint32_t units, uint32_t wanted, uint32_t passes) {
  const uint32_t most = wanted < 1u ? 1u : wanted;
  return TicketOrder{units, units < 1u ? 1u : units < most ? units : most, passes};
}

// What a layer publishes: the launch number it is due at, with kLastPass if no other follows.  Launch numbers below the first
// pass's: the layer has nothing to do here.
constexpr uint32_t kLastPass = 0x80000000u;

enum class Due { kSkip, kRun, kWait };

constexpr Due due_at(uint32_t published, uint32_t launch, uint32_t first) {
  const uint32_t at = published & ~kLastPass;
  if (at == launch) return Due::kRun;
  return at < first || at > launch || (published & kLastPass) != 0u ? Due::kSkip : Due::kWait;
}

// take(): the next ticket, the same for all threads of the workgroup; unit(u, launch): waits while due_at() says so, then does
// the unit if it is due.
template <typename Work>
constexpr void run_tickets(const TicketOrder& o, uint32_t first, Work& work) {
  for (uint32_t t = work.take(); t < o.slices * o.passes; t = work.take()) {
    for (uint32_t u = t % o.slices; u < o.units; u += o.slices) work.unit(u, first + t / o.slices);
  }
}

}  // namespace rgc
