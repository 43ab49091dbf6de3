// Host check of rgc_tickets.h: `resident` threads stand for the workgroups that fit on the device, each runs one workgroup after
// the other until the whole grid has run.  A unit must run once in every pass of its layer, after all the layer's units of the
// pass before, and the whole must end whatever `resident` is.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "../paper_1808_04357_amd/csrc/rgc_tickets.h"

using namespace rgc;

namespace {

struct Layer {
  uint32_t units = 1, begins = 0, passes = 0;   // passes: how many this layer goes through, from launch `begins` on
  std::atomic<uint32_t> published{0}, done{0};
};

struct Shared {
  std::vector<Layer> layers;
  std::vector<uint32_t> unit_layer;
  std::atomic<uint32_t> tickets{0}, runs{0}, faults{0};
  uint32_t first = 0;
  std::chrono::steady_clock::time_point limit;
};

struct Work {
  Shared& S;
  uint32_t take() { return S.tickets.fetch_add(1); }
  void unit(uint32_t u, uint32_t launch) {
    Layer& L = S.layers[S.unit_layer[u]];
    Due d;
    while ((d = due_at(L.published.load(std::memory_order_acquire), launch, S.first)) == Due::kWait) {
      if (std::chrono::steady_clock::now() > S.limit) { std::printf("stuck\n"); std::fflush(stdout); std::_Exit(2); }
      std::this_thread::yield();
    }
    if (d == Due::kSkip) return;
    if (launch < L.begins || launch >= L.begins + L.passes) S.faults.fetch_add(1);
    S.runs.fetch_add(1);
    if (L.done.fetch_add(1) + 1u == L.units) {               // the layer's last unit of the pass
      L.done.store(0);
      const uint32_t next = launch + 1u;
      if (next < L.begins + L.passes)
        L.published.store(next | (next + 1u == L.begins + L.passes ? kLastPass : 0u), std::memory_order_release);
    }
  }
};

void check(uint32_t num_layers, uint32_t grid, uint32_t resident, uint32_t seed) {
  const uint32_t first = 4, passes = 5;
  Shared S;
  S.layers = std::vector<Layer>(num_layers);
  S.first = first;
  S.limit = std::chrono::steady_clock::now() + std::chrono::seconds(60);
  uint32_t expected = 0, x = seed;
  auto random = [&](uint32_t below) { x = x * 1664525u + 1013904223u; return (x >> 16) % below; };
  for (uint32_t l = 0; l < num_layers; ++l) {
    Layer& L = S.layers[l];
    L.units = 1u + random(40);
    L.begins = first;
    L.passes = random(passes + 1u);                          // 0: the layer has nothing to do
    const uint32_t stale = random(first);                    // ... and still holds a launch number before the first pass
    L.published = L.passes == 0u ? stale : first | (L.passes == 1u ? kLastPass : 0u);
    for (uint32_t u = 0; u < L.units; ++u) S.unit_layer.push_back(l);
    expected += L.units * L.passes;
  }
  const TicketOrder order = ticket_order(static_cast<uint32_t>(S.unit_layer.size()), grid, passes);
  if (order.slices > grid) S.faults.fetch_add(1);
  std::atomic<uint32_t> started{0};
  std::vector<std::thread> slots;
  for (uint32_t r = 0; r < resident; ++r)
    slots.emplace_back([&] {
      while (started.fetch_add(1) < order.slices) {          // the grid: one workgroup per slice
        Work work{S};
        run_tickets(order, first, work);
      }
    });
  for (auto& t : slots) t.join();
  if (S.runs != expected || S.faults != 0u || S.tickets != order.slices * passes + order.slices) {
    std::printf("layers %u grid %u resident %u: %u of %u units, %u faults\n", num_layers, grid, resident, S.runs.load(), expected, S.faults.load());
    std::exit(1);
  }
}

}  // namespace

int main() {
  static_assert(due_at(4u, 4u, 4u) == Due::kRun && due_at(4u | kLastPass, 4u, 4u) == Due::kRun, "");
  static_assert(due_at(4u, 5u, 4u) == Due::kWait && due_at(4u | kLastPass, 5u, 4u) == Due::kSkip, "");
  static_assert(due_at(3u, 4u, 4u) == Due::kSkip && due_at(0u, 8u, 4u) == Due::kSkip, "");
  for (uint32_t resident : {1u, 2u, 3u, 7u})
    for (uint32_t grid : {1u, 8u, 64u, 100000u})
      for (uint32_t layers : {1u, 5u, 60u})
        for (uint32_t seed = 1; seed <= 5; ++seed) check(layers, grid, resident, seed * 7919u + layers);
  std::printf("tickets_check ok\n");
  return 0;
}
