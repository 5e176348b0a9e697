// Host check of the lanes of a serving tick with fake streams: forked lanes
// start after the main one, joins wait for them, and a tick that fails at any of
// its calls leaves nothing in flight on any lane.
#include <cstdio>
#include <vector>

#include "../../paper_2007_03847_amd/csrc/serve_lanes.hpp"

namespace {

constexpr int kN = 4;
int g_calls, g_fail_at;                     // the g_fail_at-th runtime call fails
std::vector<int> g_busy(kN + 1);            // work queued on stream 1 .. kN, not waited for by the host
std::vector<std::vector<int>> g_seen(kN + 1), g_event(kN + 1);  // what a stream (event) is ordered after

struct Ops {
  using Stream = int;
  using Event = int;
  using Error = int;
  static constexpr Error kOk = 0;
  static Error step() { return ++g_calls == g_fail_at ? 1 : 0; }
  static Error record(Event e, Stream s) {
    if (step()) return 1;
    g_event[e] = g_seen[s];
    return 0;
  }
  static Error wait(Stream s, Event e) {
    if (step()) return 1;
    for (int w : g_event[e]) g_seen[s].push_back(w);
    return 0;
  }
  static void sync(Stream s) { g_busy[s] = 0; }
};
using L = fmc::serve::Lanes<Ops, kN>;

int launch(int s, int work) {  // a launch of a piece of work on stream s
  if (Ops::step()) return 1;
  g_busy[s] = 1;
  g_seen[s].push_back(work);
  return 0;
}
bool after(int s, int work) {
  for (int w : g_seen[s])
    if (w == work) return true;
  return false;
}

int tick(L& l) {  // set-up on lane 0, a launch per lane, a last one on lane 0
  if (launch(l.st, 100)) return -1;
  if (l.fork(kN)) return -1;
  for (int k = 0; k < kN; ++k)
    if (launch(l.lane(k), 200 + k)) return -1;
  if (l.join(kN)) return -1;
  if (launch(l.st, 300)) return -1;
  Ops::sync(l.st);  // lane 0 waited for the others
  for (int k = 1; k < kN; ++k)
    if (after(l.st, 200 + k)) g_busy[l.lane(k)] = 0;
  return 0;
}

}  // namespace

int main() {
  L l;
  l.st = 1;
  for (int k = 1; k < kN; ++k) l.side[k - 1] = k + 1;
  for (int k = 0; k < kN; ++k) l.ev[k] = k;
  int total = 1;
  for (g_fail_at = 0; g_fail_at <= total; ++g_fail_at) {
    g_calls = 0;
    for (int s = 0; s <= kN; ++s) g_busy[s] = 0, g_seen[s].clear(), g_event[s].clear();
    const int rc = l.run([&] { return tick(l); });
    if (g_fail_at == 0) {
      total = g_calls;
      for (int k = 1; k < kN; ++k)
        if (!after(l.lane(k), 100) || !after(l.st, 200 + k)) return std::printf("order of lane %d\n", k), 1;
    }
    if ((rc != 0) != (g_fail_at > 0)) return std::printf("status at call %d\n", g_fail_at), 1;
    for (int s = 1; s <= kN; ++s)
      if (g_busy[s]) return std::printf("call %d failed: stream %d still busy\n", g_fail_at, s), 1;
  }
  std::printf("ALL OK %d\n", total);
  return 0;
}
