// serve_lanes.hpp -- the streams ("lanes") of a serving tick: a main one and
// side lanes forked from it and joined back.  Templated on the runtime's calls,
// so that the order of forks, joins and waits can be checked on the host.
#pragma once

namespace fmc {
namespace serve {

// Ops: Stream, Event and Error types, kOk, and record(Event, Stream), wait(Stream,
// Event), sync(Stream).
template <typename Ops, int N>
struct Lanes {
  typename Ops::Stream st{};            // lane 0
  typename Ops::Stream side[N - 1]{};   // lanes 1 .. N - 1
  typename Ops::Event ev[N]{};          // [0]: fork, [k]: lane k done

  typename Ops::Stream lane(int k) const { return k == 0 ? st : side[k - 1]; }

  // Lanes 1 .. n - 1 go on after what lane 0 has now.
  typename Ops::Error fork(int n) {
    if (n < 2) return Ops::kOk;
    typename Ops::Error e = Ops::record(ev[0], st);
    for (int k = 1; k < n && e == Ops::kOk; ++k) e = Ops::wait(lane(k), ev[0]);
    return e;
  }

  // Lane 0 goes on after what lanes 1 .. n - 1 have now.
  typename Ops::Error join(int n) {
    typename Ops::Error e = Ops::kOk;
    for (int k = 1; k < n && e == Ops::kOk; ++k) {
      e = Ops::record(ev[k], lane(k));
      if (e == Ops::kOk) e = Ops::wait(st, ev[k]);
    }
    return e;
  }

  // The host waits for every lane, joined or not.
  void drain() {
    for (int k = 0; k < N; ++k)
      if (lane(k)) Ops::sync(lane(k));
  }

  // Runs a tick (0: done, and lane 0 drained by itself).  A tick that fails
  // between a fork and its join leaves work on the side lanes that nothing waits
  // for: the lanes are drained before the caller gives the requests' memory back.
  template <typename F>
  int run(F&& tick) {
    const int rc = tick();
    if (rc) drain();
    return rc;
  }
};

}  // namespace serve
}  // namespace fmc
