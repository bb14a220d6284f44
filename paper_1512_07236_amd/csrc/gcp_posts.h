// gcp_posts.h -- the scalars of a solve and how reductions report them to the
// host.  Plain C++, without HIP.
//
// Every reduction of a context has a number.  One that has something to say
// stores it to the host's copy of the scalars, after what it reports, and the
// host waits for the number.  Numbers wrap at 2^32, so they are compared by
// their signed difference, which is right while the two lie within 2^31 of
// each other: the host's copy keeps the last number posted when its other
// fields start anew.
#pragma once

#include <stdint.h>

#include <cmath>

namespace gcp {

// FP64 traces and the decision (device, and the host's copy).
struct Scalars {
  double t1, t2, t3, omega, c, step;
  int32_t status;   // 0 continue, 1 converged, 2 max_iter reached, 3 breakdown,
                    // 4 stopped at the rounding floor
  int32_t iter;     // update at which status became non-zero
  double hstat[4];  // Gershgorin min, max, Tr H
  double prev_ddbar;   // |Tr(D Dbar)| of the previous iterate (+inf before the first)
  int32_t on_traces;   // 1: the stop was decided from the update's traces, before
                       // the square of the last iterate was formed
  uint32_t seq;        // host copy only: the last reduction posted to it
};

// What a reduction tells the host: nothing, that it has run (seq), or also the
// scalars.  A reduction that stops the solve always posts everything.
enum { POST_NONE = 0, POST_SEQ = 1, POST_ALL = 2 };

// A context's numbers start 64 below the wrap: every context passes it in its
// first solves instead of after hours.
constexpr uint32_t kFirstSeq = 0u - 64u;

// Whether reduction `seq` has posted, from the last number posted.
inline bool posted(uint32_t last, uint32_t seq) { return (int32_t)(last - seq) >= 0; }

// The scalars at iterate (t1, t2), from which a solve or a recomputed segment
// starts; seq: the context's last number.
inline Scalars start_scalars(double t1, double t2, uint32_t seq) {
  Scalars s{};
  s.t1 = t1;
  s.t2 = t2;
  s.prev_ddbar = INFINITY;
  s.seq = seq;
  return s;
}

}  // namespace gcp
