// Launches of more workgroups than one HIP launch takes.
#pragma once

#include <cstdint>

#include "rdf2v.h"

namespace rdf2v {

// HIP takes fewer than 2^32 threads in one dimension of a launch; of more it
// may run only what is left of their number modulo 2^32, without an error.
constexpr int64_t kMaxLaunchThreads = (int64_t(1) << 32) - 1;

// Calls launch(first, count) for consecutive parts of `blocks` workgroups of
// `threads` threads, none of them larger than a launch may be, every part but
// the last a multiple of `step` workgroups; ends at the first error. One part
// wherever a single launch takes them all.
template <class Launch>
rdf2v_status for_each_launch(int64_t blocks, int threads, int64_t step, Launch launch) {
  const int64_t most = kMaxLaunchThreads / threads / step * step;
  for (int64_t first = 0; first < blocks; first += most) {
    const rdf2v_status st = launch(first, blocks - first < most ? blocks - first : most);
    if (st != RDF2V_OK) return st;
  }
  return RDF2V_OK;
}

}  // namespace rdf2v
