// Rules by which the host chooses among launches: plain functions of sizes,
// without HIP, so that they can be checked on any machine.
#pragma once
#include <algorithm>
#include <cstdint>

namespace zk {
namespace rules {

// MSM: fewest sorted entries per accumulation lane, for `windows` windows of c
// bits and n points.  A mixed addition in a lane takes about twice as long as
// the addition of a run's head by a quad, so where lanes are to spare runs of
// about an eighth of a bucket end soonest, and no fewer than eight entries.
// No more than 32: the heads of a bucket that spans many runs are added by
// workgroups (the large-bucket lists), while a longer run is a longer serial
// chain in one lane, and an eighth of the bucket has no bound when n is large
// for the window (n = 4096, c = 1: 65,280 entries in each of 16 lanes, 690 ms;
// with runs of 32, 0.55 ms.  n = 2^16, c = 8: 10.6 and 0.86 ms).
inline uint32_t msm_min_run(uint64_t windows, uint64_t n, int c) {
  const uint64_t eighth = (windows * n) >> (c + 3);
  return (uint32_t)std::min<uint64_t>(32, std::max<uint64_t>(8, eighth));
}

}  // namespace rules
}  // namespace zk
