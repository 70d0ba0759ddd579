// Rules by which the host chooses among launches: plain functions of sizes,
// without HIP, so that they can be checked on any machine.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace zk {
namespace rules {

// Whole transforms of 2^log_n points in one tile each, `elements` elements in
// the launch: true where the register kernels take them.  Up to 2^7 points
// always.  From 2^8 to 2^10 points the matrix-core kernels hold one element
// per lane, for the latency of a launch that does not fill the chip; one that
// does is shorter in the register kernels, four per lane (matrix cores and
// registers, us: 16,384 of 2^8 points 174 and 154, 4,096 of them 53 and 53;
// 8,192 of 2^9 185 and 176, 2,048 of them 57 and 60; 4,096 of 2^10 238 and
// 202, 1,024 of them 72 and 69, 512 of them 41 and 44).
constexpr bool register_whole(uint32_t log_n, uint64_t elements) {
  return log_n <= 7 || (log_n <= 10 && (elements >> (log_n == 10 ? 20 : 21)) != 0);
}

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

// Batches: estimated times of the two ways to run a group of transforms, in
// microseconds; only their order matters.
constexpr double kLaunchUs = 4.0;                // gap between dependent launches
constexpr double kPassUs = 6.0;                  // shortest matrix-core pass
constexpr double kUsPerElem = 33.0 / (1 << 20);  // a pass that fills the chip, per element
constexpr double kBatchItemUs = 70.0;            // one 2^11-element item of the persistent kernel

// One pass of `jobs` transforms of 2^log_n points as one launch.  `whole`:
// whole transforms of at most 2^7 points, a workgroup of the register kernels
// each, 4 per CU at once and shorter with the size (40 us at 2^10 points), in
// a batch that holds nothing larger.  These have no floor of kPassUs: the
// persistent kernel's estimate, which has no floor either, would win, and 64
// transforms of 2^2 (2^6) points take 13 (18) us as a launch and 34 (43) us in
// the persistent kernel.  Beside larger transforms, where the launch does not
// save the persistent kernel, they are better left to it (40 transforms of 2^2
// and 40 of 2^12 points: 59 us, and 67 with both as launches).
inline double grouped_pass_us(uint32_t log_n, bool whole, uint64_t jobs, int cus) {
  if (whole) {
    const uint64_t rounds = (jobs + 4u * (uint64_t)cus - 1) / (4u * (uint64_t)cus);
    return kLaunchUs + (double)rounds * 40.0 * (double)(1u << log_n) / 1024.0;
  }
  return kLaunchUs + std::max(kPassUs, kUsPerElem * (double)(1ull << log_n) * (double)jobs);
}

// The persistent kernel over `items` items with room for `slots` at once.
inline double persistent_us(double items, double slots) { return items * kBatchItemUs / slots; }

// Side streams a batch's direct work is dealt to, at most.  In a graph they
// are parallel branches, and a fourth costs nothing: the 64-job batch takes
// 0.411 ms with three, 0.390 with four, 0.397 with six.  A batch launched
// without one pays for each on the host, at every launch, with a wait, a
// record and another wait, and its launches come later (five transforms of 2^8
// points in five launches 89 us with three, 105 with four; 64 transforms of
// 2^10 to 2^18 points, all as launches, 413 and 501).  Not always: 16 of 2^10
// points in twelve groups, waited for one batch at a time, 147 us with four and
// 163 to 212 with three; one after the other 118 to 164 with three and 163.
inline size_t side_streams(bool graph) { return graph ? 4 : 3; }

}  // namespace rules
}  // namespace zk
