// MSM launch helpers (internal); see msm.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace zk {
namespace msm {

constexpr int kPointWords = 24;  // affine point: x, y as twelve 32-bit words each
constexpr int kXyzzWords = 48;   // the result: X, Y, ZZ, ZZZ, twelve words each
constexpr int kAccWords = 56;    // a working point: X, Y, ZZ, ZZZ, fourteen limbs each
constexpr int kScratchWords = kAccWords + 14;  // precomputation, per window: a point and a prefix product
constexpr int kTreeLevels = 8;   // levels of the bucket tree in one workgroup

// Buckets that span many runs, and the items their sums are cut into.
constexpr uint32_t kBigRuns = 128;  // runs per item
struct BigLists {
  uint32_t* count;   // buckets listed, items listed
  uint4* bucket;     // max_big_buckets(lanes): bucket, first item, items
  uint32_t* item;    // max_big_items(lanes): index into bucket
  uint32_t* part;    // max_big_items(lanes) working points
};

// Everything one MSM launch touches; the buffers are slices of the caller's
// workspace (sizes in msm_workspace_bytes).
struct MsmLaunch {
  const uint32_t* table;    // windows x n affine points: 2^(c w) P_i
  const uint32_t* scalars;  // n x 8 limbs, Montgomery form over BLS12-381 Fr
  uint64_t n;
  int c;                    // window bits
  int windows;
  uint32_t per_group;       // scalars per histogram group, per_group x windows <= 65535
  uint32_t groups;          // ceil(n / per_group)
  uint32_t lanes;           // accumulation lanes (accumulate_lanes)
  uint32_t kmin;            // fewest sorted entries per lane
  uint16_t* digits;         // windows x n
  uint16_t* ranks;          // windows x n: an entry's place among its group's entries of its bucket
  uint32_t* hist;           // groups x 2^c
  uint32_t* counts;         // 2^c
  uint32_t* offsets;        // 2^c + 1
  uint32_t* entries;        // windows x n
  uint32_t* head;           // lanes working points
  uint32_t* tail;           // lanes working points
  BigLists big;
  uint32_t* buckets;        // 2^c working points
  uint32_t* level_a;        // (1 + min(c, kTreeLevels)) x 2^(c - min(c, kTreeLevels)) working points
  uint32_t* level_b;        // c working points
  uint32_t* result;         // one XYZZ point
};

// table[w n + i] = 2^(c w) P_i for points first .. first + count of n;
// scratch: count x windows x kScratchWords words.
hipError_t launch_precompute(const uint32_t* pts, uint64_t n, uint64_t first, uint64_t count, int c, int windows,
                             uint32_t* table, uint32_t* scratch, hipStream_t s);
// A combine quad adds at most kCombineSerial runs' heads; a bucket spanning
// more runs is listed.  Such buckets own more than kCombineSerial run starts
// each, so at most lanes / kCombineSerial + 1 of them, and each has one item
// per kBigRuns run starts, rounded up.
constexpr uint32_t kCombineSerial = 16;
inline uint32_t max_big_buckets(uint32_t lanes) { return lanes / kCombineSerial + 1u; }
inline uint32_t max_big_items(uint32_t lanes) { return lanes / kBigRuns + max_big_buckets(lanes); }

// Accumulation lanes that are resident on the current device at once.
hipError_t accumulate_lanes(uint32_t* lanes);
hipError_t launch_msm(const MsmLaunch& m, hipStream_t s);

}  // namespace msm
}  // namespace zk
