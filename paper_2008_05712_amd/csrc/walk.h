// Barnes-Hut interaction lists on the device: the lists of every bucket's work request, from a tree
// whose nodes are numbered in pre-order (children in ascending index, each node's ids contiguous).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gc {

struct WalkArgs {
  const int2* range;          // per node (first id, count)
  const double* com;          // per node centre of mass, 3 doubles
  const double* side;         // per node cube side
  const int32_t* skip;        // per node: index just past its subtree
  const float4* rec;          // per id (x, y, z, m)
  const int32_t* bucket_node; // per bucket: its leaf node
  int32_t n_nodes, n_buckets, n_ids;
  double theta;
  int32_t* n_first;           // count pass: per-bucket node count; fill pass: offsets (n_buckets + 1)
  int32_t* r_first;           // the same for direct ranges
  int32_t* node_idx;          // fill pass outputs
  int32_t* ranges;            // (first, count) pairs
  unsigned long long* bad;    // count of buckets whose leaf index or id range is invalid
  int32_t* sn;                // count pass: each bucket's first kWalkCapNodes node entries (or nullptr)
  int2* sr;                   // and first kWalkCapRanges ranges
  const int32_t* over;        // fill pass after a group walk: only buckets of these groups (or nullptr)
  const int32_t* rank;        // with `over`: the buckets' order in the groups
};
// Per-bucket room of the count pass's copy of the lists; a bucket with more is walked again.
constexpr int kWalkCapNodes = 2048;
constexpr int kWalkCapRanges = 128;
// The walk without allocation: its scratch (256 bytes of totals, then 4 bytes per node) is a fixed
// device array of 8 MiB + 256 bytes, so trees of up to 2^21 nodes.
constexpr int kWalkNoAllocMaxNodes = 1 << 21;
constexpr size_t kWalkScratchBytes = 256 + sizeof(int32_t) * (size_t)kWalkNoAllocMaxNodes;

// The group walk (dense bucket lists): one wavefront walks one interval of the node indices for 64
// buckets of consecutive leaves at once.
constexpr int kWalkGroup = 64;      // buckets per group
constexpr int kWalkPart0 = 128;     // nodes of the rings next to a group's own; each further one doubles
constexpr int kWalkSplit = 4;       // intervals per ring
constexpr int kWalkPartCap = 384;   // kept steps per (group, interval); a group with more is walked again
// One node as the group walk reads it: the smallest squared distance at which the node is taken, its id
// range and the index past its subtree.
struct alignas(64) WalkNodeRec {
  double com[3];
  double s_take;
  int32_t begin, end, skip, pad[5];
};
struct WalkBox {  // one bucket: the tight box of its positions and its id range (end < begin: invalid)
  float lo[3], hi[3];
  int32_t begin, end;
};
struct GroupWalkArgs {
  WalkNodeRec* node;          // n_nodes
  int32_t* parent;            // n_nodes (-1: the root)
  WalkBox* box;               // per bucket
  int32_t* perm;              // buckets in the order of their leaves
  int2* count;                // per bucket: node entries, direct ranges
  int32_t* mark;              // n_nodes, used when the bucket list is not in leaf order
  int32_t* unsorted;          // != 0: some bucket's leaf precedes the one before it (cleared by the caller)
  int32_t* over;              // per group: an interval had more steps than its room
  unsigned long long* n_over; // groups with `over` set (cleared by the caller)
  int32_t* part_n;            // per (group, interval): kept steps
  int32_t* step_node;         // kept steps: the node,
  ulonglong2* step_mask;      // the group's buckets that take it and those that list it as a leaf
  int32_t n_groups, n_parts;  // n_parts = walk_parts(n_nodes)
};
constexpr int walk_rings(int32_t n_nodes) {
  int r = 1;
  while (((int64_t)kWalkPart0 << r) - kWalkPart0 < n_nodes) ++r;
  return r;
}
constexpr int walk_parts(int32_t n_nodes) { return 2 * kWalkSplit * walk_rings(n_nodes) + 1; }
constexpr int32_t kWalkGroupMaxNodes = (1 << 25) - 1;
constexpr int kWalkMaxParts = 256;  // (the list fill takes an interval a thread)
static_assert(walk_parts(kWalkGroupMaxNodes) == 153 && walk_parts(kWalkGroupMaxNodes) <= kWalkMaxParts, "intervals");

hipError_t launch_group_walk(const WalkArgs& a, const GroupWalkArgs& g, hipStream_t s);
// After the scan: every group's lists at their offsets, from the kept steps (groups marked `over` are
// left to launch_walk(true)).
hipError_t launch_group_fill(const WalkArgs& a, const GroupWalkArgs& g, hipStream_t s);
hipError_t launch_subtree_end(const int2* range, int32_t n_nodes, int32_t* skip, hipStream_t s);
hipError_t launch_walk(bool fill, const WalkArgs& a, hipStream_t s);
// After the scan: the lists of every bucket that fit the count pass's room, copied to their offsets.
hipError_t launch_walk_copy(const WalkArgs& a, hipStream_t s);
// In-place exclusive scan of two count arrays of n entries (entry n receives the total); the two
// totals, as 64-bit sums, go to totals[0] and totals[1].
hipError_t launch_scan_counts(int32_t* a, int32_t* b, int32_t n, long long* totals, hipStream_t s);

}  // namespace gc
