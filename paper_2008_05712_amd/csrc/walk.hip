// Barnes-Hut interaction lists of the buckets' work requests (Sec. 4.1: a bucket's particles share
// one node list and one direct list), built on the device.
//
// Opening test (FP64, no contraction, correctly rounded square root): bucket B takes node N when
// theta > 0, N's id range does not overlap B's and side(N) < theta * dist(com(N), box(B)); box(B) is
// the tight bounding box of B's FP32 positions and dist the distance from a point to the box, per
// axis e = lo - c below, c - hi above, else 0, summed as (e_x^2 + e_y^2) + e_z^2.  A node that is not
// taken goes, if a leaf, to the direct list as its id range and is otherwise opened.
//
// Nodes are numbered in pre-order with every node's ids contiguous, so a node's subtree is the
// index range [k, skip[k]) and the walk is one forward pass over the indices: a taken node or a leaf
// continues at skip[k], an opened node at k + 1.  Every step moves forward, so each lane ends within
// n_nodes steps.  One lane per bucket.  The count pass also keeps each bucket's lists, up to a fixed
// room; after the scan of the counts they are copied to their offsets, and only a bucket that did
// not fit is walked again.
//
// That form serves sparse bucket lists and the walk without allocation; dense lists (all the leaves of
// a tree, or a stretch of them) are walked 64 buckets at a time, further below.
#include "walk.h"

#include "mem_dev.h"

namespace gc {
namespace {

using dev::gld;
using dev::gst;

// First node after k's subtree: the first later node whose id range starts at or after the end of
// k's (first ids never decrease along a pre-order numbering with contiguous id ranges), else n.
__global__ void __launch_bounds__(256) k_subtree_end(const int2* __restrict__ range, int32_t n,
                                                     int32_t* __restrict__ skip) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int2 r = gld(range + k);
  const int end = r.x + r.y;
  int lo = k + 1, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (gld(range + mid).x >= end) hi = mid;
    else lo = mid + 1;
  }
  skip[k] = lo;
}

struct WalkNode {
  int2 range;
  double com[3];
  double side;
  int skip;
};

// Node k's walk data; past the last node, a record that is never used (the walk stops there).
__device__ __forceinline__ WalkNode load_node(const WalkArgs& a, int k) {
  WalkNode w;
  if (k < a.n_nodes) {
    w.range = gld(a.range + k);
    w.com[0] = a.com[3 * (int64_t)k];
    w.com[1] = a.com[3 * (int64_t)k + 1];
    w.com[2] = a.com[3 * (int64_t)k + 2];
    w.side = a.side[k];
    w.skip = gld(a.skip + k);
  } else {
    w.range = make_int2(0, 0);
    w.com[0] = w.com[1] = w.com[2] = 0.0;
    w.side = 0.0;
    w.skip = k + 1;
  }
  return w;
}

template <bool FILL>
__global__ void __launch_bounds__(256) k_walk(WalkArgs a) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= a.n_buckets) return;
  if (FILL && a.over) {
    if (!gld(a.over + b / kWalkGroup)) return;
    b = gld(a.rank + b);
  }
  const int leaf = gld(a.bucket_node + b);
  int2 br = make_int2(0, 0);
  bool ok = leaf >= 0 && leaf < a.n_nodes;
  if (ok) {
    br = gld(a.range + leaf);
    ok = br.x >= 0 && br.y >= 0 && br.x <= a.n_ids - br.y;
  }
  if (!ok) {  // an invalid bucket gets empty lists and is counted
    if (!FILL) {
      a.n_first[b] = 0;
      a.r_first[b] = 0;
      atomicAdd(a.bad, 1ull);
    }
    return;
  }
  double lo[3] = {__builtin_inf(), __builtin_inf(), __builtin_inf()};
  double hi[3] = {-__builtin_inf(), -__builtin_inf(), -__builtin_inf()};
  for (int i = br.x; i < br.x + br.y; ++i) {
    const float4 p = gld(a.rec + i);
    const double v[3] = {p.x, p.y, p.z};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      lo[d] = v[d] < lo[d] ? v[d] : lo[d];
      hi[d] = v[d] > hi[d] ? v[d] : hi[d];
    }
  }
  int n_lim = 0, r_lim = 0, n_at = 0, r_at = 0;
  if (FILL) {  // the fill pass never writes past the bucket's counted share
    n_at = gld(a.n_first + b);
    n_lim = gld(a.n_first + b + 1) - n_at;
    r_at = gld(a.r_first + b);
    r_lim = gld(a.r_first + b + 1) - r_at;
    if (a.sn && n_lim <= kWalkCapNodes && r_lim <= kWalkCapRanges) return;  // copied from the count pass
  }
  int32_t* keep_n = (!FILL && a.sn) ? a.sn + (int64_t)kWalkCapNodes * b : nullptr;
  int2* keep_r = (!FILL && a.sn) ? a.sr + (int64_t)kWalkCapRanges * b : nullptr;
  int cn = 0, cr = 0;
  int kb0 = 0, kb1 = 0, kb2 = 0;  // node entries not yet kept (the last cn % 4)
  // both possible successors (k + 1 when k is opened, the end of k's subtree otherwise) are loaded at
  // the top of each step, so their latency overlaps the opening test of k
  WalkNode cur = load_node(a, 0);
  for (int k = 0; k < a.n_nodes;) {
    const int nxt = cur.skip;
    const WalkNode on_open = load_node(a, k + 1), on_skip = load_node(a, nxt);
    const int2 nr = cur.range;
    const bool disjoint = nr.x + nr.y <= br.x || br.x + br.y <= nr.x;
    double s = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double c = cur.com[d];
      double e = 0.0;
      if (c < lo[d]) e = __dsub_rn(lo[d], c);
      else if (c > hi[d]) e = __dsub_rn(c, hi[d]);
      s = __dadd_rn(s, __dmul_rn(e, e));
    }
    if (a.theta > 0.0 && disjoint && cur.side < __dmul_rn(a.theta, __dsqrt_rn(s))) {
      if (FILL && cn < n_lim) a.node_idx[n_at + cn] = k;
      if (!FILL && keep_n) {  // kept four at a time: one aligned 16-byte store per four entries
        const int slot = cn & 3;
        kb0 = slot == 0 ? k : kb0;
        kb1 = slot == 1 ? k : kb1;
        kb2 = slot == 2 ? k : kb2;
        if (slot == 3 && cn < kWalkCapNodes) *reinterpret_cast<int4*>(keep_n + (cn - 3)) = make_int4(kb0, kb1, kb2, k);
      }
      ++cn;
      k = nxt;
      cur = on_skip;
    } else if (nxt == k + 1) {
      if (FILL && cr < r_lim) {
        a.ranges[2 * (int64_t)(r_at + cr)] = nr.x;
        a.ranges[2 * (int64_t)(r_at + cr) + 1] = nr.y;
      }
      if (!FILL && keep_r && cr < kWalkCapRanges) keep_r[cr] = nr;
      ++cr;
      k = nxt;
      cur = on_skip;
    } else {
      k = k + 1;
      cur = on_open;
    }
  }
  if (!FILL && keep_n) {  // the last cn % 4 entries
    const int tail = cn & 3, at = cn - tail;
    if (tail > 0 && at < kWalkCapNodes) keep_n[at] = kb0;
    if (tail > 1 && at + 1 < kWalkCapNodes) keep_n[at + 1] = kb1;
    if (tail > 2 && at + 2 < kWalkCapNodes) keep_n[at + 2] = kb2;
  }
  if (!FILL) {
    a.n_first[b] = cn;
    a.r_first[b] = cr;
  }
}

// One wavefront per bucket: a bucket whose lists fit the count pass's room has them copied to its
// offsets (lanes over entries).
__global__ void __launch_bounds__(256) k_walk_copy(WalkArgs a) {
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (b >= a.n_buckets) return;
  const int n_at = gld(a.n_first + b), n_cnt = gld(a.n_first + b + 1) - n_at;
  const int r_at = gld(a.r_first + b), r_cnt = gld(a.r_first + b + 1) - r_at;
  if (n_cnt > kWalkCapNodes || r_cnt > kWalkCapRanges) return;  // walked again by the fill pass
  const int32_t* src_n = a.sn + (int64_t)kWalkCapNodes * b;
  for (int i = lane; i < n_cnt; i += 64) a.node_idx[n_at + i] = gld(src_n + i);
  const int2* src_r = a.sr + (int64_t)kWalkCapRanges * b;
  for (int i = lane; i < r_cnt; i += 64) {
    const int2 v = gld(src_r + i);
    a.ranges[2 * (int64_t)(r_at + i)] = v.x;
    a.ranges[2 * (int64_t)(r_at + i) + 1] = v.y;
  }
}

// ---------------------------------------------------------------- group walk
//
// Consecutive buckets of the tree open nearly the same nodes, so one wavefront walks the nodes that any
// of 64 of them reaches, its lanes being the buckets: the node's record comes once, by scalar loads,
// and the opening test is 18 FP64 operations for all 64 (the square root and the product with theta are
// folded, exactly, into one threshold per node).  The bound is the serial chain of steps of a wavefront,
// so a group's walk is cut into intervals of the node indices, short next to the group's own leaves
// and doubling away from them (a Barnes-Hut walk visits about as many nodes in each): 2 rings + 1
// wavefronts per group.  A wavefront that starts in the middle of the numbering first applies the
// tests of its first node's ancestors, from the parent up, so that the topmost taken one decides.
// A lane that takes a node sleeps until the end of its subtree; the next node is the first child if
// any lane opened this one, else the end of its subtree.  A step that gave any bucket an entry is
// kept as (node, mask of the buckets that take it, mask of those that list it as a leaf), and after
// the scan of the counts a second kernel turns the masks into the buckets' lists with coalesced
// stores.
//
// Plummer 262,144, buckets of 32 (26,714 buckets, 30,548 nodes; 821 nodes visited per bucket, 1,618 by
// a group's union, so half the lanes of a step are awake): 969 us with one lane per bucket (418
// wavefronts of divergent loads, up to a thousand dependent steps each) -> 162 us here, bound by the
// scalar loads' misses (the node table is 2 MB) rather than the 40 M vector instructions (65 us).
// Loading both successors ahead doubles those misses: 206 us against 180 us with two intervals per
// ring; one, two and four intervals per ring: 219, 180 and 155 us (shorter chains, more ancestors).

// P(s): a node of side `side` is taken at squared distance s
__device__ __forceinline__ bool takes(double side, double theta, double s) {
  return side < __dmul_rn(theta, __dsqrt_rn(s));
}

// The smallest s >= 0 with P(s), or NaN if there is none (no s compares >= NaN).  Both roundings are
// monotone, so P is a step function of s: bracketed around (side / theta)^2 and bisected over the bit
// patterns.
__device__ double take_threshold(double side, double theta) {
  constexpr long long kInf = 0x7ff0000000000000ll;
  if (!(theta > 0.0)) return __builtin_nan("");
  const double q = side / theta, g = q * q;
  long long lo = 0, hi = kInf;
  if (g >= 0.0 && g < __builtin_inf()) {
    const long long m = __double_as_longlong(g);
    if (m > 16 && !takes(side, theta, __longlong_as_double(m - 16))) lo = m - 16;
    if (m + 16 < kInf && takes(side, theta, __longlong_as_double(m + 16))) hi = m + 16;
  }
  if (lo == 0 && takes(side, theta, 0.0)) return 0.0;
  if (hi == kInf && !takes(side, theta, __builtin_inf())) return __builtin_nan("");
  while (hi - lo > 1) {  // !P(lo), P(hi)
    const long long mid = lo + (hi - lo) / 2;
    if (takes(side, theta, __longlong_as_double(mid))) hi = mid;
    else lo = mid;
  }
  return __longlong_as_double(hi);
}

// Node records (and their subtree ends, for the per-bucket walk), and per bucket: its counts cleared,
// and whether the list is in leaf order.
__global__ void __launch_bounds__(256) k_walk_prep(WalkArgs a, GroupWalkArgs g, int32_t* __restrict__ skip) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < a.n_buckets) {
    g.count[k] = make_int2(0, 0);
    if (k > 0 && gld(a.bucket_node + k) < gld(a.bucket_node + k - 1)) *g.unsorted = 1;
    if (k < g.n_groups) g.over[k] = 0;
  }
  if (k >= a.n_nodes) return;
  const int2 r = gld(a.range + k);
  const int end = r.x + r.y;
  int lo = k + 1, hi = a.n_nodes;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (gld(a.range + mid).x >= end) hi = mid;
    else lo = mid + 1;
  }
  WalkNodeRec n;
#pragma unroll
  for (int d = 0; d < 3; ++d) n.com[d] = a.com[3 * (int64_t)k + d];
  n.s_take = take_threshold(a.side[k], a.theta);
  n.begin = r.x;
  n.end = end;
  n.skip = lo;
#pragma unroll
  for (int d = 0; d < 5; ++d) n.pad[d] = 0;
  g.node[k] = n;
  skip[k] = lo;
  g.parent[k] = -1;
  g.mark[k] = 0;
}

// Parents of each node's children (node blocks), then boxes of the buckets, eight lanes per bucket, and
// the identity order when the list is in leaf order (bucket blocks).  A bucket whose leaf index or id
// range is invalid gets an empty range and is counted.
__global__ void __launch_bounds__(256) k_walk_boxes(WalkArgs a, GroupWalkArgs g, int32_t node_blocks) {
  if ((int)blockIdx.x < node_blocks) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= a.n_nodes) return;
    const int end = gld(a.skip + k);
    for (int c = k + 1; c < end; c = gld(a.skip + c)) g.parent[c] = k;
    return;
  }
  const int b = (blockIdx.x - node_blocks) * 32 + (threadIdx.x >> 3), sub = threadIdx.x & 7;
  if (b >= a.n_buckets) return;  // (the eight lanes of a bucket together)
  const int leaf = gld(a.bucket_node + b);
  int2 br = make_int2(0, 0);
  bool ok = leaf >= 0 && leaf < a.n_nodes;
  if (ok) {
    br = gld(a.range + leaf);
    ok = br.x >= 0 && br.y >= 0 && br.x <= a.n_ids - br.y;
  }
  const float inf = __builtin_inff();
  float lo[3] = {inf, inf, inf}, hi[3] = {-inf, -inf, -inf};
  if (ok)
    for (int i = br.x + sub; i < br.x + br.y; i += 8) {
      const float4 p = gld(a.rec + i);
      const float v[3] = {p.x, p.y, p.z};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        lo[d] = v[d] < lo[d] ? v[d] : lo[d];
        hi[d] = v[d] > hi[d] ? v[d] : hi[d];
      }
    }
#pragma unroll
  for (int o = 4; o > 0; o >>= 1)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float l = __shfl_xor(lo[d], o, 8), h = __shfl_xor(hi[d], o, 8);
      lo[d] = l < lo[d] ? l : lo[d];
      hi[d] = h > hi[d] ? h : hi[d];
    }
  if (sub == 0) {
    WalkBox w;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      w.lo[d] = lo[d];
      w.hi[d] = hi[d];
    }
    w.begin = ok ? br.x : 0;
    w.end = ok ? br.x + br.y : -1;
    g.box[b] = w;
    if (!ok) atomicAdd(a.bad, 1ull);
    if (*g.unsorted == 0) g.perm[b] = b;
  }
}

__device__ __forceinline__ int wave_scan_excl(int v, int* total) {
  const int lane = threadIdx.x & 63;
  int inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(inc, d, 64);
    if (lane >= d) inc += u;
  }
  *total = __shfl(inc, 63, 64);
  return inc - v;
}

// Buckets in leaf order when the list is not (one workgroup: a counting sort over the node indices;
// buckets of one leaf, and those with an invalid one, in any order).
__global__ void __launch_bounds__(1024) k_walk_sort(WalkArgs a, GroupWalkArgs g) {
  __shared__ int wsum[16];
  __shared__ int carry;
  if (*g.unsorted == 0) return;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  auto key = [&](int b) {
    const int l = gld(a.bucket_node + b);
    return l < 0 ? 0 : l >= a.n_nodes ? a.n_nodes - 1 : l;
  };
  for (int b = t; b < a.n_buckets; b += 1024) atomicAdd(g.mark + key(b), 1);
  if (t == 0) carry = 0;
  __threadfence();
  __syncthreads();
  for (int base = 0; base < a.n_nodes; base += 1024) {
    const int k = base + t;
    const int v = k < a.n_nodes ? dev::aload(g.mark + k) : 0;
    int tot;
    const int ex = wave_scan_excl(v, &tot);
    if (lane == 0) wsum[wv] = tot;
    __syncthreads();
    int before = carry + ex;
    for (int w = 0; w < wv; ++w) before += wsum[w];
    if (k < a.n_nodes) dev::astore(g.mark + k, before);
    __syncthreads();
    if (t == 1023) carry = before + v;
    __syncthreads();
  }
  __threadfence();
  __syncthreads();
  for (int b = t; b < a.n_buckets; b += 1024) g.perm[atomicAdd(g.mark + key(b), 1)] = b;
}

typedef const __attribute__((address_space(4))) uint32_t* cst_words;

// A node's record by scalar loads (k is uniform); past the last node, one that is never used.
__device__ __forceinline__ WalkNodeRec scalar_node(const WalkNodeRec* p, int k, int n) {
  WalkNodeRec r;
  constexpr int kWords = 11;  // com, s_take, begin, end, skip
  // (a 32-bit byte offset: at most kWalkGroupMaxNodes nodes)
  typedef const __attribute__((address_space(4))) char* cst_bytes;
  cst_words q = (cst_words)((cst_bytes)(const void*)p + (uint32_t)(k < n ? k : n - 1) * 64u);
  uint32_t w[16];
#pragma unroll
  for (int i = 0; i < kWords; ++i) w[i] = q[i];
#pragma unroll
  for (int i = kWords; i < 16; ++i) w[i] = 0;
  __builtin_memcpy(&r, w, sizeof r);
  return r;
}

__device__ __forceinline__ int wave_min_int(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
  return v;
}

__global__ void __launch_bounds__(256) k_group_walk(WalkArgs a, GroupWalkArgs g) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int grp = w / g.n_parts, part = w - grp * g.n_parts;
  if (grp >= g.n_groups) return;
  const int slot = grp * kWalkGroup + lane;
  const int n = a.n_nodes;
  const bool have = slot < a.n_buckets;
  const int b = have ? gld(g.perm + slot) : 0;
  const int leaf = have ? gld(a.bucket_node + b) : -1;
  const bool inside = leaf >= 0 && leaf < n;
  // the group's own interval [c0, c1) and this wavefront's [s, e)
  const int c0 = __builtin_amdgcn_readfirstlane(min(wave_min_int(inside ? leaf : n), n));
  const int c1 = __builtin_amdgcn_readfirstlane(-wave_min_int(inside ? -(leaf + 1) : 0));
  const int arm = g.n_parts >> 1;  // intervals on either side
  int64_t s, e;
  if (part == arm) {
    s = c0;
    e = c1;
  } else {
    const int j = part < arm ? arm - 1 - part : part - arm - 1;  // nearest first
    const int64_t ring = (int64_t)kWalkPart0 << (j / kWalkSplit), piece = ring / kWalkSplit;
    const int64_t near = ring - kWalkPart0 + piece * (j % kWalkSplit), far = near + piece;
    s = part < arm ? c0 - far : c1 + near;
    e = part < arm ? c0 - near : c1 + far;
  }
  s = s < 0 ? 0 : s;
  e = e > n ? n : e;
  int32_t* part_n = g.part_n + w;
  if (s >= e) {
    if (lane == 0) *part_n = 0;
    return;
  }
  double lo[3] = {0.0, 0.0, 0.0}, hi[3] = {0.0, 0.0, 0.0};
  int bb = 0, be = -1;
  if (have) {
    const int4* q = reinterpret_cast<const int4*>(g.box + b);
    const int4 u = gld(q), v = gld(q + 1);
    lo[0] = __int_as_float(u.x); lo[1] = __int_as_float(u.y); lo[2] = __int_as_float(u.z);
    hi[0] = __int_as_float(u.w); hi[1] = __int_as_float(v.x); hi[2] = __int_as_float(v.y);
    bb = v.z;
    be = v.w;
  }
  const bool valid = be >= bb;  // (an invalid bucket has empty lists)
  auto take = [&](const WalkNodeRec& r) {
#pragma clang fp contract(off)
    double e2[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double x = __builtin_fmax(__builtin_fmax(lo[d] - r.com[d], r.com[d] - hi[d]), 0.0);
      e2[d] = x * x;
    }
    const double s2 = (e2[0] + e2[1]) + e2[2];
    return (r.end <= bb || be <= r.begin) && s2 >= r.s_take;
  };
  int k = (int)s;
  const int last = (int)e;
  int wake = valid ? k : INT32_MAX;  // this lane sleeps until the walk reaches `wake`
  for (int p = __builtin_amdgcn_readfirstlane(gld(g.parent + k)); p >= 0;
       p = __builtin_amdgcn_readfirstlane(gld(g.parent + p))) {
    const WalkNodeRec r = scalar_node(g.node, p, n);
    if (valid && take(r)) wake = r.skip;
  }
  const int64_t base = (int64_t)w * kWalkPartCap;
  int cn = 0, cr = 0, kept = 0;
  int vk = 0, vt0 = 0, vt1 = 0, vl0 = 0, vl1 = 0;  // lane i: kept step i of the open group of 64
  auto flush = [&](int m) {
    const int at = kept - m;
    if (lane < m && at + lane < kWalkPartCap) {
      gst(g.step_node + base + at + lane, vk);
      const int4 mk = make_int4(vt0, vt1, vl0, vl1);
      *reinterpret_cast<int4*>(g.step_mask + base + at + lane) = mk;
    }
  };
  WalkNodeRec cur = scalar_node(g.node, k, n);
  while (k < last) {
    const uint64_t act = __ballot(wake <= k);
    if (act == 0) {  // every bucket sleeps (or is invalid): on to the first that wakes
      k = __builtin_amdgcn_readfirstlane(wave_min_int(wake));
      if (k >= last) break;
      cur = scalar_node(g.node, k, n);
      continue;
    }
    const int nxt = cur.skip;
    const bool tk = wake <= k && take(cur);
    const uint64_t tm = __ballot(tk);
    const uint64_t rest = act & ~tm;
    const bool is_leaf = nxt == k + 1;
    const uint64_t lm = is_leaf ? rest : 0;
    if (tm | lm) {
      cn += tk ? 1 : 0;
      cr += (int)((lm >> lane) & 1);
      const int i = kept & 63;
      const bool me = lane == i;
      vk = me ? k : vk;
      vt0 = me ? (int)(uint32_t)tm : vt0;
      vt1 = me ? (int)(uint32_t)(tm >> 32) : vt1;
      vl0 = me ? (int)(uint32_t)lm : vl0;
      vl1 = me ? (int)(uint32_t)(lm >> 32) : vl1;
      ++kept;
      if (i == 63) flush(64);
    }
    wake = tk ? nxt : wake;
    const bool open = !is_leaf && rest != 0;
    k = open ? k + 1 : nxt;
    cur = scalar_node(g.node, k, n);
  }
  flush(kept & 63);
  if (cn) atomicAdd(&g.count[b].x, cn);
  if (cr) atomicAdd(&g.count[b].y, cr);
  if (lane == 0) {
    *part_n = kept < kWalkPartCap ? kept : kWalkPartCap;
    if (kept > kWalkPartCap && atomicExch(g.over + grp, 1) == 0) atomicAdd(g.n_over, 1ull);
  }
}

// A quarter of a group's buckets per workgroup, four per wavefront: the group's kept steps (its
// intervals' in order, flattened through the prefix of their counts) go through LDS kFillChunk at a
// time, and each wavefront compacts the steps of its buckets, 64 at a time, by ballot onto their offsets.
constexpr int kFillChunk = 512;

__global__ void __launch_bounds__(256) k_group_fill(WalkArgs a, GroupWalkArgs g) {
  __shared__ int s_first[kWalkMaxParts + 1];  // first flat step of each interval
  __shared__ int s_wave[4];
  __shared__ int2 s_range[kFillChunk];
  __shared__ int s_node[kFillChunk];
  __shared__ uint32_t s_taken[kFillChunk], s_leaf[kFillChunk];  // the half of the masks that holds these buckets
  const int grp = blockIdx.x >> 2, quarter = blockIdx.x & 3;
  if (gld(g.over + grp)) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int bit0 = quarter * 16 + wv * 4;  // this wavefront's buckets: bits bit0 .. bit0 + 3
  int n_at[4], r_at[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int slot = grp * kWalkGroup + bit0 + q;
    const int b = slot < a.n_buckets ? gld(g.perm + slot) : -1;
    n_at[q] = __builtin_amdgcn_readfirstlane(b >= 0 ? gld(a.n_first + b) : 0);
    r_at[q] = __builtin_amdgcn_readfirstlane(b >= 0 ? gld(a.r_first + b) : 0);
  }
  {
    const int v = t < g.n_parts ? gld(g.part_n + grp * g.n_parts + t) : 0;
    int tot;
    const int ex = wave_scan_excl(v, &tot);
    if (lane == 0) s_wave[wv] = tot;
    __syncthreads();
    int at = ex;
    for (int w = 0; w < wv; ++w) at += s_wave[w];
    s_first[t] = at;
    if (t == 255) s_first[256] = at + v;
    __syncthreads();
  }
  const int total = s_first[256];
  const int half = quarter >> 1, sh = bit0 & 31;
  for (int f0 = 0; f0 < total; f0 += kFillChunk) {
    const int cnt = total - f0 < kFillChunk ? total - f0 : kFillChunk;
    for (int i = t; i < cnt; i += 256) {
      const int f = f0 + i;
      int lo = 0, hi = g.n_parts - 1;  // the last interval that starts at or before f
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_first[mid] <= f) lo = mid;
        else hi = mid - 1;
      }
      const int64_t at = ((int64_t)grp * g.n_parts + lo) * kWalkPartCap + (f - s_first[lo]);
      const int nd = gld(g.step_node + at);
      const int4 m = gld(reinterpret_cast<const int4*>(g.step_mask + at));
      s_node[i] = nd;
      s_taken[i] = (uint32_t)(half ? m.y : m.x);
      s_leaf[i] = (uint32_t)(half ? m.w : m.z);
      if (m.z | m.w) s_range[i] = gld(a.range + nd);
    }
    __syncthreads();
    for (int i0 = 0; i0 < cnt; i0 += 64) {
      const int i = i0 + lane;
      const bool in = i < cnt;
      const uint32_t tk = in ? (s_taken[i] >> sh) & 15u : 0u;
      const uint32_t lf = in ? (s_leaf[i] >> sh) & 15u : 0u;
      const int nd = in ? s_node[i] : 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint64_t m = __ballot((tk >> q) & 1u);
        if (m) {
          if ((tk >> q) & 1u)
            gst(a.node_idx + n_at[q] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)), nd);
          n_at[q] += __popcll(m);
        }
      }
      if (__ballot(lf != 0u)) {
        const int2 r = lf ? s_range[i] : make_int2(0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint64_t m = __ballot((lf >> q) & 1u);
          if (m) {
            if ((lf >> q) & 1u) {
              int32_t* o = a.ranges + 2 * ((int64_t)r_at[q] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)));
              gst(o, r.x);
              gst(o + 1, r.y);
            }
            r_at[q] += __popcll(m);
          }
        }
      }
    }
    __syncthreads();
  }
}

__device__ __forceinline__ long long wave_scan64(long long v) {  // inclusive
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const long long u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// One workgroup of 1024 threads over tiles of 4096 entries of both arrays: each thread takes four
// consecutive entries, wavefront scans and the 16 wavefronts' sums give its prefix, and a carry runs
// from tile to tile.  The next tile's entries are loaded before this one is scanned.
__global__ void __launch_bounds__(1024) k_scan_counts(int32_t* __restrict__ a, int32_t* __restrict__ b, int32_t n,
                                                      long long* __restrict__ totals) {
  __shared__ long long sum[2][2][16];  // by tile parity (one barrier per tile), array, wavefront
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  long long carry_a = 0, carry_b = 0;
  int va[4], vb[4], na[4], nb[4];
  auto fetch = [&](int64_t base, int (&x)[4], int (&y)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = base + 4 * t + q;
      x[q] = i < n ? gld(a + i) : 0;
      y[q] = i < n ? gld(b + i) : 0;
    }
  };
  fetch(0, va, vb);
  int par = 0;
  for (int64_t base = 0; base < n; base += 4096, par ^= 1) {
    fetch(base + 4096, na, nb);
    const long long ta = (long long)va[0] + va[1] + va[2] + va[3], tb = (long long)vb[0] + vb[1] + vb[2] + vb[3];
    const long long ia = wave_scan64(ta), ib = wave_scan64(tb);
    if (lane == 63) {
      sum[par][0][wv] = ia;
      sum[par][1][wv] = ib;
    }
    __syncthreads();
    long long pa = carry_a + ia - ta, pb = carry_b + ib - tb;  // exclusive prefix of the thread's entries
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const long long xa = sum[par][0][w], xb = sum[par][1][w];
      if (w < wv) {
        pa += xa;
        pb += xb;
      }
      carry_a += xa;
      carry_b += xb;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = base + 4 * t + q;
      if (i < n) {
        a[i] = (int32_t)pa;
        b[i] = (int32_t)pb;
      }
      pa += va[q];
      pb += vb[q];
      va[q] = na[q];
      vb[q] = nb[q];
    }
  }
  if (t == 0) {
    a[n] = (int32_t)carry_a;
    b[n] = (int32_t)carry_b;
    totals[0] = carry_a;
    totals[1] = carry_b;
  }
}

}  // namespace

hipError_t launch_group_walk(const WalkArgs& a, const GroupWalkArgs& g, hipStream_t s) {
  const int nb = (a.n_nodes + 255) / 256;
  const int prep = a.n_nodes > a.n_buckets ? a.n_nodes : a.n_buckets;
  hipLaunchKernelGGL(k_walk_prep, dim3((prep + 255) / 256), dim3(256), 0, s, a, g, const_cast<int32_t*>(a.skip));
  hipLaunchKernelGGL(k_walk_boxes, dim3(nb + (a.n_buckets + 31) / 32), dim3(256), 0, s, a, g, nb);
  hipLaunchKernelGGL(k_walk_sort, dim3(1), dim3(1024), 0, s, a, g);
  const int64_t waves = (int64_t)g.n_groups * g.n_parts;
  hipLaunchKernelGGL(k_group_walk, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, a, g);
  return hipGetLastError();
}

hipError_t launch_group_fill(const WalkArgs& a, const GroupWalkArgs& g, hipStream_t s) {
  hipLaunchKernelGGL(k_group_fill, dim3(4 * g.n_groups), dim3(256), 0, s, a, g);
  return hipGetLastError();
}

hipError_t launch_subtree_end(const int2* range, int32_t n_nodes, int32_t* skip, hipStream_t s) {
  if (n_nodes <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_subtree_end, dim3((n_nodes + 255) / 256), dim3(256), 0, s, range, n_nodes, skip);
  return hipGetLastError();
}

hipError_t launch_walk(bool fill, const WalkArgs& a, hipStream_t s) {
  if (a.n_buckets <= 0) return hipSuccess;
  // one wavefront per workgroup: tens of thousands of buckets then spread over every CU
  const dim3 g((a.n_buckets + 63) / 64);
  if (fill) hipLaunchKernelGGL(k_walk<true>, g, dim3(64), 0, s, a);
  else hipLaunchKernelGGL(k_walk<false>, g, dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_walk_copy(const WalkArgs& a, hipStream_t s) {
  if (a.n_buckets <= 0 || !a.sn) return hipSuccess;
  hipLaunchKernelGGL(k_walk_copy, dim3((a.n_buckets + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_scan_counts(int32_t* a, int32_t* b, int32_t n, long long* totals, hipStream_t s) {
  hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, s, a, b, n, totals);
  return hipGetLastError();
}

}  // namespace gc
