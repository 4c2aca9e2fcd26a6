// Device code of the combined Barnes-Hut force pass (Sec. 3.1: many work
// requests in one launch; Sec. 4.1: a bucket's particles share one list of
// nodes and direct particles), shared by the per-batch kernel and the
// whole-step persistent kernel.
//
// Schedule: one workgroup of W wavefronts per task; the W waves split the
// task's node and direct lists.  A bucket holds few targets (about 10 on
// average for a Plummer sphere with buckets of 32), so within a wavefront the
// 64 lanes are split as (target i) x (source slice s): S = floor(64 / i_count)
// slices, lane = s * i_count + i.  Source records (direct particles, or node records) are
// staged by the wavefront into its private LDS tile with coalesced loads; the
// tile is padded with zero-mass entries to S * C records so every slice runs
// exactly C iterations with no per-iteration bounds test; a lane reads its
// slice's records from LDS (lanes of one slice read the same address: an LDS
// broadcast).  Node records of the next tile are prefetched into registers
// while the current tile is computed.  Each lane sums its slices in FP32 and
// adds that partial to an FP64 running sum at about 64 terms (a tile holds no
// more a slice), and at the end of the chunk; at the end the
// slices and then the waves of each target are reduced in FP64 through LDS in
// a fixed order and the target's float4 is written once.  No atomics: results
// are bitwise independent of task order and of the schedule.
//
// What bounds it: the rate at which vector instructions issue (9 cycles in 10 of a large pass).  A wave of a Plummer
// pass (131,072 to 262,144 particles, buckets of 32) runs 43 to 48 terms, 600 to 1,110 instructions, so
// what a wave does besides counts: loads that need no branch (raw buffers that end where the data
// does), divisions by 16-bit reciprocals, a scan by lane moves, ranges found without a search, two
// monopole nodes a lane, sums reduced by component, and a target found among its sources as they are
// copied instead of by a walk over its ranges.  Before and after: 202 to 180 us (quadrupole,
// 200,003 particles; 1,487 to 1,400 instructions a wave), 536 to 357 us (monopole with the potential, 16 systems
// of 535 k particles together; 1,063 to 900 instructions, and the walk's loads).
//
// The inner loops are plain FP32 VALU code (v_sub / v_fma / v_mul) with the
// hardware reciprocal square root; pairwise forces are not a dense
// contraction, so no MFMA.
#pragma once

#include "gc_internal.h"
#include "mem_dev.h"

namespace gc {
namespace dev {

__device__ __forceinline__ void wave_sync() {
  // Lanes of one wavefront exchange data through wavefront-private LDS; the
  // LDS unit executes a wavefront's instructions in order, so only compiler
  // reordering must be prevented here.
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Six data-parallel moves: within a row of 16 lanes, then row 0 into 1 and 2 into 3, then rows 0-1 into 2-3.
__device__ __forceinline__ int wave_excl_scan(int v, int* total) {
  int inc = v;
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x111, 0xf, 0xf, true);   // row_shr 1
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x112, 0xf, 0xf, true);   // row_shr 2
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x114, 0xf, 0xf, true);   // row_shr 4
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x118, 0xf, 0xf, true);   // row_shr 8
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x142, 0xa, 0xf, false);  // lane 15 of the row before
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x143, 0xc, 0xf, false);  // lane 31
  *total = __builtin_amdgcn_readlane(inc, 63);
  return inc - v;
}

// ceil(2^16 / h) for a uniform h of 1 to 64: floor(x / h) = x * that >> 16 for every x <= 64 and for every multiple
// of 64 up to 1,024 (all checked).  65535.5 / h is at least 0.5 / h away from an integer, far beyond the
// reciprocal's rounding, so its floor is that of 65535 / h.
__device__ __forceinline__ uint32_t recip16(int h) {
  return (uint32_t)uniform((int)(65535.5f * __builtin_amdgcn_rcpf((float)h)) + 1);
}

// The records of up to 64 ranges, flattened: this lane's range has `n` records from record b, the first of them at flat
// position o.  flat_table writes, for the non-empty ranges in order, the record of flat position 0 as if the range
// reached back there; flat_record then gives the record at position first + lane: the ranges that start after
// `first` mark the place before their start, so the marks below a lane count the starts up to its own
// place.  About 12 vector instructions each (a binary search over the offsets in LDS took 55 and six
// dependent reads).  Positions past the last range give the last one's continuation (not read).
// slots: 128 words of LDS.
__device__ __forceinline__ void flat_table(int* slots, int o, int n, int b) {
  const uint64_t full = __ballot(n > 0);
  const int k = __builtin_amdgcn_mbcnt_hi((uint32_t)(full >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)full, 0u));
  wave_sync();
  if (n > 0) slots[64 + k] = b - o;
}
__device__ __forceinline__ int flat_record(int* slots, int o, int n, int first) {
  const int lane = threadIdx.x & 63;
  const int rel = o - first;
  const int base = __popcll(__ballot(n > 0 && rel <= 0)) - 1;
  slots[lane] = 0;
  wave_sync();
  if (n > 0 && (unsigned)(rel - 1) < 64u) slots[rel - 1] = 1;
  wave_sync();
  const uint64_t m = __ballot(slots[lane] != 0);
  const int e = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)base));
  const int at0 = slots[64 + e];
  wave_sync();
  return at0 + first + lane;
}

// Sum over a tile of C pair/monopole records per slice: p = records of this lane's slice.
__device__ __forceinline__ void tile_pairs(const float4* __restrict__ p, int C, float xi, float yi, float zi,
                                           float eps2, float& ax, float& ay, float& az) {
  int k = 0;
  for (; k + 4 <= C; k += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float4 j = p[k + u];
      float dx = j.x - xi, dy = j.y - yi, dz = j.z - zi;
      float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
      float ri = __builtin_amdgcn_rsqf(r2);
      float mr = j.w * ri;
      float ri2 = ri * ri;
      float sc = mr * ri2;
      ax = __builtin_fmaf(dx, sc, ax);
      ay = __builtin_fmaf(dy, sc, ay);
      az = __builtin_fmaf(dz, sc, az);
    }
  }
  for (; k < C; ++k) {
    float4 j = p[k];
    float dx = j.x - xi, dy = j.y - yi, dz = j.z - zi;
    float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
    float ri = __builtin_amdgcn_rsqf(r2);
    float mr = j.w * ri;
    float ri2 = ri * ri;
    float sc = mr * ri2;
    ax = __builtin_fmaf(dx, sc, ax);
    ay = __builtin_fmaf(dy, sc, ay);
    az = __builtin_fmaf(dz, sc, az);
  }
}

// Quadrupole node records in LDS, with l = Szz: (com, M), -7.5 (Sxx - l, Syy - l, Sxy, Sxz),
// (-7.5 Syz, 1.5 T - 4.5 l, 7.5 l eps^2, 0).  Taking l I out of the second moments leaves a matrix without a
// zz element, and its part of the force is along d, d.d being r^2 - eps^2; the sums of r^-5 S' d are
// scaled by -0.4 = 3 / -7.5 once a tile.  30 vector instructions a term where the plain form
// -M d r^-3 + 3 S d r^-5 + 1.5 T d r^-5 - 7.5 (d.S.d) d r^-7 took 32.
struct QuadTerm {
  float dx, dy, dz, ri, r3, r5, sx, sy, sz, t, cf;
  __device__ __forceinline__ QuadTerm(const float4 a, const float4 b, const float4 c, float xi, float yi, float zi,
                                      float eps2) {
    dx = xi - a.x, dy = yi - a.y, dz = zi - a.z;
    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
    ri = __builtin_amdgcn_rsqf(r2);
    const float q = ri * ri;
    r3 = ri * q;
    r5 = r3 * q;
    sx = __builtin_fmaf(b.w, dz, __builtin_fmaf(b.z, dy, b.x * dx));
    sy = __builtin_fmaf(c.x, dz, __builtin_fmaf(b.y, dy, b.z * dx));
    sz = __builtin_fmaf(c.x, dy, b.w * dx);
    t = __builtin_fmaf(dz, sz, __builtin_fmaf(dy, sy, __builtin_fmaf(dx, sx, c.z)));
    cf = r3 * __builtin_fmaf(q, __builtin_fmaf(q, t, c.y), -a.w);
  }
};

__device__ __forceinline__ void quad_term(const float4 a, const float4 b, const float4 c, float xi, float yi, float zi,
                                          float eps2, float& ax, float& ay, float& az, float& bx, float& by,
                                          float& bz) {
  const QuadTerm g(a, b, c, xi, yi, zi, eps2);
  ax = __builtin_fmaf(g.cf, g.dx, ax);
  ay = __builtin_fmaf(g.cf, g.dy, ay);
  az = __builtin_fmaf(g.cf, g.dz, az);
  bx = __builtin_fmaf(g.r5, g.sx, bx);
  by = __builtin_fmaf(g.r5, g.sy, by);
  bz = __builtin_fmaf(g.r5, g.sz, bz);
}

__device__ __forceinline__ void tile_quads(const float4* __restrict__ p, int C, float xi, float yi, float zi,
                                           float eps2, float& ax, float& ay, float& az) {
  float bx = 0.f, by = 0.f, bz = 0.f;
#pragma unroll 2
  for (int k = 0; k < C; ++k) quad_term(p[3 * k], p[3 * k + 1], p[3 * k + 2], xi, yi, zi, eps2, ax, ay, az, bx, by, bz);
  ax = __builtin_fmaf(-0.4f, bx, ax);
  ay = __builtin_fmaf(-0.4f, by, ay);
  az = __builtin_fmaf(-0.4f, bz, az);
}

// The same tiles with the potential: ph accumulates m r^-1 (pair, monopole) and, for a quadrupole
// node, M/r + 3/2 d.S.d/r^5 - T/(2r^3), in the record's terms M r^-1 - 1/3 (1.5 T - 4.5 l) r^-3 -
// 1/5 (-7.5 d.S'd + 7.5 l eps^2) r^-5; the caller scales by -G.
__device__ __forceinline__ void tile_pairs_pot(const float4* __restrict__ p, int C, float xi, float yi, float zi,
                                               float eps2, float& ax, float& ay, float& az, float& ph) {
#pragma unroll 4
  for (int k = 0; k < C; ++k) {
    float4 j = p[k];
    float dx = j.x - xi, dy = j.y - yi, dz = j.z - zi;
    float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
    float ri = __builtin_amdgcn_rsqf(r2);
    float mr = j.w * ri;
    float ri2 = ri * ri;
    float sc = mr * ri2;
    ax = __builtin_fmaf(dx, sc, ax);
    ay = __builtin_fmaf(dy, sc, ay);
    az = __builtin_fmaf(dz, sc, az);
    ph += mr;
  }
}

__device__ __forceinline__ void tile_quads_pot(const float4* __restrict__ p, int C, float xi, float yi, float zi,
                                               float eps2, float& ax, float& ay, float& az, float& ph) {
  float bx = 0.f, by = 0.f, bz = 0.f, p3 = 0.f, p5 = 0.f;
#pragma unroll 2
  for (int k = 0; k < C; ++k) {
    const float4 a = p[3 * k], c = p[3 * k + 2];
    const QuadTerm g(a, p[3 * k + 1], c, xi, yi, zi, eps2);
    ax = __builtin_fmaf(g.cf, g.dx, ax);
    ay = __builtin_fmaf(g.cf, g.dy, ay);
    az = __builtin_fmaf(g.cf, g.dz, az);
    bx = __builtin_fmaf(g.r5, g.sx, bx);
    by = __builtin_fmaf(g.r5, g.sy, by);
    bz = __builtin_fmaf(g.r5, g.sz, bz);
    ph = __builtin_fmaf(a.w, g.ri, ph);
    p3 = __builtin_fmaf(c.y, g.r3, p3);
    p5 = __builtin_fmaf(g.t, g.r5, p5);
  }
  ax = __builtin_fmaf(-0.4f, bx, ax);
  ay = __builtin_fmaf(-0.4f, by, ay);
  az = __builtin_fmaf(-0.4f, bz, az);
  ph = __builtin_fmaf(-0.2f, p5, __builtin_fmaf(-1.f / 3.f, p3, ph));
}

// One pair or monopole term for one target (the same arithmetic as the loop above), used by the
// two-targets-per-lane tile below.
__device__ __forceinline__ void pair_term(const float4 j, float xi, float yi, float zi, float eps2, float& ax,
                                          float& ay, float& az) {
  float dx = j.x - xi, dy = j.y - yi, dz = j.z - zi;
  float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
  float ri = __builtin_amdgcn_rsqf(r2);
  float mr = j.w * ri;
  float ri2 = ri * ri;
  float sc = mr * ri2;
  ax = __builtin_fmaf(dx, sc, ax);
  ay = __builtin_fmaf(dy, sc, ay);
  az = __builtin_fmaf(dz, sc, az);
}

// Terms per lane summed in FP32 before they are added into the FP64 sums of a target chunk.
constexpr int kFlushTerms = 64;

// Two targets per lane: each record read from LDS serves both (half the LDS reads per interaction,
// two independent dependency chains per lane).
struct Acc2 {
  float ax, ay, az, bx, by, bz;
};

__device__ __forceinline__ void tile_pairs2(const float4* __restrict__ p, int C, const float3 A, const float3 B,
                                            float eps2, Acc2& r) {
  int k = 0;
  for (; k + 2 <= C; k += 2) {
    const float4 j0 = p[k], j1 = p[k + 1];
    pair_term(j0, A.x, A.y, A.z, eps2, r.ax, r.ay, r.az);
    pair_term(j0, B.x, B.y, B.z, eps2, r.bx, r.by, r.bz);
    pair_term(j1, A.x, A.y, A.z, eps2, r.ax, r.ay, r.az);
    pair_term(j1, B.x, B.y, B.z, eps2, r.bx, r.by, r.bz);
  }
  if (k < C) {
    const float4 j0 = p[k];
    pair_term(j0, A.x, A.y, A.z, eps2, r.ax, r.ay, r.az);
    pair_term(j0, B.x, B.y, B.z, eps2, r.bx, r.by, r.bz);
  }
}

__device__ __forceinline__ void tile_quads2(const float4* __restrict__ p, int C, const float3 A, const float3 B,
                                            float eps2, Acc2& r) {
  Acc2 s{0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < C; ++k) {
    const float4 a = p[3 * k], b = p[3 * k + 1], c = p[3 * k + 2];
    quad_term(a, b, c, A.x, A.y, A.z, eps2, r.ax, r.ay, r.az, s.ax, s.ay, s.az);
    quad_term(a, b, c, B.x, B.y, B.z, eps2, r.bx, r.by, r.bz, s.bx, s.by, s.bz);
  }
  r.ax = __builtin_fmaf(-0.4f, s.ax, r.ax);
  r.ay = __builtin_fmaf(-0.4f, s.ay, r.ay);
  r.az = __builtin_fmaf(-0.4f, s.az, r.az);
  r.bx = __builtin_fmaf(-0.4f, s.bx, r.bx);
  r.by = __builtin_fmaf(-0.4f, s.by, r.by);
  r.bz = __builtin_fmaf(-0.4f, s.bz, r.bz);
}

// A node's records as they lie in the table: monopole (com, M); quadrupole adds (Sxx, Syy, Szz, Sxy), (Sxz, Syz, T, 0).
template <int ORDER>
struct NodeRegs {
  float4 v0, v1, v2;
};

// The node table as a raw buffer (three records, 48 bytes, a node).  A load past its end returns
// zeros, so a lane without a node (index < 0) loads a zero record with no branch and no zeroing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t node_rsrc(const float4* nodes, int32_t n_nodes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float4*>(nodes), (short)0, n_nodes * 48, 0x00020000);
}

__device__ __forceinline__ float4 u4f(const __attribute__((ext_vector_type(4))) unsigned v) {
  return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
}

template <int ORDER>
__device__ __forceinline__ NodeRegs<ORDER> load_node(__amdgpu_buffer_rsrc_t nodes, int idx) {
  NodeRegs<ORDER> r;
  // (node indices are below 2^24, checked on the host: a full-rate 24-bit multiply)
  const int off = idx >= 0 ? (int)__umul24((unsigned)idx, 48u) : 0x7ffffff0;  // past the end of any node table
  r.v0 = u4f(__builtin_amdgcn_raw_buffer_load_b128(nodes, off, 0, 0));
  if (ORDER == 2) {
    r.v1 = u4f(__builtin_amdgcn_raw_buffer_load_b128(nodes, off + 16, 0, 0));
    // the third record's fourth word is padding: three words
    const __attribute__((ext_vector_type(3))) unsigned c = __builtin_amdgcn_raw_buffer_load_b96(nodes, off + 32, 0, 0);
    r.v2 = make_float4(__uint_as_float(c[0]), __uint_as_float(c[1]), __uint_as_float(c[2]), 0.f);
  } else {
    r.v1 = r.v2 = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  return r;
}

template <int ORDER>
__device__ __forceinline__ void store_node(float4* L, int e, const NodeRegs<ORDER>& r, float eps2) {
  if (ORDER == 1) {
    L[e] = r.v0;
  } else {  // the form that quad_term reads
    const float l = r.v1.z, m = 7.5f * l;
    L[3 * e] = r.v0;
    L[3 * e + 1] = make_float4(-7.5f * (r.v1.x - l), -7.5f * (r.v1.y - l), -7.5f * r.v1.w, -7.5f * r.v2.x);
    L[3 * e + 2] = make_float4(-7.5f * r.v2.y, __builtin_fmaf(-4.5f, l, 1.5f * r.v2.z), m * eps2, 0.f);
  }
}

// Nodes per lane of a node tile: a monopole node is one record and its term 13 instructions, so a tile of 64
// would cost more to stage than to sum.  Two per lane: three, the room of a quadrupole tile, take registers that
// the potential's form does not have (535 k particles in 16 systems: 398 us with two, 420 with three).  With address
// lists one: the second takes them from seven wavefronts a SIMD to six (Plummer 131,072, two targets a lane:
// 91.6 us with one, 101.3 with two; 60,000 uniform in buckets of 16: 52.8 and 60.2).
template <int ORDER, bool LISTS>
constexpr int kNodesPerLane = ORDER == 1 && !LISTS ? 2 : 1;
template <int ORDER, bool LISTS>
constexpr int kNodesPerTile = kNodesPerLane<ORDER, LISTS> * kNodeTile;

// This wavefront's entries w, w + W, ... of a task's node list (nw of them) as a raw buffer: entry e + lane is
// word (e + lane) W, and a load past the last one returns zero with no branch.  A longer list than kOneBuffer entries
// a wavefront (byte offsets below 2^31 at eight wavefronts) is read in stretches of as many.
constexpr int kOneBuffer = 1 << 25;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t idx_rsrc(const int* first, int nw, int W) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<int*>(first), (short)0, nw > 0 ? ((nw - 1) * W + 1) * 4 : 0,
                                           0x00020000);
}

// The first node tile of a task for the calling wavefront (nodes w, w + W, ... of the task's list): the
// records in registers, entries lane, lane + 64, ..., and the indices of the nodes a whole tile on.
template <int ORDER, bool LISTS>
struct NodePrefetch {
  NodeRegs<ORDER> cur[kNodesPerLane<ORDER, LISTS>];
  int idx_next[kNodesPerLane<ORDER, LISTS>];
};

// Entries e + 64 q + lane of the wavefront's nodes (nw of them): their indices, and the records of given indices.
template <int ORDER, bool LISTS>
__device__ __forceinline__ void load_idx(__amdgpu_buffer_rsrc_t il, int e, int W, int* __restrict__ idx) {
  // (the whole offset in the vector part, which alone the bounds check is certain to cover)
  const int v = ((int)(threadIdx.x & 63) + e) * W * 4;
#pragma unroll
  for (int q = 0; q < kNodesPerLane<ORDER, LISTS>; ++q)
    idx[q] = (int)__builtin_amdgcn_raw_buffer_load_b32(il, v + 64 * q * W * 4, 0, 0);
}
template <int ORDER, bool LISTS>
__device__ __forceinline__ void load_nodes(__amdgpu_buffer_rsrc_t nodes, int e, int nw,
                                           const int* __restrict__ idx, NodeRegs<ORDER>* __restrict__ r) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < kNodesPerLane<ORDER, LISTS>; ++q)
    r[q] = load_node<ORDER>(nodes, lane < nw - e - 64 * q ? idx[q] : -1);
}

template <int ORDER, bool LISTS>
__device__ __forceinline__ void node_prefetch(__amdgpu_buffer_rsrc_t nodes, const int* __restrict__ node_idx,
                                              int n_first, int n_count, NodePrefetch<ORDER, LISTS>& pf) {
  const int wid = uniform(threadIdx.x >> 6);
  const int W = blockDim.x >> 6;
  const int nw = n_count > wid ? (int)((uint32_t)(n_count - wid + W - 1) / (uint32_t)W) : 0;
  const __amdgpu_buffer_rsrc_t il = idx_rsrc(node_idx + n_first + wid, nw < kOneBuffer ? nw : kOneBuffer, W);
  int idx[kNodesPerLane<ORDER, LISTS>];
  load_idx<ORDER, LISTS>(il, 0, W, idx);
  load_idx<ORDER, LISTS>(il, kNodesPerTile<ORDER, LISTS>, W, pf.idx_next);
  load_nodes<ORDER, LISTS>(nodes, 0, nw, idx, pf.cur);
}

// Records of LDS per wavefront for a direct tile of `tile` records: the larger of a direct tile and
// a quadrupole node tile (3 records per node), plus 96 records of reduction scratch.  A tile holds a
// multiple of the slice count S and is padded to S * ceil(count / S) records, which never exceeds
// that multiple, so the padding needs no room of its own.  (The larger area also holds the 6 x 64
// FP64 sums of the two-targets reduction: 192 records.)
__host__ __device__ __forceinline__ int grav_rec_cap(int tile) {
  return tile > 3 * kNodeTile ? tile : 3 * kNodeTile;
}
// With the potential (POT) the reduction scratch holds four sums per lane: 128 records.
__host__ __device__ __forceinline__ int grav_lds_per_wave(int tile, bool pot = false) {
  return grav_rec_cap(tile) + (pot ? 128 : 96);
}

// Two targets per lane fill more of the wavefront than one for a task of n targets (n = i_count,
// at most 64 counted) when floor(64 / ceil(n / 2)) slices of lane pairs hold more than twice
// floor(64 / n) slices of single lanes (n = 6, 13, 14, 17, 18, 22, 23, 24 and 33 to 42); otherwise
// one target per lane is at least as full and reads no duplicate target.
__host__ __device__ __forceinline__ bool two_fills_more(int n) {
  n = n < 64 ? n : 64;
  return n > 0 && 64 / ((n + 1) >> 1) > 2 * (64 / n);
}

// A task as the force code reads it: the submitted fields and the first target's position in the
// record array (its packed position, or i_begin when records are read in place).
struct TaskDesc {
  int32_t i_begin, i_count, j_first, j_nranges, n_first, n_count, ibeg;
};

// One task on one workgroup of W = blockDim.x / 64 wavefronts.  Wave w takes the task's nodes
// w, w + W, ... and the w-th of W contiguous, nearly equal shares of its direct records (address
// lists: windows w, w + W, ...), so W waves share one task's lists.  Within a wave the lanes are (lane-target j) x (slice s): with
// two targets per lane (TPL 2) each lane carries targets j and j + h (h = ceil(i_count / 2)),
// otherwise (TPL 1) target j (h = i_count); S = floor(64 / h) slices.  The per-target sums are reduced across slices within each
// wave and then across the W waves, in a fixed order.  `smem` is the block's dynamic LDS of
// W * grav_lds_per_wave(tile) records; the call starts and ends with every wave of the block
// converged (it contains block barriers).  pf holds the task's first node tile when `have_pf`
// (loaded ahead by the caller), else it is loaded here.  ready() is called by every thread once the
// first node tile's loads are out and before any record is read (the records may still be being
// written).  In the last target chunk next(0) and, after a block barrier, next(1) are called by
// every thread before the cross-wave sum; next(1) may load the following task's first node tile
// into pf.  The last barrier is the caller's: it must sync the block before the LDS is reused.
// POT (one target per lane, records in position space): acc.w also receives the potential of the
// task's terms, -G times the sum above, without the target's own direct term (a target found in its
// task's direct ranges has contributed m r^-1 at r = eps, which is taken out again).
template <int ORDER, bool LISTS, int TPL, bool POT = false, class Ready, class Next>
__device__ __forceinline__ void grav_task_body(const GravArgs& a, const int t, const TaskDesc& tk,
                                          float4* __restrict__ smem, NodePrefetch<ORDER, LISTS>& pf, bool have_pf,
                                          Ready&& ready, Next&& next) {
  static_assert(TPL == 1 || TPL == 2, "one or two targets per lane");
  static_assert(!POT || (TPL == 1 && !LISTS), "the potential runs one target per lane in position space");
  constexpr int NC = POT ? 4 : 3;  // sums per target
  const int lane = threadIdx.x & 63;
  const int wid = uniform(threadIdx.x >> 6);
  const int W = blockDim.x >> 6;
  const int tile = a.tile;
  const int rec_cap = grav_rec_cap(tile);
  const int per_wave = grav_lds_per_wave(tile, POT);
  float4* L = smem + wid * per_wave;
  double* red = reinterpret_cast<double*>(L + rec_cap);
  // the direct phase's range slots (128 words) share the reduction scratch (live at different times)
  int* slots = reinterpret_cast<int*>(red);
  int* own = slots + 128;  // POT: 1 where a target is among the wave's share of its sources (64 words)
  const int ic = tk.i_count;
  // this wave's nodes; the first tile does not depend on the records, so its loads go out first
  const int nw = tk.n_count > wid ? (int)((uint32_t)(tk.n_count - wid + W - 1) / (uint32_t)W) : 0;
  const __amdgpu_buffer_rsrc_t nodes = node_rsrc(a.nodes, a.n_nodes);
  if (!have_pf) node_prefetch<ORDER, LISTS>(nodes, a.node_idx, tk.n_first, tk.n_count, pf);
  ready();
  // 64 of the task's ranges, through a raw buffer (zeros past the last); the first are loaded ahead of the node tiles, but
  // with two targets a lane, where there are no registers to hold them over those (they were spilled, and the bench's
  // step moved 574 MB for 532)
  auto load_ranges = [&](int rg) {
    const int n = tk.j_nranges - rg < 64 ? tk.j_nranges - rg : 64;
    const __amdgpu_buffer_rsrc_t ranges = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int2*>(a.ranges + tk.j_first + rg), (short)0, n > 0 ? n * 8 : 0, 0x00020000);
    const __attribute__((ext_vector_type(2))) unsigned v =
        __builtin_amdgcn_raw_buffer_load_b64(ranges, lane * 8, 0, 0);
    return make_int2((int)v[0], (int)v[1]);
  };
  int2 g0 = make_int2(0, 0);
  constexpr bool ahead = !LISTS && TPL == 1;
  if (ahead) g0 = load_ranges(0);
  for (int i0 = 0; i0 < ic; i0 += 64) {
    if (i0 > 0) node_prefetch<ORDER, LISTS>(nodes, a.node_idx, tk.n_first, tk.n_count, pf);
    const bool last = i0 + 64 >= ic;
    const int icc = ic - i0 < 64 ? ic - i0 : 64;
    constexpr bool two = TPL == 2;
    const int h = two ? (icc + 1) >> 1 : icc;
    // every division here is a multiply by a 16-bit reciprocal
    const uint32_t mh = recip16(h);
    const int S = (int)((64u * mh) >> 16);
    const uint32_t mS = recip16(S);
    const int sl = (int)(((uint32_t)lane * mh) >> 16);
    const int il = lane - sl * h;
    const int sl3 = 3 * sl;
    const bool active = sl < S;
    // tiles hold a multiple of S records, so that only a share's last tile is padded
    // (and at most kFlushTerms a slice)
    auto fit = [&](int room) {
      const int c = (int)(((uint32_t)room * mS) >> 16);
      return S * (c < kFlushTerms ? c : kFlushTerms);
    };
    const int NT = fit(kNodesPerTile<ORDER, LISTS>);  // nodes per node tile
    const int DT = fit(tile);                  // records per direct tile
    const int ib = il + h < icc ? il + h : il;  // two: second target (a copy of the first if absent)
    float3 A = make_float3(0.f, 0.f, 0.f), B = A;
    if (active) {
      const int pb = LISTS ? 0 : tk.ibeg + i0;
      const float4 r = gld(a.rec + (LISTS ? gld(a.ilist + gld(a.ioff + t) + i0 + il) : pb + il));
      A = make_float3(r.x, r.y, r.z);
      if (two) {
        const float4 q = gld(a.rec + (LISTS ? gld(a.ilist + gld(a.ioff + t) + i0 + ib) : pb + ib));
        B = make_float3(q.x, q.y, q.z);
      }
    }
    double Ax = 0.0, Ay = 0.0, Az = 0.0, Bx = 0.0, By = 0.0, Bz = 0.0, Ap = 0.0;
    // FP32 sums carried across tiles and added into the FP64 ones before they hold more than kFlushTerms terms a
    // lane (monopoles), or once they hold as many (quadrupole tiles have a third of the nodes: the stricter
    // rule's second flush a wave cost 2 %)
    Acc2 f{0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float fp = 0.f;
    int fcnt = 0;  // uniform
    auto flush = [&]() {
      Ax += f.ax; Ay += f.ay; Az += f.az;
      if (two) {
        Bx += f.bx; By += f.by; Bz += f.bz;
      }
      if (POT) Ap += fp;
      f = Acc2{0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      fp = 0.f;
      fcnt = 0;
    };
    // one tile of C <= kFlushTerms records per slice starting at L + rec_stride * sl * C: accumulate it
    auto tile_sum = [&](int C, bool quads) {
      if (ORDER == 1 ? fcnt + C > kFlushTerms : fcnt >= kFlushTerms) flush();
      if (active) {
        const float4* p = L + __mul24(quads ? sl3 : sl, C);
        if (two) {
          if (quads) tile_quads2(p, C, A, B, a.eps2, f);
          else tile_pairs2(p, C, A, B, a.eps2, f);
        } else if (POT) {
          if (quads) tile_quads_pot(p, C, A.x, A.y, A.z, a.eps2, f.ax, f.ay, f.az, fp);
          else tile_pairs_pot(p, C, A.x, A.y, A.z, a.eps2, f.ax, f.ay, f.az, fp);
        } else {
          if (quads) tile_quads(p, C, A.x, A.y, A.z, a.eps2, f.ax, f.ay, f.az);
          else tile_pairs(p, C, A.x, A.y, A.z, a.eps2, f.ax, f.ay, f.az);
        }
      }
      fcnt += C;
    };

    // ---- node terms: this wave's nodes are list entries w, w + W, ...
    for (int64_t n0 = 0; n0 < nw; n0 += kOneBuffer) {
      const int n = nw - n0 < kOneBuffer ? (int)(nw - n0) : kOneBuffer;
      const __amdgpu_buffer_rsrc_t mine = idx_rsrc(a.node_idx + tk.n_first + wid + n0 * W, n, W);
      if (n0 > 0) {
        load_idx<ORDER, LISTS>(mine, 0, W, pf.idx_next);
        load_nodes<ORDER, LISTS>(nodes, 0, n, pf.idx_next, pf.cur);
        load_idx<ORDER, LISTS>(mine, kNodesPerTile<ORDER, LISTS>, W, pf.idx_next);
      }
      // the prefetched indices are those of a whole tile on; with NT below that the next tile starts at
      // node NT.  A tile is read up to S * C <= NT records, and past its last node it holds zero records
      // (entries past NT are the next tile's first ones, not read in this one)
      if (NT < kNodesPerTile<ORDER, LISTS>) load_idx<ORDER, LISTS>(mine, NT, W, pf.idx_next);
      for (int nb = 0; nb < n; nb += NT) {
        const int cnt = n - nb < NT ? n - nb : NT;
        const int C = uniform((int)((uint32_t)(cnt + S - 1) / (uint32_t)S));
#pragma unroll
        for (int q = 0; q < kNodesPerLane<ORDER, LISTS>; ++q) store_node<ORDER>(L, 64 * q + lane, pf.cur[q], a.eps2);
        // prefetch the next tile's records and the indices of the one after
        if (nb + NT < n) {
          load_nodes<ORDER, LISTS>(nodes, nb + NT, n, pf.idx_next, pf.cur);
          load_idx<ORDER, LISTS>(mine, nb + 2 * NT, W, pf.idx_next);
        }
        wave_sync();
        // monopole: a = -M d / r^3 with d = x_i - com, the same as a pair term from a source at com
        tile_sum(C, ORDER == 2);
        wave_sync();
      }
    }

    // ---- direct terms
    if (POT) own[lane] = 0;
    if (LISTS) {
      const int jb = gld(a.joff + t), jn = gld(a.joff + t + 1) - jb;
      for (int ws = wid * DT; ws < jn; ws += W * DT) {
        const int cnt = jn - ws < DT ? jn - ws : DT;
        const int C = uniform((cnt + S - 1) / S);
        const int padded = S * C;
        for (int e = lane; e < padded; e += 64) {
          float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
          if (e < cnt) v = gld(a.rec + gld(a.jlist + jb + ws + e));
          L[e] = v;
        }
        wave_sync();
        tile_sum(C, false);
        wave_sync();
      }
    } else {
      // the task's ranges in groups of 64, each flattened by a wave scan; wave w takes the w-th of
      // W contiguous, nearly equal shares of every group's records, and each lane copies one flat
      // position at a time (flat_record)
      for (int rg = 0; rg < tk.j_nranges; rg += 64) {
        const int2 g = ahead && rg == 0 ? g0 : load_ranges(rg);
        int total;
        const int o = wave_excl_scan(g.y, &total);
        total = uniform(total);
        flat_table(slots, o, g.y, g.x);
        // share boundaries rounded down to multiples of S (the last share ends at the total)
        // (32-bit: a task's direct records stay below 2^28)
        const uint32_t WS = (uint32_t)(W * S);
        const int lo = uniform((int)((uint32_t)total * (uint32_t)wid / WS) * S);
        const int hi = wid + 1 == W ? total : uniform((int)((uint32_t)total * (uint32_t)(wid + 1) / WS) * S);
        for (int ws = lo; ws < hi; ws += DT) {
          const int cnt = hi - ws < DT ? hi - ws : DT;
          const int C = uniform((int)((uint32_t)(cnt + S - 1) / (uint32_t)S));
          const int padded = S * C;
          // (whole wavefronts: the last lanes of the last 64 may lie past `padded`)
          for (int e = lane; e - lane < padded; e += 64) {
            const int p = flat_record(slots, o, g.y, ws + e - lane);
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (e < cnt) {
              v = gld(a.rec + p);
              const unsigned j = (unsigned)(p - (tk.ibeg + i0));
              if (POT && j < (unsigned)icc) own[j] = 1;
            }
            L[e] = v;
          }
          wave_sync();
          tile_sum(C, false);
          wave_sync();
        }
      }
    }

    // ---- reduce: slices within the wave, then the W waves, in a fixed order.  A lane sums one component
    // of one target (word n of a slice's NC x targets words), so 64 lanes serve 21 targets at a time
    flush();
    if (two) {
      // 6 sums per lane: the tile area is free now
      double* R2 = reinterpret_cast<double*>(L);
      R2[6 * lane] = Ax; R2[6 * lane + 1] = Ay; R2[6 * lane + 2] = Az;
      R2[6 * lane + 3] = Bx; R2[6 * lane + 4] = By; R2[6 * lane + 5] = Bz;
      wave_sync();
      for (int n = lane; n < 6 * h; n += 64) {
        double v = 0.0;
        for (int s = 0; s < S; ++s) v += R2[6 * h * s + n];
        const int j = (int)(((uint32_t)n * 10923u) >> 16), k = n - 6 * j;  // n / 6 for n < 192
        const int o = 3 * (k < 3 ? j : j + h - 1) + k;                     // target j, or j + h
        if (o < 3 * icc) red[o] = v;
      }
    } else {
      if (POT) {  // (the tile area is free now, and the sums take the flags' place)
        wave_sync();
        const int self = own[lane];
        wave_sync();
        reinterpret_cast<int*>(L)[lane] = self;
      }
      red[NC * lane] = Ax;
      red[NC * lane + 1] = Ay;
      red[NC * lane + 2] = Az;
      if (POT) red[NC * lane + 3] = Ap;
      wave_sync();
      // (S > 1 only up to 32 targets: a pass over at most 128 words reads slices that no later one writes over)
      if (S > 1) {
        const int nc = NC * icc;
        for (int n = lane; n < nc; n += 64) {
          double v = 0.0;
          for (int s = 0; s < S; ++s) v += red[nc * s + n];
          wave_sync();
          red[n] = v;
        }
      }
    }
    if (last) next(0);
    __syncthreads();
    if (last) next(1);
    // wave 0: lane l holds component l & 3 of target l >> 2 (the fourth is the potential, or zero)
    if (wid == 0) {
      float* out = reinterpret_cast<float*>(a.acc + tk.i_begin + i0);
      for (int n = lane; n < 4 * icc; n += 64) {
        const int j = n >> 2, k = n & 3;
        double v = 0.0;
        if (k < NC) {
          for (int w = 0; w < W; ++w) v += reinterpret_cast<const double*>(smem + w * per_wave + rec_cap)[NC * j + k];
        }
        if (POT && k == 3) {
          // the target's own direct term, where a wave met it among its records
          int self = 0;
          for (int w = 0; w < W; ++w) self |= reinterpret_cast<const int*>(smem + w * per_wave)[j];
          if (self) v -= (double)(gld(a.rec + tk.ibeg + i0 + j).w * __builtin_amdgcn_rsqf(a.eps2));
        }
        gst(out + n, k < NC ? (float)((k == 3 ? -a.G : a.G) * v) : 0.f);
      }
    }
    if (!last) __syncthreads();
  }
}

// A task in targets-per-lane mode TPL: 1 or 2 as above; 3 chooses per task, two where they fill more
// lanes (two_fills_more), so that each form's registers are live only in its own branch.
template <int ORDER, bool LISTS, int TPL, bool POT = false, class Ready, class Next>
__device__ __forceinline__ void grav_task(const GravArgs& a, const int t, const TaskDesc& tk,
                                          float4* __restrict__ smem, NodePrefetch<ORDER, LISTS>& pf, bool have_pf,
                                          Ready&& ready, Next&& next) {
  if constexpr (TPL == 3) {
    if (two_fills_more(tk.i_count))
      grav_task_body<ORDER, LISTS, 2, POT>(a, t, tk, smem, pf, have_pf, ready, next);
    else
      grav_task_body<ORDER, LISTS, 1, POT>(a, t, tk, smem, pf, have_pf, ready, next);
  } else {
    grav_task_body<ORDER, LISTS, TPL, POT>(a, t, tk, smem, pf, have_pf, ready, next);
  }
}

}  // namespace dev
}  // namespace gc
