// Staging shared by the Lennard-Jones gather kernels (forces, and their adjoint): the entries of a target range and the
// search of a source among them.
#pragma once

#include "gc_internal.h"
#include "grav_dev.h"
#include "mem_dev.h"

namespace gc {
namespace dev {

constexpr int kEGroup = 32;  // entries (tasks) whose sources a wavefront stages at a time
// Up to this many target ranges a block's wavefronts share one: with a wavefront each, fewer than three would lie on
// a SIMD and each would wait for its own loads.  Measured at 216, 2,197 and 4,096 cells of 18 atoms: 9.1, 14.4 and
// 20.9 us shared, 18.9, 19.1 and 19.0 us alone; the adjoint 16.1, 31.4 and 49.8 shared, 36.0, 42.0 and 43.9 alone.
constexpr int kGSplit = 3000;
constexpr float kFar = 1e18f;  // padding sources: r^2 ~ 3e36, finite and outside any cutoff

// The bounding interval of a coordinate over the wavefront's lanes with a target (a NaN counts as none; kFar to -kFar
// if there is none).  Taken on ordered integers, whose minimum and maximum fold into the lane moves: floats need
// a move and two quieting instructions for each (150 instructions for three coordinates against 50).
__device__ __forceinline__ int ordered(float x) {
  const int b = __float_as_int(x);
  return b ^ ((b >> 31) & 0x7fffffff);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ void fold_interval(int& lo, int& hi) {
  // (a lane without a source takes the operation's neutral value, so each line is one instruction)
  const int l = __builtin_amdgcn_update_dpp(0x7fffffff, lo, CTRL, ROWS, 0xf, false);
  const int h = __builtin_amdgcn_update_dpp((int)0x80000000, hi, CTRL, ROWS, 0xf, false);
  lo = l < lo ? l : lo;
  hi = h > hi ? h : hi;
}
__device__ __forceinline__ void wave_interval(float x, bool active, float& low, float& high) {
  const bool in = active && x == x;
  const int o = ordered(x);
  int lo = in ? o : ordered(kFar), hi = in ? o : ordered(-kFar);
  fold_interval<0x111, 0xf>(lo, hi);
  fold_interval<0x112, 0xf>(lo, hi);
  fold_interval<0x114, 0xf>(lo, hi);
  fold_interval<0x118, 0xf>(lo, hi);
  fold_interval<0x142, 0xa>(lo, hi);
  fold_interval<0x143, 0xc>(lo, hi);
  lo = __builtin_amdgcn_readlane(lo, 63);
  hi = __builtin_amdgcn_readlane(hi, 63);
  low = __int_as_float(lo ^ ((lo >> 31) & 0x7fffffff));
  high = __int_as_float(hi ^ ((hi >> 31) & 0x7fffffff));
}

// A wavefront's LDS tables over the non-empty entries of a group, in order.
struct EntryTable {
  float4 sh[kEGroup], to[kEGroup];  // source-side and target-side shifts
  int rec[kEGroup];                 // record of flat source 0, as if the entry reached back there
  int id[kEGroup];                  // its id (the adjoint's)
  int mark[64];
};

// This lane's entry of a group: the flat position of its first source and its sources; `total` sources and whether any
// entry has a shift are the group's.
struct EntryGroup {
  int off, n, total;
  bool shifted;
};

// A target range is on side 0 (the task's i range: its sources are the j atoms at x_j + b) or side 1 (its j
// range: sources x_i - a) of each of its tasks, with a = max(shift, 0), b = min(shift, 0).
template <bool IDS>
__device__ __forceinline__ EntryGroup load_entries(const LJArgs& a, int first, int count, EntryTable& T) {
  const int lane = threadIdx.x & 63;
  const int32_t* tw0 = reinterpret_cast<const int32_t*>(a.tasks);
  constexpr int kTaskWords = sizeof(gc_task) / 4;
  EntryGroup g{0, 0, 0, false};
  int sb = 0, sid = 0;
  float4 sh = make_float4(0.f, 0.f, 0.f, 0.f), to = sh;
  if (lane < count) {
    const int en = gld(a.ent + first + lane);
    const int t = en >> 1;
    const int32_t* w = tw0 + (int64_t)t * kTaskWords;
    const float s0 = __int_as_float(gld(w + 7)), s1 = __int_as_float(gld(w + 8)), s2 = __int_as_float(gld(w + 9));
    const float4 ma = make_float4(s0 > 0.f ? -s0 : -0.f, s1 > 0.f ? -s1 : -0.f, s2 > 0.f ? -s2 : -0.f, 0.f);
    const float4 mb = make_float4(s0 < 0.f ? s0 : 0.f, s1 < 0.f ? s1 : 0.f, s2 < 0.f ? s2 : 0.f, 0.f);
    if (en & 1) {
      sb = a.ibeg ? gld(a.ibeg + t) : gld(w);
      if (IDS) sid = gld(w);
      g.n = gld(w + 1);
      sh = ma;
      to = mb;
    } else {
      const int jf = gld(w + 2);
      const int2 jr = gld(a.ranges + jf);
      sb = jr.x;
      if (IDS) sid = gld(a.ranges_id + jf).x;
      g.n = jr.y;
      sh = mb;
      to = ma;
    }
  }
  g.n = g.n > 0 ? g.n : 0;
  g.off = wave_excl_scan(g.n, &g.total);
  g.total = uniform(g.total);
  g.shifted = __ballot(sh.x != 0.f || sh.y != 0.f || sh.z != 0.f || to.x != 0.f || to.y != 0.f || to.z != 0.f) != 0ull;
  const uint64_t full = __ballot(g.n > 0);
  const int k = __builtin_amdgcn_mbcnt_hi((uint32_t)(full >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)full, 0u));
  if (g.n > 0) {
    T.rec[k] = sb - g.off;
    if (IDS) T.id[k] = sid - g.off;
    if (g.shifted) {
      T.sh[k] = sh;
      T.to[k] = to;
    }
  }
  wave_sync();
  return g;
}

// The entry (among the non-empty ones) of flat source `first + lane`: entries that start after `first` mark the place
// before their start, so the marks below a lane count the starts up to its own place.  (Places past the total give
// the last entry.)
__device__ __forceinline__ int entry_at(const EntryGroup& g, int first, EntryTable& T) {
  const int lane = threadIdx.x & 63;
  const int base = __popcll(__ballot(g.n > 0 && g.off <= first)) - 1;
  const unsigned place = (unsigned)(g.off - first - 1);
  T.mark[lane] = 0;
  wave_sync();
  if (g.n > 0 && place < 64u) T.mark[place] = 1;
  wave_sync();
  const uint64_t m = __ballot(T.mark[lane] != 0);
  wave_sync();
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)base));
}

// Squared distance of a point from a box.  (A coordinate that is not a number counts as no distance, so such a source is
// kept, and its pairs are evaluated: atoms that it is listed with become NaN rather than go on without it.)
__device__ __forceinline__ float box_d2(float px, float py, float pz, float blx, float bly, float blz, float bhx,
                                        float bhy, float bhz) {
  const float dx = fmaxf(fmaxf(blx - px, px - bhx), 0.f), dy = fmaxf(fmaxf(bly - py, py - bhy), 0.f),
              dz = fmaxf(fmaxf(blz - pz, pz - bhz), 0.f);
  return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
}

}  // namespace dev
}  // namespace gc
