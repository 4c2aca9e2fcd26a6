// Device-side commit of a combined request whose tasks and lists are already on the device (from
// the list walk): validation, the per-task offsets, the union U of the request and every id's
// position in it (Sec. 3.2: the runtime keeps the request's indices sorted), the packed-space
// ranges and the longest-first launch order.  Nothing crosses to the host but a few totals.
//
// The union is built without sorting: every target and direct range leaves its end at its first id
// (the largest end, where several start there); an id is in U iff a prefix maximum of those ends lies
// past it, and a prefix sum over those flags gives its rank.  Target ranges also add +1 at their first
// id and -1 past their last into a difference array, whose prefix sum finds ids targeted twice.  Every
// prefix is block aggregates, one small scan of them, and a rescan per block.
//
// A leaf is in the lists of about 45 buckets, nearly always as the same range, so the marks are plain
// stores and a second pass replaces an end that a longer range should have left (atomically; hardly
// ever).  Atomics on one cache line are performed one at a time (about 10 ns each), so the tasks'
// maxima go to kDcLines lines, one addition per four tasks: with an atomic at both ends of every
// range and two on one line per task, k_dc_tasks took 629 us for the 26,714 tasks of Plummer 262,144.
#include "reorg_dev.h"

namespace gc {
namespace {

constexpr int kCT = 256;                 // threads per block of the id-space kernels
constexpr int kCI = 16;                  // ids per thread
constexpr int kCB = kCT * kCI;           // ids per block
constexpr int kScanT = 1024;             // threads of the one-block scans

__device__ __forceinline__ int64_t wave_sum64(int64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// One wavefront per task: a task that breaks the contract is counted and emptied; otherwise its
// target and direct counts and its cost are recorded and its ranges are marked (`mark`: x the largest
// end of a range that starts at this id, y the target difference array).
__global__ void __launch_bounds__(256) k_dc_tasks(DevCommitArgs a) {
  __shared__ int64_t s_max[4][2];  // per wavefront: direct entries, node index
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t t = (int64_t)blockIdx.x * 4 + wv;
  int64_t d = 0;
  int32_t nmax = -1;
  if (t < a.n_tasks) {
    gc_task tk = a.tasks[t];
    bool bad = tk.i_count < 0 || tk.i_begin < 0 || (int64_t)tk.i_begin + tk.i_count > a.n_ids || tk.j_nranges < 0 ||
               tk.j_first < 0 || (int64_t)tk.j_first + tk.j_nranges > a.n_ranges || tk.n_count < 0 || tk.n_first < 0 ||
               (int64_t)tk.n_first + tk.n_count > a.n_node_refs || tk.flags != 0 || tk.shift[0] != 0.f ||
               tk.shift[1] != 0.f || tk.shift[2] != 0.f;
    if (!bad) {
      for (int r = lane; r < tk.j_nranges; r += 64) {
        const int2 g = a.ranges[tk.j_first + r];
        bool b = g.x < 0 || g.y < 0 || (int64_t)g.x + g.y > a.n_ids;
        if (r > 0) {
          const int2 p = a.ranges[tk.j_first + r - 1];
          b = b || (int64_t)p.x + p.y > g.x;  // ascending and disjoint
        }
        bad = bad || b;
        d += g.y;
      }
      const int32_t* nl = a.nodes + tk.n_first;
      for (int k = lane; k < tk.n_count; k += 512) {  // (eight loads in flight)
        int32_t nd[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) nd[q] = k + 64 * q < tk.n_count ? dev::gld(nl + k + 64 * q) : -1;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          if (k + 64 * q < tk.n_count) bad = bad || nd[q] < 0 || nd[q] >= a.n_nodes;
          nmax = max(nmax, nd[q]);
        }
      }
    }
    bad = __ballot(bad) != 0ull;
    d = wave_sum64(d);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nmax = max(nmax, __shfl_xor(nmax, o, 64));
    if (bad) {
      d = 0;
      nmax = -1;
      if (lane == 0) {
        atomicAdd(reinterpret_cast<unsigned long long*>(a.tot + kDcBad), 1ull);
        tk.i_count = 0;
        tk.j_nranges = 0;
        tk.n_count = 0;
        a.tasks[t] = tk;
        a.counts[t] = make_int2(0, 0);
        a.cost[t] = 0;
      }
    } else {
      if (lane == 0) {
        a.counts[t] = make_int2(tk.i_count, (int32_t)min<int64_t>(d, INT32_MAX));
        a.cost[t] = (int64_t)tk.i_count * (31 * (int64_t)tk.n_count + 12 * d);
        if (tk.i_count > 0) {
          dev::gst(&a.mark[tk.i_begin].x, tk.i_begin + tk.i_count);
          atomicAdd(&a.mark[tk.i_begin].y, 1);
          atomicAdd(&a.mark[tk.i_begin + tk.i_count].y, -1);
        }
      }
      for (int r = lane; r < tk.j_nranges; r += 64) {
        const int2 g = a.ranges[tk.j_first + r];
        if (g.y > 0) dev::gst(&a.mark[g.x].x, g.x + g.y);
      }
    }
  }
  if (lane == 0) {
    s_max[wv][0] = d;
    s_max[wv][1] = (int64_t)nmax + 1;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    int64_t m = 0;
    for (int w = 0; w < 4; ++w) m = max(m, s_max[w][threadIdx.x]);
    atomicMax(reinterpret_cast<unsigned long long*>(a.tot + kDcTot + kDcLine * (blockIdx.x % kDcLines) + threadIdx.x),
              (unsigned long long)m);
  }
}

// After the marks, which are plain stores: where ranges of different lengths start at one id any of
// their ends may have been left, and a longer range puts its own in its place.
__global__ void __launch_bounds__(256) k_dc_longest(DevCommitArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= a.n_tasks) return;
  const int32_t* tw = reinterpret_cast<const int32_t*>(a.tasks + t);  // (refused tasks were emptied)
  const int ib = dev::gld(tw), ic = dev::gld(tw + 1), jf = dev::gld(tw + 2), jn = dev::gld(tw + 3);
  for (int r = lane; r <= jn; r += 64) {
    const int2 g = r < jn ? dev::gld(a.ranges + jf + r) : make_int2(ib, ic);
    if (g.y > 0 && dev::gld(&a.mark[g.x].x) < g.x + g.y) atomicMax(&a.mark[g.x].x, g.x + g.y);
  }
}

// Exclusive prefix maximum over the block (values >= 0; 0 before the first), and the block's maximum.
__device__ __forceinline__ int block_excl_max(int v, int* sh_wave, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(inc, d, 64);
    if (lane >= d) inc = max(inc, u);
  }
  int ex = __shfl_up(inc, 1, 64);
  if (lane == 0) ex = 0;
  if (lane == 63) sh_wave[w] = inc;
  __syncthreads();
  int m = 0;
  for (int k = 0; k < nw; ++k) {
    if (k < w) ex = max(ex, sh_wave[k]);
    m = max(m, sh_wave[k]);
  }
  __syncthreads();
  *total = m;
  return ex;
}

// Per block of kCB ids: the largest end and the sum of the target differences.
__global__ void __launch_bounds__(kCT) k_dc_bsum(DevCommitArgs a) {
  __shared__ int sh[kCT / 64];
  const int64_t i0 = (int64_t)blockIdx.x * kCB + (int64_t)threadIdx.x * kCI;
  int me = 0, st = 0;
  for (int k = 0; k < kCI; ++k)
    if (i0 + k <= a.n_ids) {
      const int2 v = a.mark[i0 + k];
      me = max(me, v.x);
      st += v.y;
    }
  int ta, tt;
  (void)block_excl_max(me, sh, &ta);
  (void)dev::block_excl_scan(st, sh, &tt);
  if (threadIdx.x == 0) {
    a.bs[2 * blockIdx.x] = ta;
    a.bs[2 * blockIdx.x + 1] = tt;
  }
}

// One block: in place, the exclusive prefix maximum (column 0) and sum (column 1) of n pairs.
__global__ void __launch_bounds__(kScanT) k_dc_scan_marks(int2* v, int32_t n) {
  __shared__ int sh[kScanT / 64];
  int end = 0, sum = 0;
  for (int64_t base = 0; base < n; base += kScanT) {
    const int64_t k = base + threadIdx.x;
    const int2 x = k < n ? v[k] : make_int2(0, 0);
    int tm, ts;
    const int em = block_excl_max(x.x, sh, &tm);
    const int es = dev::block_excl_scan(x.y, sh, &ts);
    if (k < n) v[k] = make_int2(max(end, em), sum + es);
    end = max(end, tm);
    sum += ts;
  }
}

// One block: exclusive scan in place of the blocks' U counts, and the task maxima from their lines.
__global__ void __launch_bounds__(kScanT) k_dc_scan(int32_t* v, int32_t n, int64_t* tot) {
  __shared__ int sh[kScanT / 64];
  int64_t carry = 0;
  for (int64_t base = 0; base < n; base += kScanT) {
    const int64_t k = base + threadIdx.x;
    const int x = k < n ? v[k] : 0;
    int t;
    const int ex = dev::block_excl_scan(x, sh, &t);
    if (k < n) v[k] = (int32_t)(carry + ex);
    carry += t;
  }
  if (threadIdx.x == 0) tot[kDcUnion] = carry;
  if (threadIdx.x < 64) {
    static_assert(kDcLines == 32, "one wavefront, two maxima");
    int64_t m = tot[kDcTot + kDcLine * (threadIdx.x & 31) + (threadIdx.x >> 5)];
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) m = max<int64_t>(m, __shfl_xor(m, o, 64));
    if (threadIdx.x == 0) tot[kDcMaxDirect] = m;
    if (threadIdx.x == 32) tot[kDcMaxNode] = m > 0 ? m - 1 : 0;
  }
}

// Which of this thread's ids are in U, from the scanned block aggregates (and, in the first pass, how
// many are covered by two target ranges).
template <bool EMIT>
__device__ __forceinline__ void dc_cover(const DevCommitArgs& a, int* sh) {
  const int64_t i0 = (int64_t)blockIdx.x * kCB + (int64_t)threadIdx.x * kCI;
  int2 v[kCI];
  int me = 0, st = 0;
#pragma unroll
  for (int k = 0; k < kCI; ++k) {
    v[k] = i0 + k <= a.n_ids ? a.mark[i0 + k] : make_int2(0, 0);
    me = max(me, v[k].x);
    st += v[k].y;
  }
  int tm, tt;
  int end = max(block_excl_max(me, sh, &tm), a.bs[2 * blockIdx.x]);
  int ct = dev::block_excl_scan(st, sh, &tt) + a.bs[2 * blockIdx.x + 1];
  uint32_t need = 0;
  int over = 0;
#pragma unroll
  for (int k = 0; k < kCI; ++k) {
    end = max(end, v[k].x);
    ct += v[k].y;
    if (i0 + k < a.n_ids) {
      if (end > i0 + k) need |= 1u << k;
      if (ct > 1) ++over;
    }
  }
  int tn;
  int rank = dev::block_excl_scan(__popc(need), sh, &tn);
  if (!EMIT) {
    int to;
    (void)dev::block_excl_scan(over, sh, &to);
    if (threadIdx.x == 0) {
      a.ns[blockIdx.x] = tn;
      if (to) atomicAdd(reinterpret_cast<unsigned long long*>(a.tot + kDcBadTargets), (unsigned long long)to);
    }
    return;
  }
  rank += a.ns[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kCI; ++k) {
    const int64_t id = i0 + k;
    if (id >= a.n_ids) break;
    if ((need >> k) & 1u) {
      a.pos[id] = rank;
      a.U[rank] = (int32_t)id;
      ++rank;
    } else {
      a.pos[id] = -1;
    }
  }
}

__global__ void __launch_bounds__(kCT) k_dc_need(DevCommitArgs a) {
  __shared__ int sh[kCT / 64];
  dc_cover<false>(a, sh);
}

__global__ void __launch_bounds__(kCT) k_dc_emit(DevCommitArgs a) {
  __shared__ int sh[kCT / 64];
  dc_cover<true>(a, sh);
}

// Packed-space ranges and first targets (positions in U).
__global__ void k_dc_maps(DevCommitArgs a) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < (int64_t)a.n_ranges + a.n_tasks;
       k += (int64_t)gridDim.x * blockDim.x) {
    if (k < a.n_ranges) {
      const int2 g = a.ranges[k];
      const bool ok = g.y > 0 && g.x >= 0 && (int64_t)g.x + g.y <= a.n_ids;
      a.pranges[k] = make_int2(ok ? a.pos[g.x] : 0, g.y);
    } else {
      const gc_task tk = a.tasks[k - a.n_ranges];
      a.pibeg[k - a.n_ranges] = tk.i_count > 0 ? a.pos[tk.i_begin] : 0;
    }
  }
}

// Exclusive prefixes of n pairs into two arrays (a and b; b[n], and a[n] where a_end, receive the
// totals) and the 64-bit totals.  Each block takes `span` consecutive pairs and first sums all that
// come before them itself: a chain of tiles in one block (61 us for 26,714 pairs) or a second launch
// would cost more than reading the pairs again (at most kOffsetBlocks / 2 times).
constexpr int kOffsetBlocks = 64;
__global__ void __launch_bounds__(kScanT) k_pair_offsets(const int2* __restrict__ v, int64_t n, int64_t span,
                                                         int32_t* __restrict__ a, int32_t* __restrict__ b, bool a_end,
                                                         int64_t* __restrict__ tot) {
  __shared__ int64_t part[2][kScanT / 64];
  __shared__ int sh[kScanT / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * span;
  int64_t ca = 0, cb = 0;
#pragma unroll 8
  for (int64_t k = threadIdx.x; k < first; k += kScanT) {
    const int2 x = dev::gld(v + k);
    ca += x.x;
    cb += x.y;
  }
  ca = wave_sum64(ca);
  cb = wave_sum64(cb);
  if (lane == 0) {
    part[0][w] = ca;
    part[1][w] = cb;
  }
  __syncthreads();
  ca = cb = 0;
  for (int k = 0; k < kScanT / 64; ++k) {
    ca += part[0][k];
    cb += part[1][k];
  }
  // (the offsets are 32-bit, so a tile's sums are carried modulo 2^32; the totals are not)
  int64_t sa = 0, sb = 0;
  const int64_t all_a = ca, all_b = cb;
  const int64_t last = min(first + span, n);
  for (int64_t base = first; base < last; base += kScanT) {
    const int64_t k = base + threadIdx.x;
    const int2 x = k < last ? dev::gld(v + k) : make_int2(0, 0);
    int ta, tb;
    const int ea = dev::block_excl_scan(x.x, sh, &ta);
    const int eb = dev::block_excl_scan(x.y, sh, &tb);
    if (k < last) {
      a[k] = (int32_t)(ca + ea);
      b[k] = (int32_t)(cb + eb);
    }
    ca += (uint32_t)ta;
    cb += (uint32_t)tb;
    sa += x.x;
    sb += x.y;
  }
  if (blockIdx.x == gridDim.x - 1) {
    sa = wave_sum64(sa);
    sb = wave_sum64(sb);
    __syncthreads();  // (part has been read)
    if (lane == 0) {
      part[0][w] = sa;
      part[1][w] = sb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      sa = all_a;
      sb = all_b;
      for (int k = 0; k < kScanT / 64; ++k) {
        sa += part[0][k];
        sb += part[1][k];
      }
      if (a_end) a[n] = (int32_t)sa;
      b[n] = (int32_t)sb;
      tot[0] = sa;
      tot[1] = sb;
    }
  }
}

// Longest first within each run of kLptChunk consecutive tasks, ties in task order: (cost descending, index
// ascending) keys, all distinct.  One wavefront sorts 512 of them in registers with a bitonic network (8 a lane, strides
// below 8 within a lane, the others between lanes; no barrier), and a second kernel finds each key's place
// in its run: the sum, over the up to sixteen sorted pieces, of the keys before it, by binary searches in LDS,
// four of them side by side.  (One block sorted a whole run: 49 us for the 26,714 tasks of Plummer
// 262,144, the time of the network's 91 serial steps; now 11.5 + 11.5 us.)
constexpr int kOrderKeys = 8, kOrderPiece = 64 * kOrderKeys, kOrderPieces = kLptChunk / kOrderPiece;

__device__ __forceinline__ void order_pair(unsigned long long& lo, unsigned long long& hi, bool up) {
  const unsigned long long x = lo, y = hi;
  const bool swap = (x > y) == up;
  lo = swap ? y : x;
  hi = swap ? x : y;
}

// The value of lane `lane ^ x`: by data-parallel moves for 1, 2 and 8, else through the LDS crossbar.
__device__ __forceinline__ unsigned long long order_lane_xor(unsigned long long v, int x) {
  const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
  int l, h;
  if (x == 1) {
    l = __builtin_amdgcn_update_dpp(0, lo, 0xb1, 0xf, 0xf, true);  // quad_perm 1 0 3 2
    h = __builtin_amdgcn_update_dpp(0, hi, 0xb1, 0xf, 0xf, true);
  } else if (x == 2) {
    l = __builtin_amdgcn_update_dpp(0, lo, 0x4e, 0xf, 0xf, true);  // quad_perm 2 3 0 1
    h = __builtin_amdgcn_update_dpp(0, hi, 0x4e, 0xf, 0xf, true);
  } else if (x == 8) {
    l = __builtin_amdgcn_update_dpp(0, lo, 0x128, 0xf, 0xf, true);  // row_ror 8: lane ^ 8 of 16
    h = __builtin_amdgcn_update_dpp(0, hi, 0x128, 0xf, 0xf, true);
  } else {
    return __shfl_xor(v, x, 64);
  }
  return (unsigned long long)(uint32_t)h << 32 | (uint32_t)l;
}

// Strides within a lane: entries e and e + S of lane `base / kOrderKeys`.
template <int S>
__device__ __forceinline__ void order_regs(unsigned long long (&k)[kOrderKeys], int base, int size) {
#pragma unroll
  for (int e = 0; e < kOrderKeys; ++e)
    if (!(e & S)) order_pair(k[e], k[e | S], ((base + e) & size) == 0);
}

// Costs to keys, sorted within each piece (in place).
__global__ void __launch_bounds__(256) k_dc_order(DevCommitArgs a) {
  const int64_t p0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kOrderPiece;
  if (p0 >= a.n_tasks) return;
  const int n = (int)min<int64_t>(kOrderPiece, a.n_tasks - p0);
  const int lane = threadIdx.x & 63, base = lane * kOrderKeys;
  constexpr unsigned long long kCostMax = (1ull << 51) - 1ull;
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(a.cost) + p0;
  unsigned long long k[kOrderKeys];
#pragma unroll
  for (int e = 0; e < kOrderKeys; ++e) {  // (in any order: the network sorts them; read coalesced)
    const int i = e * 64 + lane;
    k[e] = ~0ull;
    if (i < n) {
      const unsigned long long c = (unsigned long long)min<int64_t>((int64_t)keys[i], (int64_t)kCostMax);
      k[e] = ((kCostMax - c) << 13) | (unsigned long long)((p0 + i) & (kLptChunk - 1));
    }
  }
#pragma unroll
  for (int size = 2; size <= kOrderPiece; size <<= 1) {
#pragma unroll
    for (int x = 32; x > 0; x >>= 1) {
      if (2 * x * kOrderKeys > size) continue;
      const bool low = (base & (x * kOrderKeys)) == 0;
      const bool up = (base & size) == 0;  // (size >= 16: the same for all entries)
#pragma unroll
      for (int e = 0; e < kOrderKeys; ++e) {
        const unsigned long long o = order_lane_xor(k[e], x);
        k[e] = (low == up) == (o < k[e]) ? o : k[e];
      }
    }
    if (size >= 8) order_regs<4>(k, base, size);
    if (size >= 4) order_regs<2>(k, base, size);
    order_regs<1>(k, base, size);
  }
#pragma unroll
  for (int e = 0; e < kOrderKeys; ++e)  // the absent ones, the largest, are last
    if (base + e < n) keys[base + e] = k[e];
}

// Places of kPlaceThreads keys of a run.
constexpr int kPlaceThreads = 1024;
__global__ void __launch_bounds__(kPlaceThreads) k_dc_place(DevCommitArgs a) {
  __shared__ unsigned long long key[kLptChunk];
  constexpr int kBlocks = kLptChunk / kPlaceThreads;  // blocks per run
  const int64_t c0 = (int64_t)(blockIdx.x / kBlocks) * kLptChunk;
  const int n = (int)min<int64_t>(kLptChunk, a.n_tasks - c0);
  const int i = (int)(blockIdx.x % kBlocks) * kPlaceThreads + threadIdx.x;
  if (i - (int)threadIdx.x >= n) return;
  const unsigned long long* from = reinterpret_cast<const unsigned long long*>(a.cost) + c0;
  unsigned long long v[kBlocks];  // (all loads in flight)
#pragma unroll
  for (int q = 0; q < kBlocks; ++q) {
    const int e = q * kPlaceThreads + threadIdx.x;
    v[q] = e < n ? from[e] : ~0ull;
  }
#pragma unroll
  for (int q = 0; q < kBlocks; ++q) key[q * kPlaceThreads + threadIdx.x] = v[q];
  __syncthreads();
  if (i >= n) return;
  const unsigned long long mine = key[i];
  const int pieces = (n + kOrderPiece - 1) / kOrderPiece;
  int place = 0;
  for (int p = 0; p < pieces; p += 4) {
    int at[4] = {0, 0, 0, 0};
#pragma unroll
    for (int step = kOrderPiece; step > 0; step >>= 1)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // (no branch: absent keys are the largest, and a piece past the last has only those)
        const int next = at[q] + step, last = min(next, kOrderPiece) - 1;
        const bool before = key[(p + q) * kOrderPiece + last] < mine;
        at[q] = (next <= kOrderPiece) & before ? next : at[q];
      }
    place += at[0] + at[1] + at[2] + at[3];
  }
  a.order[c0 + place] = (int32_t)(c0 + (int64_t)(mine & (unsigned long long)(kLptChunk - 1)));
}

// Tasks of buckets [b0, b1) from the list walk's offsets (lists relative to bucket b0's).
__global__ void k_walk_tasks(int32_t b0, int32_t b1, const int32_t* __restrict__ bucket_node, int32_t n_nodes,
                             const int2* __restrict__ node_range, const int32_t* __restrict__ n_first,
                             const int32_t* __restrict__ r_first, gc_task* __restrict__ out) {
  const int32_t nb0 = n_first[b0], rb0 = r_first[b0];
  for (int64_t b = b0 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < b1; b += (int64_t)gridDim.x * blockDim.x) {
    gc_task t{};
    const int32_t nd = bucket_node[b];
    if (nd >= 0 && nd < n_nodes) {
      const int2 r = node_range[nd];
      t.i_begin = r.x;
      t.i_count = r.y;
    } else {
      t.i_count = -1;  // refused at commit
    }
    t.j_first = r_first[b] - rb0;
    t.j_nranges = r_first[b + 1] - r_first[b];
    t.n_first = n_first[b] - nb0;
    t.n_count = n_first[b + 1] - n_first[b];
    out[b - b0] = t;
  }
}

inline int grid_for(int64_t n, int per_block, int cap) {
  int64_t g = (n + per_block - 1) / per_block;
  return (int)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

}  // namespace

int dc_id_blocks(int32_t n_ids) { return (int)(((int64_t)n_ids + 1 + kCB - 1) / kCB); }

hipError_t launch_pair_offsets(const int2* v, int64_t n, int32_t* a, int32_t* b, bool a_end, int64_t* tot,
                               hipStream_t s) {
  const int64_t tiles = std::max<int64_t>(1, (n + kScanT - 1) / kScanT);
  const int64_t span = (tiles + kOffsetBlocks - 1) / kOffsetBlocks * kScanT;
  const int64_t grid = std::max<int64_t>(1, (n + span - 1) / span);
  hipLaunchKernelGGL(k_pair_offsets, dim3((unsigned)grid), dim3(kScanT), 0, s, v, n, span, a, b, a_end, tot);
  return hipGetLastError();
}

hipError_t launch_dev_commit(const DevCommitArgs& a, hipStream_t s) {
  const int nb = dc_id_blocks(a.n_ids);
  if (a.n_tasks > 0) hipLaunchKernelGGL(k_dc_tasks, dim3(grid_for(a.n_tasks, 4, 1 << 30)), dim3(256), 0, s, a);
  if (a.n_tasks > 0) hipLaunchKernelGGL(k_dc_longest, dim3(grid_for(a.n_tasks, 4, 1 << 30)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_dc_bsum, dim3(nb), dim3(kCT), 0, s, a);
  hipLaunchKernelGGL(k_dc_scan_marks, dim3(1), dim3(kScanT), 0, s, reinterpret_cast<int2*>(a.bs), nb);
  hipLaunchKernelGGL(k_dc_need, dim3(nb), dim3(kCT), 0, s, a);
  hipLaunchKernelGGL(k_dc_scan, dim3(1), dim3(kScanT), 0, s, a.ns, nb, a.tot);
  hipLaunchKernelGGL(k_dc_emit, dim3(nb), dim3(kCT), 0, s, a);
  if ((int64_t)a.n_ranges + a.n_tasks > 0)
    hipLaunchKernelGGL(k_dc_maps, dim3(grid_for((int64_t)a.n_ranges + a.n_tasks, 256, 16384)), dim3(256), 0, s, a);
  static_assert(kDcDirect == kDcTargets + 1, "the two totals are adjacent");
  if (hipError_t e = launch_pair_offsets(a.counts, a.n_tasks, a.ioff, a.joff, false, a.tot + kDcTargets, s)) return e;
  if (a.n_tasks > 0) {
    const int64_t pieces = ((int64_t)a.n_tasks + kOrderPiece - 1) / kOrderPiece;
    const int64_t runs = ((int64_t)a.n_tasks + kLptChunk - 1) / kLptChunk;
    hipLaunchKernelGGL(k_dc_order, dim3((unsigned)((pieces + 3) / 4)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_dc_place, dim3((unsigned)(runs * (kLptChunk / kPlaceThreads))), dim3(kPlaceThreads),
                       0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_walk_tasks(int32_t b0, int32_t b1, const int32_t* bucket_node, int32_t n_nodes,
                             const int32_t* node_range, const int32_t* n_first, const int32_t* r_first, gc_task* out,
                             hipStream_t s) {
  if (b1 <= b0) return hipSuccess;
  hipLaunchKernelGGL(k_walk_tasks, dim3(grid_for(b1 - b0, 256, 4096)), dim3(256), 0, s, b0, b1, bucket_node, n_nodes,
                     reinterpret_cast<const int2*>(node_range), n_first, r_first, out);
  return hipGetLastError();
}

}  // namespace gc
