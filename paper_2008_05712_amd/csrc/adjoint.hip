// Adjoint (vector-Jacobian product) of the combined force pass for
// L = sum_i cot_i . a_i, recomputing every pair term (nothing is stored by
// the forward pass).
//
// Gravity (direct + monopole nodes).  With u = x_j - x_i, s^2 = |u|^2 + eps^2:
//   w = G m_j [g_i / s^3 - 3 (g_i . u) u / s^5];  dL/dx_j += w, dL/dx_i -= w,
//   dL/dm_j += G (g_i . u) / s^3   (the i = j term is skipped)
// and for a node with d = x_i - com, r^2 = |d|^2 + eps^2:
//   v = -G M [g_i / r^3 - 3 (g_i . d) d / r^5];  dL/dx_i += v, dL/dcom -= v,
//   dL/dM += -G (g_i . d) / r^3.
// and with quadrupole nodes (S the raw second moment, T = tr S, q = d.S.d) also
//   d(g.a_q)/dd = G [3 S g / r^5 - 15 (g.Sd) d / r^7 - 15 (g.d) S d / r^7 - 15/2 q g / r^7
//                    + 105/2 q (g.d) d / r^9 + 3/2 T g / r^5 - 15/2 T (g.d) d / r^7]  (to x_i, minus to com),
//   H = sym(dL/dS) = G [3/2 (g d^T + d g^T) / r^5 - 15/2 (g.d) d d^T / r^7 + 3/2 (g.d) I / r^5].
// Node gradients reach member particles through com = sum m_k x_k / M, M = sum m_k and
// S = sum m_k e_k e_k^T (e_k = x_k - com):  dL/dx_k += (m_k / M) dL/dcom + 2 m_k H e_k,
// dL/dm_k += dL/dM + e_k . dL/dcom / M + e_k . H e_k.
//
// The quadrupole term is evaluated through the traceless Q = 3 S - T I: with s = Q d, q' = d.s - T eps^2,
//   a_q = G [s / r^5 - 5/2 q' d / r^7]   (the same function: d.d = r^2 - eps^2),
//   d(g.a)/dd / G = (-M / r^3 - 5/2 q' / r^7) g + Q g / r^5 - 5 (g.d) / r^7 s
//                   + (3 M (g.d) / r^5 - 5 (g.s) / r^7 + 35/2 q' (g.d) / r^9) d.
//
// Schedule: one workgroup per item, a run of consecutive tasks (or a stretch of one long task's
// sources) whose distinct nodes, or direct sources, fit an LDS table of gradients.  Consecutive tasks
// share most of their sources (16 tasks of a Plummer sphere visit 1,120 distinct nodes, 690 each), so
// the table is written out once per item as one record per distinct source instead of one per visit:
// about 2 M records of 48 bytes for 18.4 M node visits, 2.3 M of 16 for 9.3 M direct ones.  Each
// wavefront owns a stretch of the table and walks, task by task, the sources of its stretch, so the
// table takes plain LDS reads and writes (LDS float atomics, about 160 cycles per wavefront here, made
// the kernel four times slower) and every sum has a fixed order.  Lanes are sources; the loop runs over
// blocks of kTB targets in scalar registers, whose gradients stay in vector registers over the
// stretch, are reduced across the wavefront and added with FP32 atomics (order-dependent rounding).
// The records are gathered through per-node and per-particle indices and summed; the node sums reach
// the member particles through the chain.  Bound by FP32 VALU issue: about 82 instructions per
// (target, quadrupole node) pair and 26 per direct one.
//
// Lennard-Jones: h_i = g_i / m_i, dh = h_i - h_j, p = dh . d, f' = df/d(r^2):
//   dL/dx_i += f dh + 2 f' p d, dL/dx_j -= the same,
//   dL/deps_ij = p f / eps_ij,  dL/dsigma_ij = p * 24 eps (24 s^11 r^-14 - 6 s^5 r^-8),
//   chained to the per-type parameters through Lorentz-Berthelot mixing;
//   dL/dm_i = -g_i . F_i / m_i^2 with the forces F recomputed here.
// When the batch's target ranges are equal or disjoint, the gather form runs: as the forward gather
// form, one wavefront per target cell over every task touching it from either side.  The pair term
// is the same from both sides: with e the separation seen from the target and h_t, h_s the target's
// and the source's g / m, the target takes f (h_t - h_s) + 2 f' ((h_t - h_s) . e) e, and each side
// adds half of the pair's parameter derivatives.
#include "gc_internal.h"
#include "grav_dev.h"
#include "lj_dev.h"
#include "mem_dev.h"

#include <type_traits>

namespace gc {
namespace {

using dev::gld;
using dev::gld_xyz;
using dev::gst;

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Targets per block: their positions and cotangents take 48 scalar registers (12 targets: 647 against 613 us
// on Plummer 262,144, scalar registers spilled; 4: 677 us).
constexpr int kTB = 8;

typedef const __attribute__((address_space(4))) uint32_t* cst_words;

// A 16-byte record at a uniform index, by scalar loads.
__device__ __forceinline__ float4 scalar_rec(const float4* p, int64_t k) {
  cst_words q = (cst_words)(const void*)(p + k);
  return make_float4(__uint_as_float(q[0]), __uint_as_float(q[1]), __uint_as_float(q[2]), __uint_as_float(q[3]));
}
__device__ __forceinline__ int scalar_word(const void* p, int64_t k) { return (int)((cst_words)p)[k]; }

// A block of targets: positions and cotangents in scalar registers (the same for every lane, and for every
// chunk of the task's sources), gradient sums per lane.
struct AdjTargets {
  float x[kTB], y[kTB], z[kTB], gx[kTB], gy[kTB], gz[kTB];
  float tx[kTB], ty[kTB], tz[kTB];
};

// f(integral_constant K) for K = 0 .. tb - 1 (uniform), every K a compile-time index.
template <int K, class F>
__device__ __forceinline__ void each_target(int tb, F&& f) {
  if constexpr (K < kTB) {
    if (K < tb) {
      f(std::integral_constant<int, K>{});
      each_target<K + 1>(tb, f);
    }
  }
}

__device__ __forceinline__ float half_sums(float a, float b) {  // lanes below 32: a's half sums, above: b's
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float quarter_sums(float a, float b) {  // rows 0, 2: a's, rows 1, 3: b's
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int CTRL>
__device__ __forceinline__ float row_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// The block's target gradients summed over the wavefront and added to gpos, times `scale`.  Four targets
// at a time are folded into one register (each lane swap and addition halves what is left of two values),
// so that row r of 16 lanes holds target 4 h + r: 60 operations for eight targets, 240 one by one.
__device__ __forceinline__ void add_targets(const AdjTargets& T, int tb, float scale, float4* gpos) {
  const int lane = threadIdx.x & 63, h = lane & 15;
  float v[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float* t = c == 0 ? T.tx : c == 1 ? T.ty : T.tz;
#pragma unroll
    for (int q = 0; q < kTB / 4; ++q) {
      float s = quarter_sums(half_sums(t[4 * q], t[4 * q + 2]), half_sums(t[4 * q + 1], t[4 * q + 3]));
      s = row_add<0x128>(s);  // row_ror 8, 4, 2, 1
      s = row_add<0x124>(s);
      s = row_add<0x122>(s);
      s = row_add<0x121>(s);
      v[c] = h == q ? s : v[c];
    }
  }
  const int k = 4 * h + (lane >> 4);
  if (h < kTB / 4 && k < tb) {
    unsafeAtomicAdd(&gpos[k].x, scale * v[0]);
    unsafeAtomicAdd(&gpos[k].y, scale * v[1]);
    unsafeAtomicAdd(&gpos[k].z, scale * v[2]);
  }
}

// What a lane holds of its source: a node (Q and T eps^2 with quadrupoles) or a direct source.
template <int ORDER>
struct AdjSource {
  float4 c;                                 // (com, M), or (x, y, z, m)
  float qxx, qyy, qzz, qxy, qxz, qyz, te;
  int pos;                                  // direct: position in the records (-1: none)
  int slot;                                 // place in the item's table (-1: none)

  // the record as it is in the table: Sxx Syy Szz Sxy Sxz Syz T in the second moments' places
  __device__ __forceinline__ void load_node(const float4* nodes, int node) {
    const float4* nd = nodes + 3 * (int64_t)node;
    c = gld(nd);
    if (ORDER == 2) {
      const float4 s1 = gld(nd + 1), s2 = gld_xyz(nd + 2);
      qxx = s1.x; qyy = s1.y; qzz = s1.z; qxy = s1.w;
      qxz = s2.x; qyz = s2.y; te = s2.z;
    }
  }
  __device__ __forceinline__ void prepare(float eps2) {  // (apart from the load: nothing waits for it there)
    if (ORDER == 2) {
      qxx = __builtin_fmaf(3.f, qxx, -te);
      qyy = __builtin_fmaf(3.f, qyy, -te);
      qzz = __builtin_fmaf(3.f, qzz, -te);
      qxy *= 3.f;
      qxz *= 3.f;
      qyz *= 3.f;
      te *= -eps2;
    }
  }
  __device__ __forceinline__ void none() {
    c = make_float4(0.f, 0.f, 0.f, 0.f);
    qxx = qyy = qzz = qxy = qxz = qyz = te = 0.f;
    pos = slot = -1;
  }
};

// One chunk of 64 nodes (lane = node) against one block of targets.  acc: the node's sums, without G:
// -dL/dcom (3), (g.d) / r^3, and for quadrupoles sym(dL/dS).
template <int ORDER>
__device__ __forceinline__ void adj_nodes(const AdjSource<ORDER>& S, AdjTargets& T, int tb, float eps2, float (&acc)[10]) {
  const float4 c = S.c;
  const float qxx = S.qxx, qyy = S.qyy, qzz = S.qzz, qxy = S.qxy, qxz = S.qxz, qyz = S.qyz, te = S.te;
  float hc = 0.f;
#pragma unroll
  for (int q = 0; q < 10; ++q) acc[q] = 0.f;
  each_target<0>(tb, [&](auto K) {
    constexpr int k = K;
    const float3 g = make_float3(T.gx[k], T.gy[k], T.gz[k]);
    const float dx = T.x[k] - c.x, dy = T.y[k] - c.y, dz = T.z[k] - c.z;
    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
    const float ri = __builtin_amdgcn_rsqf(r2);
    const float q = ri * ri, r3 = ri * q;
    const float gd = __builtin_fmaf(g.z, dz, __builtin_fmaf(g.y, dy, g.x * dx));
    const float mr3 = c.w * r3, b = gd * q;
    float vx, vy, vz;
    if (ORDER == 2) {
      const float r5 = r3 * q, r7 = r5 * q;
      const float sx = __builtin_fmaf(qxz, dz, __builtin_fmaf(qxy, dy, qxx * dx));
      const float sy = __builtin_fmaf(qyz, dz, __builtin_fmaf(qyy, dy, qxy * dx));
      const float sz = __builtin_fmaf(qzz, dz, __builtin_fmaf(qyz, dy, qxz * dx));
      const float dq = __builtin_fmaf(dz, sz, __builtin_fmaf(dy, sy, __builtin_fmaf(dx, sx, te)));
      const float gs = __builtin_fmaf(g.z, sz, __builtin_fmaf(g.y, sy, g.x * sx));
      const float k1 = dq * r7;
      const float cg = __builtin_fmaf(-2.5f, k1, -mr3);
      const float cd = __builtin_fmaf(-5.f, gs * r7, b * __builtin_fmaf(3.f, mr3, 17.5f * k1));
      const float t5 = gd * r5, t7 = b * r5;
      const float cw = -2.5f * t7, cs = -5.f * t7;
      const float ux = r5 * g.x, uy = r5 * g.y, uz = r5 * g.z;
      vx = __builtin_fmaf(cd, dx, __builtin_fmaf(cs, sx, cg * g.x));
      vy = __builtin_fmaf(cd, dy, __builtin_fmaf(cs, sy, cg * g.y));
      vz = __builtin_fmaf(cd, dz, __builtin_fmaf(cs, sz, cg * g.z));
      vx = __builtin_fmaf(qxz, uz, __builtin_fmaf(qxy, uy, __builtin_fmaf(qxx, ux, vx)));
      vy = __builtin_fmaf(qyz, uz, __builtin_fmaf(qyy, uy, __builtin_fmaf(qxy, ux, vy)));
      vz = __builtin_fmaf(qzz, uz, __builtin_fmaf(qyz, uy, __builtin_fmaf(qxz, ux, vz)));
      // sym(dL/dQ) = sym(d (x) w), w = g / r^5 - 5/2 (g.d) d / r^7; the trace's part is (g.d) / (2 r^5)
      const float wx = __builtin_fmaf(cw, dx, ux), wy = __builtin_fmaf(cw, dy, uy), wz = __builtin_fmaf(cw, dz, uz);
      acc[4] = __builtin_fmaf(wx, dx, acc[4]);
      acc[5] = __builtin_fmaf(wy, dy, acc[5]);
      acc[6] = __builtin_fmaf(wz, dz, acc[6]);
      acc[7] = __builtin_fmaf(wx, dy, __builtin_fmaf(wy, dx, acc[7]));
      acc[8] = __builtin_fmaf(wx, dz, __builtin_fmaf(wz, dx, acc[8]));
      acc[9] = __builtin_fmaf(wy, dz, __builtin_fmaf(wz, dy, acc[9]));
      hc += t5;
    } else {
      const float cd = 3.f * mr3 * b;
      vx = __builtin_fmaf(cd, dx, -mr3 * g.x);
      vy = __builtin_fmaf(cd, dy, -mr3 * g.y);
      vz = __builtin_fmaf(cd, dz, -mr3 * g.z);
    }
    T.tx[k] += vx;
    T.ty[k] += vy;
    T.tz[k] += vz;
    acc[0] += vx;
    acc[1] += vy;
    acc[2] += vz;
    acc[3] = __builtin_fmaf(gd, r3, acc[3]);
  });
  if (ORDER == 2) {  // dL/dS = 3 dL/dQ + dL/dT I
#pragma unroll
    for (int q = 4; q < 7; ++q) acc[q] = __builtin_fmaf(3.f, acc[q], 1.5f * hc);
#pragma unroll
    for (int q = 7; q < 10; ++q) acc[q] *= 1.5f;
  }
}

// One chunk of 64 direct sources (lane = source) against one block of targets, the first of them at position
// rec0 of the records.  acc: dL/dx (3) and dL/dm of the source, without G.
template <int ORDER>
__device__ __forceinline__ void adj_direct(const AdjSource<ORDER>& S, int rec0, AdjTargets& T, int tb, float eps2,
                                           float (&acc)[10]) {
  const float4 s = S.c;
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = 0.f;
  const int self = S.pos - rec0;  // the target this source is, if any
  each_target<0>(tb, [&](auto K) {
    constexpr int k = K;
    const float3 g = make_float3(T.gx[k], T.gy[k], T.gz[k]);
    const float dx = s.x - T.x[k], dy = s.y - T.y[k], dz = s.z - T.z[k];
    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
    // j = i is skipped (before any product: where eps^2 underflows, its 1 / r is infinite)
    const float ri = self == k ? 0.f : __builtin_amdgcn_rsqf(r2);
    const float q = ri * ri, r3 = ri * q;
    const float gd = __builtin_fmaf(g.z, dz, __builtin_fmaf(g.y, dy, g.x * dx));
    const float c1 = s.w * r3, c2 = -3.f * c1 * (gd * q);
    const float wx = __builtin_fmaf(c2, dx, c1 * g.x);
    const float wy = __builtin_fmaf(c2, dy, c1 * g.y);
    const float wz = __builtin_fmaf(c2, dz, c1 * g.z);
    T.tx[k] -= wx;
    T.ty[k] -= wy;
    T.tz[k] -= wz;
    acc[0] += wx;
    acc[1] += wy;
    acc[2] += wz;
    acc[3] = __builtin_fmaf(gd, r3, acc[3]);
  });
}

// A wavefront's position in its stretch of an item: chunk e of task t0 + k against the targets from b0.
struct AdjCursor {
  int k, b0, e, e0, e1, ic;
  int64_t flat;
};

// One item per workgroup of W wavefronts.  The table holds NV floats per
// distinct source, one array per value, for a direct source what its dL/dm lost in rounding, then the sources'
// indices.  (The mass gradients are the largest by far, and a source near 16 tasks is added to some 50 times: without that
// value their error against 64 bits was 1.58e-7 of 80,000 Plummer particles, 1.53e-7 when every visit had
// its own sum; now 1.50e-7, for 3 us of 1,100 at 262,144.)  A chunk's records are loaded while
// the one before is computed, and their places while the one before that is.
template <bool PACKED, int ORDER, bool NODES>
__device__ __forceinline__ void adj_item(const GravAdjArgs& A, const AdjItem& it, float* table) {
  constexpr int W = NODES ? kAdjNodeWaves : kAdjDirectWaves;
  constexpr int NV = NODES && ORDER == 2 ? 10 : 4;
  const int lane = threadIdx.x & 63;
  const int wid = uniform(threadIdx.x >> 6);
  const int t0 = uniform(it.t0), nt = uniform(it.nt), cap = uniform(it.count), base = uniform(it.base);
  const float G = A.f.G, eps2 = A.f.eps2;
  float* low = table + NV * cap;  // (direct)
  int* src = reinterpret_cast<int*>(table + (NODES ? NV : NV + 1) * cap);
  {
    const int32_t* from = NODES ? A.nsrc : PACKED ? A.dsrc_packed : A.dsrc_id;
    for (int k = threadIdx.x; k < (NODES ? NV : NV + 1) * cap; k += 64 * W) table[k] = 0.f;
    for (int k = threadIdx.x; k < cap; k += 64 * W) src[k] = gld(from + base + k);
  }
  __syncthreads();
  const int32_t* first = NODES ? A.noff : A.joff;
  const uint16_t* place = NODES ? A.vpos : A.dpos;
  const int32_t* cuts = (NODES ? A.ncuts : A.dcuts) + uniform(it.cuts) + wid;
  const int32_t* tw = reinterpret_cast<const int32_t*>(A.f.tasks);
  constexpr int kTaskWords = sizeof(gc_task) / 4;
  // the first chunk of the first task from k on that has any (k = nt: none)
  auto enter = [&](int k) {
    AdjCursor c{k, 0, 0, 0, 0, 0, 0};
    for (; c.k < nt; ++c.k) {
      c.e0 = scalar_word(cuts, c.k * (W + 1));
      c.e1 = scalar_word(cuts, c.k * (W + 1) + 1);
      c.ic = scalar_word(tw, (int64_t)(t0 + c.k) * kTaskWords + 1);
      if (c.e0 < c.e1 && c.ic > 0) break;
    }
    if (c.k < nt) c.flat = scalar_word(first, t0 + c.k);
    c.e = c.e0;
    return c;
  };
  auto advance = [&](AdjCursor c) {
    if (c.k >= nt) return c;
    if (c.e + 64 < c.e1) {
      c.e += 64;
    } else if (c.b0 + kTB < c.ic) {
      c.b0 += kTB;
      c.e = c.e0;
    } else {
      c = enter(c.k + 1);
    }
    return c;
  };
  auto places = [&](const AdjCursor& c) {  // this lane's place, or -1
    return c.k < nt && c.e + lane < c.e1 ? (int)place[c.flat + c.e + lane] : -1;
  };
  auto load = [&](int slot, AdjSource<ORDER>& S) {
    S.none();
    S.slot = slot;
    if (slot >= 0) {
      const int p = src[slot];
      if (NODES) {
        S.load_node(A.f.nodes, p);
      } else {
        S.c = gld(A.f.rec + p);
        S.pos = p;
      }
    }
  };
  AdjCursor cur = enter(0), n1 = advance(cur);
  AdjSource<ORDER> here, next;
  load(places(cur), here);
  int slot1 = places(n1);
  while (cur.k < nt) {
    // a block of targets
    const int t = t0 + cur.k;
    const int ib = scalar_word(tw, (int64_t)t * kTaskWords) + cur.b0;
    const int rec0 = (PACKED ? scalar_word(A.f.ibeg, t) + cur.b0 : ib);
    const int tb = cur.ic - cur.b0 < kTB ? cur.ic - cur.b0 : kTB;
    AdjTargets T;
#pragma unroll
    for (int q = 0; q < kTB; ++q) {
      const int j = q < tb ? q : tb - 1;
      const float4 x = scalar_rec(A.f.rec, rec0 + j), g = scalar_rec(A.cot, ib + j);
      T.x[q] = x.x; T.y[q] = x.y; T.z[q] = x.z;
      T.gx[q] = g.x; T.gy[q] = g.y; T.gz[q] = g.z;
      T.tx[q] = T.ty[q] = T.tz[q] = 0.f;
    }
    bool more;
    do {
      load(slot1, next);
      const AdjCursor n2 = advance(n1);
      const int slot2 = places(n2);
      here.prepare(eps2);
      float acc[10];
      if (NODES) adj_nodes<ORDER>(here, T, tb, eps2, acc);
      else adj_direct<ORDER>(here, rec0, T, tb, eps2, acc);
      if (here.slot >= 0) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          const float t = table[q * cap + here.slot], sum = t + acc[q];
          table[q * cap + here.slot] = sum;
          if (!NODES && q == 3) {
            const float b = sum - t;
            low[here.slot] += (t - (sum - b)) + (acc[q] - b);
          }
        }
      }
      more = n1.k == cur.k && n1.b0 == cur.b0;
      cur = n1;
      n1 = n2;
      slot1 = slot2;
      here = next;
    } while (more);
    add_targets(T, tb, G, A.gpos + ib);
  }
  __syncthreads();
  // one record per distinct source
  for (int u = threadIdx.x; u < cap; u += 64 * W) {
    float v[10];
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = G * table[q * cap + u];
    if (!NODES) {
      const float rest = low[u];
      if (rest == rest) v[3] = G * (table[3 * cap + u] + rest);  // (an infinite sum leaves no rest)
      gst(A.vdir + base + u, make_float4(v[0], v[1], v[2], v[3]));
    } else {
      float4* q = A.vnode + (int64_t)(ORDER == 2 ? 3 : 1) * (base + u);
      gst(q, make_float4(-v[0], -v[1], -v[2], -v[3]));
      if (ORDER == 2) {
        gst(q + 1, make_float4(v[4], v[5], v[6], v[7]));
        gst(q + 2, make_float4(v[8], v[9], 0.f, 0.f));
      }
    }
  }
}

template <bool PACKED, int ORDER, bool NODES>
__global__ void __launch_bounds__(64 * (NODES ? kAdjNodeWaves : kAdjDirectWaves)) k_grav_adj(GravAdjArgs A) {
  extern __shared__ float table[];
  adj_item<PACKED, ORDER, NODES>(A, (NODES ? A.node_items : A.direct_items)[blockIdx.x], table);
}

// Node and direct items in one launch, for batches whose items all fit the chip at once: there the two kinds
// run side by side (uniform 4,096, 540 tasks: 17 -> 11 us).  Larger batches take two launches, each with its own
// registers, LDS and wavefronts per item.  The direct items' last wavefronts only join the barriers.
template <bool PACKED, int ORDER>
__global__ void __launch_bounds__(64 * kAdjNodeWaves) k_grav_adj_both(GravAdjArgs A) {
  extern __shared__ float table[];
  static_assert(kAdjDirectWaves <= kAdjNodeWaves, "workgroup size");
  if ((int)blockIdx.x < A.n_node_items) {
    adj_item<PACKED, ORDER, true>(A, A.node_items[blockIdx.x], table);
  } else if (threadIdx.x < 64 * kAdjDirectWaves) {
    adj_item<PACKED, ORDER, false>(A, A.direct_items[blockIdx.x - A.n_node_items], table);
  } else {  // adj_item's two barriers
    __syncthreads();
    __syncthreads();
  }
}

// A node's gradient (the sum of its chunks' sums) pushed to its members:
// dx_k += (m_k / M) dL/dcom + 2 m_k H e_k, dm_k += dL/dM + e_k . dL/dcom / M + e_k.H e_k, e_k = x_k - com.
// Most nodes hold few particles and some, near the root, tens of thousands, so one wavefront takes each
// node of up to kChainSmall members, and the first blocks of the grid take the larger ones, kChainSplit
// workgroups to a node (each group of workgroups looks through every n-th window of 64 nodes for them).
// One workgroup per node, whatever its size, took 149 us for the 30,548 nodes of Plummer 262,144: idle
// wavefronts for the small nodes and a serial tail for the large; this takes 94, the rate of the atomic
// additions (four per member and level; the splits between 128 and 2,048 members differ by 8 %).
// A node whose member range is not inside [0, n_ids) is skipped and counted in *bad (its gradient is
// not pushed), so a malformed node table cannot make the member loop read or write out of bounds.
constexpr int kChainSmall = 512, kChainSplit = 8, kChainGroups = 64;

template <int NQ>
struct ChainArgs {
  const int32_t* node_range;
  int32_t n_nodes;
  const float4* nodes;
  const float4* part;
  const int32_t* chunk_first;
  const float4* rec_by_id;
  int32_t n_ids;
  float4* gpos;
  float* gmass;
  int32_t* bad;
};

template <int NQ>
__device__ __forceinline__ void chain_node(const ChainArgs<NQ>& a, int nd, int c0, int c1, int b, int n, int k0, int stride) {
  const int lane = threadIdx.x & 63;
  float gv[4 * NQ];
  if (c1 - c0 == 1) {  // (uniform)
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float4 v = gld(a.part + (int64_t)NQ * c0 + q);
      gv[4 * q] = v.x; gv[4 * q + 1] = v.y; gv[4 * q + 2] = v.z; gv[4 * q + 3] = v.w;
    }
  } else {
    float4 acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int ch = c0 + lane; ch < c1; ch += 64) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) acc[q] += gld(a.part + (int64_t)NQ * ch + q);
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      gv[4 * q] = wave_sum(acc[q].x);
      gv[4 * q + 1] = wave_sum(acc[q].y);
      gv[4 * q + 2] = wave_sum(acc[q].z);
      gv[4 * q + 3] = wave_sum(acc[q].w);
    }
  }
  const float4 c = gld(a.nodes + 3 * (int64_t)nd);
  const float invM = 1.f / c.w;
  for (int k = k0; k < n; k += stride) {
    const float4 r = gld(a.rec_by_id + b + k);
    const float f = r.w * invM;
    const float ex = r.x - c.x, ey = r.y - c.y, ez = r.z - c.z;
    float px = f * gv[0], py = f * gv[1], pz = f * gv[2];
    float dm = gv[3] + (ex * gv[0] + ey * gv[1] + ez * gv[2]) * invM;
    if constexpr (NQ == 3) {
      const float hxx = gv[4], hyy = gv[5], hzz = gv[6], hxy = gv[7], hxz = gv[8], hyz = gv[9];
      const float hx = hxx * ex + hxy * ey + hxz * ez;
      const float hy = hxy * ex + hyy * ey + hyz * ez;
      const float hz = hxz * ex + hyz * ey + hzz * ez;
      px += 2.f * r.w * hx;
      py += 2.f * r.w * hy;
      pz += 2.f * r.w * hz;
      dm += ex * hx + ey * hy + ez * hz;
    }
    float4* q = a.gpos + (b + k);
    unsafeAtomicAdd(&q->x, px);
    unsafeAtomicAdd(&q->y, py);
    unsafeAtomicAdd(&q->z, pz);
    unsafeAtomicAdd(a.gmass + (b + k), dm);
  }
}

template <int NQ>
__global__ void __launch_bounds__(256) k_node_chain(ChainArgs<NQ> a, int32_t groups) {
  const int lane = threadIdx.x & 63;
  if ((int)blockIdx.x < groups * kChainSplit) {  // nodes of more than kChainSmall members
    const int grp = blockIdx.x / kChainSplit, share = blockIdx.x - grp * kChainSplit;
    for (int64_t w0 = 64 * (int64_t)grp; w0 < a.n_nodes; w0 += 64 * (int64_t)groups) {
      const int64_t nd = w0 + lane;
      int c0 = 0, c1 = 0;
      int2 r = make_int2(0, 0);
      if (nd < a.n_nodes) {
        c0 = gld(a.chunk_first + nd);
        c1 = gld(a.chunk_first + nd + 1);
        r = make_int2(gld(a.node_range + 2 * nd), gld(a.node_range + 2 * nd + 1));
      }
      const bool large = c0 < c1 && r.y > kChainSmall && r.x >= 0 && r.x <= a.n_ids - r.y;
      for (uint64_t m = __ballot(large); m; m &= m - 1) {
        const int j = __builtin_ctzll(m);
        chain_node<NQ>(a, (int)(w0 + j), __builtin_amdgcn_readlane(c0, j), __builtin_amdgcn_readlane(c1, j),
                       __builtin_amdgcn_readlane(r.x, j), __builtin_amdgcn_readlane(r.y, j),
                       share * 256 + (int)threadIdx.x, 256 * kChainSplit);
      }
    }
    return;
  }
  const int64_t nd = ((int64_t)blockIdx.x - groups * kChainSplit) * 4 + uniform(threadIdx.x >> 6);
  if (nd >= a.n_nodes) return;
  const int c0 = uniform(gld(a.chunk_first + nd)), c1 = uniform(gld(a.chunk_first + nd + 1));
  if (c0 == c1) return;  // the node is in no task's list
  const int b = uniform(gld(a.node_range + 2 * nd)), n = uniform(gld(a.node_range + 2 * nd + 1));
  if (b < 0 || n < 0 || b > a.n_ids - n) {
    if (lane == 0) atomicAdd(a.bad, 1);
    return;
  }
  if (n <= kChainSmall) chain_node<NQ>(a, (int)nd, c0, c1, b, n, lane, 64);
}

// Sums of the gradient records, two kinds of workgroups in one launch.
//
// Direct records (the first blocks): one wavefront per 64 consecutive entries of the records sorted by
// source id.  A segmented inclusive scan (ids are sorted, so equal neighbours mean one run) sums each id's
// run within the wavefront, and the run's last lane adds it to the gradients.  A particle whose records
// span several wavefronts gets one addition from each, so no lane walks a long list.
//
// Node records: one wavefront per chunk of a node's records (at most kVisitChunk), lanes striding the
// chunk, reduced across the wavefront in a fixed order.
struct SumArgs {
  const float4* vdir;
  const int32_t* dvis;
  const int32_t* dkey;
  int32_t n_direct;
  float4* gpos;
  float* gmass;
  const float4* vnode;
  const int32_t* nvis;
  const int2* chunks;
  int32_t n_chunks;
  float4* part;
};

template <int NQ>
__global__ void __launch_bounds__(256) k_record_sums(SumArgs a, int32_t direct_blocks) {
  const int lane = threadIdx.x & 63;
  if ((int)blockIdx.x < direct_blocks) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < a.n_direct;
    int key = valid ? gld(a.dkey + i) : -1 - lane;  // distinct negative keys: past-the-end lanes form no run
    float4 v = valid ? gld(a.vdir + gld(a.dvis + i)) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int ku = __shfl_up(key, d, 64);
      const float ux = __shfl_up(v.x, d, 64), uy = __shfl_up(v.y, d, 64), uz = __shfl_up(v.z, d, 64),
                  uw = __shfl_up(v.w, d, 64);
      if (lane >= d && ku == key) {
        v.x += ux;
        v.y += uy;
        v.z += uz;
        v.w += uw;
      }
    }
    const int kn = __shfl_down(key, 1, 64);
    if (valid && (lane == 63 || kn != key)) {
      float4* q = a.gpos + key;
      unsafeAtomicAdd(&q->x, v.x);
      unsafeAtomicAdd(&q->y, v.y);
      unsafeAtomicAdd(&q->z, v.z);
      unsafeAtomicAdd(a.gmass + key, v.w);
    }
    return;
  }
  const int ch = uniform(((int)blockIdx.x - direct_blocks) * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6));
  if (ch >= a.n_chunks) return;
  const int2 r = gld(a.chunks + ch);
  float4 acc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int i = r.x + lane; i < r.y; i += 64) {
    const float4* v = a.vnode + (int64_t)NQ * gld(a.nvis + i);
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] += gld(v + q);
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const float4 t = make_float4(wave_sum(acc[q].x), wave_sum(acc[q].y), wave_sum(acc[q].z), wave_sum(acc[q].w));
    if (lane == 0) gst(a.part + (int64_t)NQ * ch + q, t);
  }
}

// What the indices hold of an item that is one task, or a stretch of one: its visits are its records, in order, and the
// wavefronts' cuts are even.  One wavefront an item, node items first.
__global__ void __launch_bounds__(64) k_adj_items(AdjFinishArgs a) {
  const int lane = threadIdx.x;
  const bool nodes = (int)blockIdx.x < a.n_node_items;
  const AdjItem it = nodes ? a.node_items[blockIdx.x] : a.direct_items[blockIdx.x - a.n_node_items];
  const gc_task& tk = a.tasks[it.t0];
  const int e0 = it.base - (nodes ? a.noff : a.joff)[it.t0];  // the item's first visit of the task
  const int W = nodes ? kAdjNodeWaves : kAdjDirectWaves;
  if (lane <= W) (nodes ? a.ncuts : a.dcuts)[it.cuts + lane] = e0 + (int)((int64_t)it.count * lane / W);
  uint16_t* place = nodes ? a.vpos : a.dpos;
  for (int u = lane; u < it.count; u += 64) place[it.base + u] = (uint16_t)u;
  if (nodes) {
    for (int u = lane; u < it.count; u += 64) a.nsrc[it.base + u] = gld(a.nodes + tk.n_first + e0 + u);
    return;
  }
  int at = -e0;  // of a range's first source among the item's
  for (int r = 0; r < tk.j_nranges && at < it.count; ++r) {
    const int2 g = gld(a.ranges + tk.j_first + r);
    const int u1 = it.count - at < g.y ? it.count - at : g.y;
    for (int u = (at < 0 ? -at : 0) + lane; u < u1; u += 64) a.dsrc_id[it.base + at + u] = g.x + u;
    at += g.y;
  }
}

// The direct records' positions in the union, and the ids of the sorted ones.
__global__ void __launch_bounds__(256) k_adj_keys(AdjFinishArgs a) {
  for (int64_t r = blockIdx.x * (int64_t)256 + threadIdx.x; r < a.n_direct; r += (int64_t)gridDim.x * 256) {
    const int id = gld(a.dsrc_id + r);
    int lo = 0, hi = a.n_union;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (gld(a.U + mid) < id) lo = mid + 1;
      else hi = mid;
    }
    a.dsrc_packed[r] = lo;
    a.dkey[r] = gld(a.dsrc_id + gld(a.dvis + r));
  }
}

constexpr int kMaxTypes = 8;
constexpr int kLJTile = 128;

// Per-lane accumulators of dL/deps_ij and dL/dsigma_ij keyed by the j type (the lane's i type is
// fixed within a run chunk).  NT = 1 or 2 keep them in registers; NT = 0 (up to kMaxTypes types)
// adds each pair term to LDS directly.
template <int NT>
struct ParamAcc {
  float e[NT > 0 ? NT : 1], s[NT > 0 ? NT : 1];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int k = 0; k < (NT > 0 ? NT : 1); ++k) e[k] = s[k] = 0.f;
  }
  __device__ __forceinline__ void add(int tj, float de, float ds, float* pg_row) {
    if (NT == 1) {
      e[0] += de;
      s[0] += ds;
    } else if (NT == 2) {
      const bool one = tj != 0;
      e[0] += one ? 0.f : de;
      s[0] += one ? 0.f : ds;
      e[1] += one ? de : 0.f;
      s[1] += one ? ds : 0.f;
    } else {
      atomicAdd(pg_row + 2 * tj, de);
      atomicAdd(pg_row + 2 * tj + 1, ds);
    }
  }
  // (times the row's factors, for sums that were kept without them)
  __device__ __forceinline__ void flush(float* pg_row, const float4* trow) {
    if (NT > 0) {
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        const float de = trow ? e[k] * trow[k].z : e[k], ds = trow && s[k] != 0.f ? s[k] * trow[k].w : s[k];
        if (de != 0.f) atomicAdd(pg_row + 2 * k, de);
        if (ds != 0.f) atomicAdd(pg_row + 2 * k + 1, ds);
      }
    }
    zero();
  }
};

// The block's dL/deps_ij, dL/dsigma_ij by type pair (summed over its 4 wavefronts) go to its own
// row of A.ppart with plain stores; k_lj_param_reduce sums the rows in a fixed order.  (Atomics from
// every block onto the few words of gparam, all in one cache line, serialise at one L2 channel.)
__device__ __forceinline__ void block_param_partial(const LJAdjArgs& A, const float* pg, int nt) {
  const int P = 2 * nt * nt;
  if ((int)threadIdx.x < P) {
    float v = 0.f;
    for (int w = 0; w < 4; ++w) v += pg[w * 2 * kMaxTypes * kMaxTypes + threadIdx.x];
    A.ppart[(int64_t)blockIdx.x * P + threadIdx.x] = v;
  }
}

// One block per type pair (ta, tb): the sum of the blocks' partials, chained to the per-type
// parameters through eps_ij = sqrt(eps_a eps_b), sigma_ij = (sigma_a + sigma_b) / 2.
__global__ void __launch_bounds__(256) k_lj_param_reduce(const float* __restrict__ ppart, int32_t n_blocks, int32_t nt,
                                                         const float* __restrict__ eps_t, float* __restrict__ gparam) {
  __shared__ float se[256], ss[256];
  const int k = blockIdx.x, P = 2 * nt * nt;
  float de = 0.f, ds = 0.f;
  // eight rows' loads at a time, summed in order (one at a time: 11.5 us for 9,000 rows)
  for (int b0 = threadIdx.x; b0 < n_blocks; b0 += 8 * blockDim.x) {
    float2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int b = b0 + q * (int)blockDim.x;
      v[q] = b < n_blocks ? *reinterpret_cast<const float2*>(ppart + (int64_t)b * P + 2 * k) : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      de += v[q].x;
      ds += v[q].y;
    }
  }
  se[threadIdx.x] = de;
  ss[threadIdx.x] = ds;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      se[threadIdx.x] += se[threadIdx.x + h];
      ss[threadIdx.x] += ss[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const int ta = k / nt, tb = k % nt;
    const float eij = sqrtf(eps_t[ta] * eps_t[tb]);
    unsafeAtomicAdd(gparam + ta, se[0] * eps_t[tb] / (2.f * eij));
    unsafeAtomicAdd(gparam + tb, se[0] * eps_t[ta] / (2.f * eij));
    unsafeAtomicAdd(gparam + nt + ta, 0.5f * ss[0]);
    unsafeAtomicAdd(gparam + nt + tb, 0.5f * ss[0]);
  }
}

// One wavefront per run of tasks sharing a target range (as in the forward kernel); lanes =
// (i atom) x (j slice) with a per-lane rotation over the slice's j entries.  j-side gradients and
// forces accumulate in LDS, i-side in registers across the run.
template <int NT>
__global__ void __launch_bounds__(256) k_lj_adj(LJAdjArgs A) {
  const LJArgs& a = A.f;
  __shared__ float2 tab[kMaxTypes * kMaxTypes];   // (24 eps_ij, sigma_ij)
  __shared__ float4 jt[4][kLJTile], jh[4][kLJTile];
  __shared__ float gj[4][6][kLJTile];              // j: dL/dx (3), force (3)
  __shared__ float red[4][6][64];
  __shared__ float pg[4][2 * kMaxTypes * kMaxTypes];  // per wave: dL/deps_ij, dL/dsigma_ij by type pair
  const int lane = threadIdx.x & 63;
  const int wid = uniform(threadIdx.x >> 6);
  const int nt = a.n_types;
  for (int k = threadIdx.x; k < nt * nt; k += blockDim.x) {
    int ta = k / nt, tb = k % nt;
    tab[k] = make_float2(24.f * sqrtf(a.eps_t[ta] * a.eps_t[tb]), 0.5f * (a.sig_t[ta] + a.sig_t[tb]));
  }
  for (int k = threadIdx.x; k < 4 * 2 * kMaxTypes * kMaxTypes; k += blockDim.x) (&pg[0][0])[k] = 0.f;
  __syncthreads();
  const int r = uniform(blockIdx.x * 4 + wid);
  if (r < a.n_runs) {
    const int t0 = uniform(a.runs[r]), t1 = uniform(a.runs[r + 1]);
    const gc_task tk0 = a.tasks[t0];
    const int ipos0 = a.ibeg ? a.ibeg[t0] : tk0.i_begin;
    for (int i0 = 0; i0 < tk0.i_count; i0 += 64) {
      const int icc = tk0.i_count - i0 < 64 ? tk0.i_count - i0 : 64;
      const int S = 64 / icc;
      const int il = lane % icc, sl = lane / icc;
      const bool active = sl < S;
      float xr = 0.f, yr = 0.f, zr = 0.f, hx = 0.f, hy = 0.f, hz = 0.f;
      int ti = 0;
      if (active) {
        float4 rr = a.rec[ipos0 + i0 + il];
        xr = rr.x; yr = rr.y; zr = rr.z;
        ti = (int)rr.w;
        float4 g = A.cot[tk0.i_begin + i0 + il];
        float m = A.mass_t[ti];
        hx = g.x / m; hy = g.y / m; hz = g.z / m;
      }
      float* pg_row = &pg[wid][2 * ti * nt];
      ParamAcc<NT> pa;
      pa.zero();
      float Gx = 0.f, Gy = 0.f, Gz = 0.f, Fx = 0.f, Fy = 0.f, Fz = 0.f;
      for (int t = t0; t < t1; ++t) {
        const gc_task tk = a.tasks[t];
        const int2 gjr = a.ranges[tk.j_first];
        const int2 gjid = a.ranges_id[tk.j_first];
        const bool self = (tk.flags & GC_TASK_SELF) != 0;
        const float xi = xr - (tk.shift[0] > 0.f ? tk.shift[0] : 0.f);
        const float yi = yr - (tk.shift[1] > 0.f ? tk.shift[1] : 0.f);
        const float zi = zr - (tk.shift[2] > 0.f ? tk.shift[2] : 0.f);
        const float sb0 = tk.shift[0] < 0.f ? tk.shift[0] : 0.f;
        const float sb1 = tk.shift[1] < 0.f ? tk.shift[1] : 0.f;
        const float sb2 = tk.shift[2] < 0.f ? tk.shift[2] : 0.f;
        for (int j0 = 0; j0 < gjr.y; j0 += kLJTile) {
          const int cnt = gjr.y - j0 < kLJTile ? gjr.y - j0 : kLJTile;
          for (int e = lane; e < cnt; e += 64) {
            float4 rj = a.rec[gjr.x + j0 + e];
            jt[wid][e] = make_float4(rj.x + sb0, rj.y + sb1, rj.z + sb2, rj.w);
            float4 g = A.cot[gjid.x + j0 + e];
            float m = A.mass_t[(int)rj.w];
            jh[wid][e] = make_float4(g.x / m, g.y / m, g.z / m, 0.f);
#pragma unroll
            for (int q = 0; q < 6; ++q) gj[wid][q][e] = 0.f;
          }
          wave_sync();
          if (active) {
            const int C = (cnt + S - 1) / S;
            const int e0 = sl * C, e1 = e0 + C < cnt ? e0 + C : cnt;
            const int cs = e1 - e0;
            if (cs > 0) {
              int e = e0 + il % cs;
              for (int k = 0; k < cs; ++k) {
                if (!(self && j0 + e <= i0 + il)) {
                  const float4 j = jt[wid][e];
                  const float dx = xi - j.x, dy = yi - j.y, dz = zi - j.z;
                  const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
                  if (r2 < a.rc2) {
                    const int tj = (int)j.w;
                    const float2 p = tab[ti * nt + tj];
                    const float e24 = p.x, sg = p.y;
                    const float ri2 = __builtin_amdgcn_rcpf(r2);
                    const float q = sg * sg * ri2;
                    const float q3 = q * q * q;
                    const float f = e24 * q3 * __builtin_fmaf(2.f, q3, -1.f) * ri2;          // force factor
                    const float fp = e24 * q3 * __builtin_fmaf(-14.f, q3, 4.f) * ri2 * ri2;  // df / d(r^2)
                    const float4 hj = jh[wid][e];
                    const float dhx = hx - hj.x, dhy = hy - hj.y, dhz = hz - hj.z;
                    const float pp = __builtin_fmaf(dhz, dz, __builtin_fmaf(dhy, dy, dhx * dx));
                    const float c2 = 2.f * fp * pp;
                    const float wx = __builtin_fmaf(f, dhx, c2 * dx);
                    const float wy = __builtin_fmaf(f, dhy, c2 * dy);
                    const float wz = __builtin_fmaf(f, dhz, c2 * dz);
                    Gx += wx; Gy += wy; Gz += wz;
                    Fx = __builtin_fmaf(f, dx, Fx);
                    Fy = __builtin_fmaf(f, dy, Fy);
                    Fz = __builtin_fmaf(f, dz, Fz);
                    atomicAdd(&gj[wid][0][e], -wx);
                    atomicAdd(&gj[wid][1][e], -wy);
                    atomicAdd(&gj[wid][2][e], -wz);
                    atomicAdd(&gj[wid][3][e], -f * dx);
                    atomicAdd(&gj[wid][4][e], -f * dy);
                    atomicAdd(&gj[wid][5][e], -f * dz);
                    // dL/deps_ij = p f / eps_ij; dL/dsigma_ij = p (24 eps)(24 s^11 r^-14 - 6 s^5 r^-8)
                    const float dle = pp * f * 24.f / e24;
                    const float fs = e24 * q3 * __builtin_fmaf(24.f, q3, -6.f) * ri2 / sg;
                    pa.add(tj, dle, pp * fs, pg_row);
                  }
                }
                e = (e + 1 == e1) ? e0 : e + 1;
              }
            }
          }
          wave_sync();
          for (int e = lane; e < cnt; e += 64) {
            const int id = gjid.x + j0 + e;
            float4* q = A.gpos + id;
            unsafeAtomicAdd(&q->x, gj[wid][0][e]);
            unsafeAtomicAdd(&q->y, gj[wid][1][e]);
            unsafeAtomicAdd(&q->z, gj[wid][2][e]);
            float4* fq = A.force + id;
            unsafeAtomicAdd(&fq->x, gj[wid][3][e]);
            unsafeAtomicAdd(&fq->y, gj[wid][4][e]);
            unsafeAtomicAdd(&fq->z, gj[wid][5][e]);
          }
          wave_sync();
        }
      }
      if (active) pa.flush(pg_row, nullptr);
      red[wid][0][lane] = Gx; red[wid][1][lane] = Gy; red[wid][2][lane] = Gz;
      red[wid][3][lane] = Fx; red[wid][4][lane] = Fy; red[wid][5][lane] = Fz;
      wave_sync();
      if (lane < icc) {
        float sm[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int sidx = 0; sidx < S; ++sidx)
#pragma unroll
          for (int q = 0; q < 6; ++q) sm[q] += red[wid][q][sidx * icc + lane];
        const int id = tk0.i_begin + i0 + lane;
        float4* q = A.gpos + id;
        unsafeAtomicAdd(&q->x, sm[0]);
        unsafeAtomicAdd(&q->y, sm[1]);
        unsafeAtomicAdd(&q->z, sm[2]);
        float4* fq = A.force + id;
        unsafeAtomicAdd(&fq->x, sm[3]);
        unsafeAtomicAdd(&fq->y, sm[4]);
        unsafeAtomicAdd(&fq->z, sm[5]);
      }
      wave_sync();
    }
  }
  __syncthreads();
  block_param_partial(A, &pg[0][0], nt);
}

// Gather form of the Lennard-Jones adjoint (see the forward gather form for the schedule, the staging and the
// cutoff arithmetic).  Each target atom's dL/dx is added to gpos and its recomputed force written
// to `force` by one wavefront; the parameter derivatives go through per-lane sums keyed by the
// source type, the block's LDS, then one row of partial sums a block.
//
// What bounds it: the issue of vector instructions, 51 a pair with two types.  A step's sources are evaluated as
// they come: 30 kB more of LDS a block to hold those of several steps leaves four wavefronts a SIMD instead of
// seven (235 against 206 us, 426 k atoms of two types), and two pairs at a time need the register bound (213 us at
// five wavefronts a SIMD, 196 at seven).  284 us before the forward form's staging and this split.
constexpr int kGRoom = 64;  // staged sources a wavefront has room for: one step's, a multiple of the slices

// A staged source: its position, and 16 x its type | its entry << 8; its g / m.  A long sum over the sources would round at
// its own size for each of a pair's two terms: a step's sources are summed on their own first, or (ONCE, where a wavefront
// has one or two steps) a pair's terms before they are added.
template <int NT, bool SHIFTED, bool ONCE>
__device__ __forceinline__ void adj_gather_tile(const float4* __restrict__ p, const float4* __restrict__ hp,
                                                const float4* __restrict__ to, int C, float tx, float ty, float tz,
                                                float hx, float hy, float hz, const char* __restrict__ trow,
                                                float4 p0, float rc2, float (&acc)[6], ParamAcc<NT>& pa,
                                                float* pg_row) {
#pragma unroll 2
  for (int k = 0; k < C; ++k) {
    const float4 sj = p[k], hj = hp[k];
    const unsigned w = __float_as_uint(sj.w);
    float ux = tx, uy = ty, uz = tz;
    if (SHIFTED) {
      const float4 o = to[w >> 8];
      ux = tx + o.x;
      uy = ty + o.y;
      uz = tz + o.z;
    }
    const float ex = ux - sj.x, ey = uy - sj.y, ez = uz - sj.z;
    const float r2 = __builtin_fmaf(ez, ez, __builtin_fmaf(ey, ey, ex * ex));
    const bool in = r2 < rc2 && r2 > 0.f;
    const unsigned tj = SHIFTED ? w & 0xffu : w;
    float4 c = p0;  // (24 eps_ij, sigma_ij^2, 12 / (24 eps_ij), 1 / sigma_ij)
    if (NT == 2) {
      const float2 two = *reinterpret_cast<const float2*>(trow + tj);
      c.x = two.x;
      c.y = two.y;
    } else if (NT == 0) {
      c = *reinterpret_cast<const float4*>(trow + tj);
    }
    const float ri2 = in ? __builtin_amdgcn_rcpf(r2) : 0.f;  // outside the cutoff every term is zero
    const float q = c.y * ri2;
    const float q3 = q * q * q;
    const float eq = c.x * q3 * ri2;
    const float f = eq * __builtin_fmaf(2.f, q3, -1.f);           // force factor
    const float fp = eq * __builtin_fmaf(-28.f, q3, 8.f) * ri2;   // 2 df / d(r^2)
    const float fs = eq * __builtin_fmaf(12.f, q3, -3.f);         // sigma_ij times half of d(f r^2 ...)/dsigma
    const float dhx = hx - hj.x, dhy = hy - hj.y, dhz = hz - hj.z;
    const float pp = __builtin_fmaf(dhz, ez, __builtin_fmaf(dhy, ey, dhx * ex));
    const float c2 = fp * pp;
    if (ONCE) {
      acc[0] += __builtin_fmaf(f, dhx, c2 * ex);
      acc[1] += __builtin_fmaf(f, dhy, c2 * ey);
      acc[2] += __builtin_fmaf(f, dhz, c2 * ez);
    } else {
      acc[0] = __builtin_fmaf(f, dhx, __builtin_fmaf(c2, ex, acc[0]));
      acc[1] = __builtin_fmaf(f, dhy, __builtin_fmaf(c2, ey, acc[1]));
      acc[2] = __builtin_fmaf(f, dhz, __builtin_fmaf(c2, ez, acc[2]));
    }
    acc[3] = __builtin_fmaf(f, ex, acc[3]);
    acc[4] = __builtin_fmaf(f, ey, acc[4]);
    acc[5] = __builtin_fmaf(f, ez, acc[5]);
    if (NT > 0) pa.add((int)tj, pp * f, pp * fs, pg_row);
    else pa.add((int)(tj >> 4), pp * f * c.z, pp * fs * c.w, pg_row);
  }
}

// SPLIT: the block's wavefronts share a target range, as in the forward form.
template <int NT, bool SPLIT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7))) k_lj_adj_gather(LJAdjArgs A) {
  const LJArgs& a = A.f;
  __shared__ float4 tab[kMaxTypes * kMaxTypes];
  __shared__ float4 stage[4][2 * kGRoom];  // per wavefront: staged sources and their g / m; the sums at the end
  __shared__ dev::EntryTable tables[4];
  __shared__ float pg[4][2 * kMaxTypes * kMaxTypes];
  const int lane = threadIdx.x & 63;
  const int wid = uniform(threadIdx.x >> 6);
  float4* src = stage[wid];
  float4* hsr = stage[wid] + kGRoom;
  dev::EntryTable& T = tables[wid];
  static_assert(2 * kGRoom * 4 >= 6 * 64, "reduction area");
  const int nt = a.n_types;
  for (int k = threadIdx.x; k < nt * nt; k += blockDim.x) {
    const int ta = k / nt, tb = k % nt;
    const float e24 = 24.f * sqrtf(a.eps_t[ta] * a.eps_t[tb]), sg = 0.5f * (a.sig_t[ta] + a.sig_t[tb]);
    tab[k] = make_float4(e24, sg * sg, 12.f / e24, 1.f / sg);
  }
  for (int k = threadIdx.x; k < 4 * 2 * kMaxTypes * kMaxTypes; k += blockDim.x) (&pg[0][0])[k] = 0.f;
  __syncthreads();
  const float4 p0 = tab[0];
  const int32_t* tw0 = reinterpret_cast<const int32_t*>(a.tasks);
  constexpr int kTaskWords = sizeof(gc_task) / 4;
  const int g = uniform(SPLIT ? (int)blockIdx.x : (int)blockIdx.x * 4 + wid);
  if (g < a.n_tgt) {
    const int4 tg = dev::gld(a.tgt + g);
    const int id0 = uniform(tg.x), cnt = uniform(tg.y), e0 = uniform(tg.z), ne = uniform(tg.w);
    const int en0 = uniform(dev::gld(a.ent + e0));
    const int32_t* tw = tw0 + (int64_t)(en0 >> 1) * kTaskWords;
    const int rb = (en0 & 1) ? uniform(dev::gld(a.ranges + uniform(dev::gld(tw + 2))).x)
                             : (a.ibeg ? uniform(dev::gld(a.ibeg + (en0 >> 1))) : uniform(dev::gld(tw)));
    for (int i0 = 0; i0 < cnt; i0 += 64) {
      const int icc = cnt - i0 < 64 ? cnt - i0 : 64;
      const uint32_t mh = dev::recip16(icc);
      const int S = (int)((64u * mh) >> 16);
      const int sl = (int)(((uint32_t)lane * mh) >> 16), il = lane - sl * icc;
      const bool active = sl < S;
      float tx = 0.f, ty = 0.f, tz = 0.f, hx = 0.f, hy = 0.f, hz = 0.f;
      int ti = 0;
      if (active) {
        const float4 r = dev::gld(a.rec + rb + i0 + il);
        tx = r.x; ty = r.y; tz = r.z;
        ti = (int)r.w;
        const float4 gc4 = dev::gld(A.cot + id0 + i0 + il);
        const float m = A.mass_t[ti];
        hx = gc4.x / m; hy = gc4.y / m; hz = gc4.z / m;
      }
      const float4* trow = tab + ti * nt;
      float* pg_row = &pg[wid][2 * ti * nt];
      ParamAcc<NT> pa;
      pa.zero();
      float acc[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      // candidates pruned against the targets' bounding box as in the forward gather (every term of a
      // pair outside the cutoff is zero, so a source beyond r_c of the box adds nothing)
      float blx, bly, blz, bhx, bhy, bhz;
      dev::wave_interval(tx, active, blx, bhx);
      dev::wave_interval(ty, active, bly, bhy);
      dev::wave_interval(tz, active, blz, bhz);
      const float keep2 = a.rc2 * 1.001f;
      const int step = S * (int)((64u * dev::recip16(S)) >> 16);  // sources staged at a time
      for (int eg = 0; eg < ne; eg += dev::kEGroup) {
        const dev::EntryGroup G =
            dev::load_entries<true>(a, e0 + eg, ne - eg < dev::kEGroup ? ne - eg : dev::kEGroup, T);
        for (int ws = SPLIT ? step * wid : 0; ws < G.total; ws += SPLIT ? 4 * step : step) {
          const int e = dev::entry_at(G, ws, T);
          float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
          int type = 0;
          bool keep = false;
          if (lane < step && ws + lane < G.total) {
            v = dev::gld(a.rec + (T.rec[e] + ws + lane));
            type = (int)v.w;
            unsigned w = NT == 1 ? 0u : 16u * (unsigned)type;
            float px = v.x, py = v.y, pz = v.z;
            if (G.shifted) {
              const float4 q = T.sh[e], o = T.to[e];
              v.x += q.x; v.y += q.y; v.z += q.z;
              px = v.x - o.x; py = v.y - o.y; pz = v.z - o.z;
              w |= (unsigned)e << 8;
            }
            v.w = __uint_as_float(w);
            keep = dev::box_d2(px, py, pz, blx, bly, blz, bhx, bhy, bhz) <= keep2;
          }
          const uint64_t km = __ballot(keep);
          const int kc = uniform(__popcll(km));
          const int C = uniform((int)((uint32_t)(kc + S - 1) / (uint32_t)S));
          if (keep) {
            const int k = __builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
            const float4 gs = dev::gld(A.cot + (T.id[e] + ws + lane));
            const float ms = A.mass_t[type];
            src[k] = v;
            hsr[k] = make_float4(gs.x / ms, gs.y / ms, gs.z / ms, 0.f);
          }
          if (lane >= kc && lane < S * C) {
            src[lane] = make_float4(dev::kFar, dev::kFar, dev::kFar, 0.f);
            hsr[lane] = make_float4(0.f, 0.f, 0.f, 0.f);
          }
          wave_sync();
          if (active) {
            const char* row = reinterpret_cast<const char*>(trow);
            float part[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (G.shifted)
              adj_gather_tile<NT, true, SPLIT>(src + sl * C, hsr + sl * C, T.to, C, tx, ty, tz, hx, hy, hz, row, p0, a.rc2,
                                               part, pa, pg_row);
            else
              adj_gather_tile<NT, false, SPLIT>(src + sl * C, hsr + sl * C, T.to, C, tx, ty, tz, hx, hy, hz, row, p0,
                                                a.rc2, part, pa, pg_row);
#pragma unroll
            for (int q = 0; q < 6; ++q) acc[q] += part[q];
          }
          wave_sync();
        }
      }
      if (active) pa.flush(pg_row, trow);
      float* red = reinterpret_cast<float*>(src);  // 6 x 64 floats
#pragma unroll
      for (int q = 0; q < 6; ++q) red[q * 64 + lane] = acc[q];
      if (SPLIT) __syncthreads();
      else wave_sync();
      if (lane < icc && (!SPLIT || wid == 0)) {
        float sm[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int x = 0; x < (SPLIT ? 4 : 1); ++x) {
          const float* part = SPLIT ? reinterpret_cast<const float*>(stage[x]) : red;
          float of[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // (each wavefront's slices on their own)
          for (int sidx = 0; sidx < S; ++sidx)
#pragma unroll
            for (int q = 0; q < 6; ++q) of[q] += part[q * 64 + sidx * icc + lane];
#pragma unroll
          for (int q = 0; q < 6; ++q) sm[q] += of[q];
        }
        const int id = id0 + i0 + lane;
        const float4 g0 = dev::gld(A.gpos + id);
        dev::gst(A.gpos + id, make_float4(g0.x + sm[0], g0.y + sm[1], g0.z + sm[2], g0.w));
        dev::gst(A.force + id, make_float4(sm[3], sm[4], sm[5], 0.f));
      }
      if (SPLIT && i0 + 64 < cnt) __syncthreads();
      else wave_sync();
    }
  }
  __syncthreads();
  block_param_partial(A, &pg[0][0], nt);
}

__global__ void k_lj_mass_grad(const float4* __restrict__ cot, const float4* __restrict__ force,
                               const float* __restrict__ mass_t, const float4* __restrict__ rec_by_id,
                               float* __restrict__ gmass, int32_t n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const float4 g = cot[i], F = force[i];
    const float m = mass_t[(int)rec_by_id[i].w];
    gmass[i] += -(g.x * F.x + g.y * F.y + g.z * F.z) / (m * m);
  }
}

}  // namespace

namespace {
template <bool PACKED, int ORDER, bool NODES>
hipError_t adj_items(const GravAdjArgs& a, int n_items, int most, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  const size_t lds = 4 * (NODES && ORDER == 2 ? 11 : NODES ? 5 : 6) * (size_t)most;
  if (lds > (NODES ? kAdjNodeBytes : kAdjDirectBytes)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_grav_adj<PACKED, ORDER, NODES>), dim3(n_items),
                     dim3(64 * (NODES ? kAdjNodeWaves : kAdjDirectWaves)), lds, s, a);
  return hipGetLastError();
}
template <bool PACKED, int ORDER>
hipError_t adj_both(const GravAdjArgs& a, int n_cu, hipStream_t s) {
  const size_t nodes = 4 * (ORDER == 2 ? 11 : 5) * (size_t)a.max_nodes, direct = 4 * 6 * (size_t)a.max_direct;
  const size_t lds = nodes > direct ? nodes : direct;
  if (lds > kAdjNodeBytes) return hipErrorInvalidValue;
  const int by_lds = (int)(163840 / (lds + 1)), by_regs = ORDER == 2 ? 4 : 6;  // workgroups per CU
  if (a.n_node_items > 0 && a.n_direct_items > 0 &&
      a.n_node_items + a.n_direct_items <= (by_lds < by_regs ? by_lds : by_regs) * n_cu) {
    hipLaunchKernelGGL((k_grav_adj_both<PACKED, ORDER>), dim3(a.n_node_items + a.n_direct_items),
                       dim3(64 * kAdjNodeWaves), lds, s, a);
    return hipGetLastError();
  }
  const hipError_t e = adj_items<PACKED, ORDER, true>(a, a.n_node_items, a.max_nodes, s);
  return e != hipSuccess ? e : adj_items<PACKED, ORDER, false>(a, a.n_direct_items, a.max_direct, s);
}
}  // namespace

hipError_t launch_grav_adjoint(bool packed, int order, const GravAdjArgs& a, int n_cu, hipStream_t s) {
  if (order == 2) return packed ? adj_both<true, 2>(a, n_cu, s) : adj_both<false, 2>(a, n_cu, s);
  return packed ? adj_both<true, 1>(a, n_cu, s) : adj_both<false, 1>(a, n_cu, s);
}

hipError_t launch_adj_finish(const AdjFinishArgs& a, hipStream_t s) {
  if (a.one_task && a.n_node_items + a.n_direct_items > 0)
    hipLaunchKernelGGL(k_adj_items, dim3(a.n_node_items + a.n_direct_items), dim3(64), 0, s, a);
  if (a.n_direct > 0)
    hipLaunchKernelGGL(k_adj_keys, dim3(a.n_direct < 4096 * 256 ? (a.n_direct + 255) / 256 : 4096), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_record_sums(int order, const float4* vdir, const int32_t* dvis, const int32_t* dkey, int32_t n_direct,
                              float4* gpos, float* gmass, const float4* vnode, const int32_t* nvis, const int2* chunks,
                              int32_t n_chunks, float4* part, hipStream_t s) {
  const int db = (n_direct + 255) / 256, nb = (n_chunks + 3) / 4;
  if (db + nb <= 0) return hipSuccess;
  const SumArgs a{vdir, dvis, dkey, n_direct, gpos, gmass, vnode, nvis, chunks, n_chunks, part};
  if (order == 2) hipLaunchKernelGGL(k_record_sums<3>, dim3(db + nb), dim3(256), 0, s, a, db);
  else hipLaunchKernelGGL(k_record_sums<1>, dim3(db + nb), dim3(256), 0, s, a, db);
  return hipGetLastError();
}

hipError_t launch_node_chain(int order, const int32_t* node_range, int32_t n_nodes, const float4* nodes,
                             const float4* part, const int32_t* chunk_first, const float4* rec_by_id, int32_t n_ids,
                             float4* gpos, float* gmass, int32_t* bad, hipStream_t s) {
  if (n_nodes <= 0) return hipSuccess;
  const int windows = (n_nodes + 63) / 64, groups = windows < kChainGroups ? windows : kChainGroups;
  const dim3 grid(groups * kChainSplit + (n_nodes + 3) / 4);
  if (order == 2)
    hipLaunchKernelGGL(k_node_chain<3>, grid, dim3(256), 0, s,
                       (ChainArgs<3>{node_range, n_nodes, nodes, part, chunk_first, rec_by_id, n_ids, gpos, gmass, bad}),
                       groups);
  else
    hipLaunchKernelGGL(k_node_chain<1>, grid, dim3(256), 0, s,
                       (ChainArgs<1>{node_range, n_nodes, nodes, part, chunk_first, rec_by_id, n_ids, gpos, gmass, bad}),
                       groups);
  return hipGetLastError();
}

int lj_adjoint_blocks(const LJArgs& f, bool gather) {
  if (!gather) return (f.n_runs + 3) / 4;
  return f.n_tgt <= dev::kGSplit ? f.n_tgt : (f.n_tgt + 3) / 4;
}

hipError_t launch_lj_adjoint(const LJAdjArgs& a, int wpb, hipStream_t s) {
  (void)wpb;
  if (a.f.n_runs <= 0) return hipSuccess;
  const int nb = lj_adjoint_blocks(a.f, false);
  if (a.f.n_types == 1) hipLaunchKernelGGL(k_lj_adj<1>, dim3(nb), dim3(256), 0, s, a);
  else if (a.f.n_types == 2) hipLaunchKernelGGL(k_lj_adj<2>, dim3(nb), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_lj_adj<0>, dim3(nb), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_lj_param_reduce, dim3(a.f.n_types * a.f.n_types), dim3(256), 0, s, a.ppart, nb, a.f.n_types,
                     a.f.eps_t, a.gparam);
  return hipGetLastError();
}

namespace {
template <int NT>
void adj_gather_launch(const LJAdjArgs& a, int nb, hipStream_t s) {
  if (a.f.n_tgt <= dev::kGSplit) hipLaunchKernelGGL((k_lj_adj_gather<NT, true>), dim3(nb), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_lj_adj_gather<NT, false>), dim3(nb), dim3(256), 0, s, a);
}
}  // namespace

hipError_t launch_lj_adjoint_gather(const LJAdjArgs& a, hipStream_t s) {
  if (a.f.n_tgt <= 0) return hipSuccess;
  const int nb = lj_adjoint_blocks(a.f, true);
  if (a.f.n_types == 1) adj_gather_launch<1>(a, nb, s);
  else if (a.f.n_types == 2) adj_gather_launch<2>(a, nb, s);
  else adj_gather_launch<0>(a, nb, s);
  hipLaunchKernelGGL(k_lj_param_reduce, dim3(a.f.n_types * a.f.n_types), dim3(256), 0, s, a.ppart, nb, a.f.n_types,
                     a.f.eps_t, a.gparam);
  return hipGetLastError();
}

hipError_t launch_lj_mass_grad(const float4* cot, const float4* force, const float* mass_t, const float4* rec_by_id,
                               float* gmass, int32_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int g = (n + 255) / 256;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_lj_mass_grad, dim3(g), dim3(256), 0, s, cot, force, mass_t, rec_by_id, gmass, n);
  return hipGetLastError();
}

}  // namespace gc
