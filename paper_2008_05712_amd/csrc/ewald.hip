// Combined Ewald kernel: the correction of periodic gravity (Sec. 4.1: ChaNGa sums the periodic
// images by Ewald summation on the GPU; Sec. 4.3: its work requests are combined like the force
// requests).  Every target of every task of a batch in one launch.
//
// For a cubic box of side L holding total mass M with centre of mass c, at r = x - c (nearest
// image) and splitting parameter alpha, the correction is the pull of every periodic image of M
// plus the neutralising background, less the central copy's direct pull (the tree walk computes
// that one):
//   a = G M [ sum_{n != 0, |n_d| <= nrep} -(erfc(alpha s)/s^3 + 2 alpha/sqrt(pi) e^{-alpha^2 s^2}/s^2) s_vec
//           + (erf(alpha s)/s^3 - 2 alpha/sqrt(pi) e^{-alpha^2 s^2}/s^2) s_vec          (n = 0)
//           - 2/L^2 sum_{0 < |h|^2 <= hmax2} e^{-pi^2 |h|^2/(alpha L)^2}/|h|^2 sin(2 pi h.r/L) h ],
// s_vec = r + n L.  The n = 0 bracket cancels (at alpha s = 1/2 to a sixth of its terms) and is taken below alpha s = 1 from
// its series, that of l = 1 below; with the difference itself from 1/2 on, this one term set the error of the
// whole sum (80,000 targets: 3.3e-7 of it with second moments and 2.4e-7 without; 2.7e-7 and 1.4e-7 now).
//
// With the box's second moment S about c the same kernel is expanded to second order: each image
// adds G [1/2 (tr(S) s_vec + 2 S s_vec) B_2 - 1/2 (s_vec.S.s_vec) s_vec B_3], with the radial
// derivatives B_l = ((2l - 1) B_{l-1} + (2 alpha^2)^l / (alpha sqrt(pi)) e^{-alpha^2 s^2}) / s^2 of
// B_0 = erfc(alpha s)/s (n != 0) or -erf(alpha s)/s (n = 0, from its series below alpha s = 1:
// -(2/sqrt(pi)) 2^l alpha^{2l+1} sum_j (-1)^j x^{2j} / (j! (2j + 2l + 1))), and each wave vector adds
// G 4 pi^2/L^4 e^{-pi^2 |h|^2/(alpha L)^2}/|h|^2 (h.S.h) sin(2 pi h.r/L) h, which is target independent
// apart from the sine and so joins the monopole's weight in the table.
//
// A bucket holds about ten targets and each target costs thousands of VALU operations, so the lanes
// take the batch's targets in flat order rather than one workgroup per bucket, which would leave most of a
// wave64 idle; below kEwaldSplit targets four neighbouring lanes share a target (its images and its wave
// vectors by |h_x|), else there would be too few wavefronts to fill the chip.  A wavefront finds its
// targets' tasks by probing the per-task target offsets 64 at a time (three dependent loads where a search by
// each lane takes fifteen).
//
// Wave vectors: the terms h and -h are equal (sin is odd), so only h_x > 0 (and half of the plane h_x = 0)
// is summed, with twice the weight.  sin(2 pi h.r/L) comes from products of the three components' sines and
// cosines, advanced by one multiplication a step, and +-h_z share theirs: with E = e^{2 pi i (h_x x + h_y y)},
// w+- the weights, p = Im E cos(2 pi h_z z), q = Re E sin(2 pi h_z z), the pair is w+ (p + q) + w- (p - q); the table
// (built in LDS by each block) holds w+ + w-, w+ - w- and the same times h_z.
//
// Images: erfc(x) = e^{-x^2} erfcx(x) with one exponential for all radial derivatives, reciprocals by the
// hardware approximation and one Newton step.  erfcx(x) (x + 2) is a polynomial of degree 10 in t = (x - 2)/(x + 2)
// (the variable of Shepherd and Laframboise 1981), fitted by least squares of the relative error on Chebyshev
// nodes: within 9.1e-8 everywhere with the coefficients in FP32.
//
// What bounds it: vector instructions.  A target took 7,100 (27 images, 73 half-space wave vectors, second
// moments): sinpif for each vector, erfcf, expf, a square root and three divisions for each image; now 2,840.
// 262,144 targets: 47.6 -> 20.6 us.
#include "gc_internal.h"
#include "mem_dev.h"

namespace gc {
namespace {

constexpr int kEwThreads = 256;

// sum_{j <= 10} (-1)^j x2^j / (j! (2j + 2l + 1)) for l = 1, 2, 3 (Horner; the next term is below 1e-8
// of the first for x2 < 1)
__device__ __forceinline__ float erf_series_1(float x2) {
  float p = 1.f / 83462400.f;
  p = __builtin_fmaf(p, x2, -1.f / 7620480.f);
  p = __builtin_fmaf(p, x2, 1.f / 766080.f);
  p = __builtin_fmaf(p, x2, -1.f / 85680.f);
  p = __builtin_fmaf(p, x2, 1.f / 10800.f);
  p = __builtin_fmaf(p, x2, -1.f / 1560.f);
  p = __builtin_fmaf(p, x2, 1.f / 264.f);
  p = __builtin_fmaf(p, x2, -1.f / 54.f);
  p = __builtin_fmaf(p, x2, 1.f / 14.f);
  p = __builtin_fmaf(p, x2, -1.f / 5.f);
  return __builtin_fmaf(p, x2, 1.f / 3.f);
}
__device__ __forceinline__ float erf_series_2(float x2) {
  float p = 1.f / 90720000.f;
  p = __builtin_fmaf(p, x2, -1.f / 8346240.f);
  p = __builtin_fmaf(p, x2, 1.f / 846720.f);
  p = __builtin_fmaf(p, x2, -1.f / 95760.f);
  p = __builtin_fmaf(p, x2, 1.f / 12240.f);
  p = __builtin_fmaf(p, x2, -1.f / 1800.f);
  p = __builtin_fmaf(p, x2, 1.f / 312.f);
  p = __builtin_fmaf(p, x2, -1.f / 66.f);
  p = __builtin_fmaf(p, x2, 1.f / 18.f);
  p = __builtin_fmaf(p, x2, -1.f / 7.f);
  return __builtin_fmaf(p, x2, 1.f / 5.f);
}
__device__ __forceinline__ float erf_series_3(float x2) {
  float p = 1.f / 97977600.f;
  p = __builtin_fmaf(p, x2, -1.f / 9072000.f);
  p = __builtin_fmaf(p, x2, 1.f / 927360.f);
  p = __builtin_fmaf(p, x2, -1.f / 105840.f);
  p = __builtin_fmaf(p, x2, 1.f / 13680.f);
  p = __builtin_fmaf(p, x2, -1.f / 2040.f);
  p = __builtin_fmaf(p, x2, 1.f / 360.f);
  p = __builtin_fmaf(p, x2, -1.f / 78.f);
  p = __builtin_fmaf(p, x2, 1.f / 22.f);
  p = __builtin_fmaf(p, x2, -1.f / 9.f);
  return __builtin_fmaf(p, x2, 1.f / 7.f);
}

// erfcx(x) = e^{x^2} erfc(x) for x >= 0
__device__ __forceinline__ float erfcx_pos(float x) {
  const float d = x + 2.f;
  float q = __builtin_amdgcn_rcpf(d);
  q = __builtin_fmaf(__builtin_fmaf(-d, q, 1.f), q, q);
  const float t = __builtin_fmaf(-4.f, q, 1.f);
  float p = 8.436608067e-05f;
  p = __builtin_fmaf(p, t, 7.326729099e-05f);
  p = __builtin_fmaf(p, t, -5.988875914e-04f);
  p = __builtin_fmaf(p, t, -8.614828529e-04f);
  p = __builtin_fmaf(p, t, 3.058435791e-03f);
  p = __builtin_fmaf(p, t, 6.487009153e-03f);
  p = __builtin_fmaf(p, t, -2.150330270e-02f);
  p = __builtin_fmaf(p, t, -3.644336768e-02f);
  p = __builtin_fmaf(p, t, 2.794714745e-01f);
  p = __builtin_fmaf(p, t, -6.871606353e-01f);
  p = __builtin_fmaf(p, t, 1.021582714e+00f);
  return p * q;
}

// e^{-v} for v >= 0 (zero from about 104 on): the product with log2(e) in two parts
__device__ __forceinline__ float exp_neg(float v) {
  v = fminf(v, 1000.f);
  const float hi = v * -1.44269502f;
  const float lo = __builtin_fmaf(v, -1.92596303e-8f, __builtin_fmaf(v, -1.44269502f, -hi));
  const float e = __builtin_amdgcn_exp2f(hi);
  return __builtin_fmaf(e, lo * 0.69314718f, e);
}

// The task of flat target f: the last with ioff[t] <= f.
__device__ __forceinline__ int task_of(const EwaldArgs& a, int64_t f) {
  const int lane = threadIdx.x & 63;
  const int first = __builtin_amdgcn_readfirstlane((int)f), last = __builtin_amdgcn_readlane((int)f, 63);
  // the wavefront's first task is in [lo, lo + n)
  int lo = 0, n = a.n_tasks;
  while (n > 64) {
    const int step = (n + 63) >> 6, at = lane * step;
    const uint64_t m = __ballot(at < n && dev::gld(a.ioff + lo + at) <= first);  // lanes 0 .. k
    const int k = 63 - __builtin_clzll(m | 1ull);
    lo += k * step;
    n = n - k * step < step ? n - k * step : step;
  }
  {
    const uint64_t m = __ballot(lane < n && dev::gld(a.ioff + lo + lane) <= first);
    lo += 63 - __builtin_clzll(m | 1ull);
  }
  // the lanes' tasks among the 64 from there, unless those end before the last target
  const int o = lo + lane < a.n_tasks ? dev::gld(a.ioff + lo + lane) : INT32_MAX;
  if (__builtin_amdgcn_readlane(o, 63) > last) {
    int t = 0;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
      const int v = __shfl(o, t + s, 64);
      t += v <= (int)f ? s : 0;
    }
    return lo + t;
  }
  int hi = a.n_tasks - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (dev::gld(a.ioff + mid) <= f) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <bool QUAD, int P>
__global__ void __launch_bounds__(kEwThreads) k_ewald(EwaldArgs a) {
  // at (hx, hy + hmax, hz): w+ + w-, w+ - w-, hz (w+ - w-), hz (w+ + w-) of (hx, hy, +-hz); x at hz = 0 is w+
  extern __shared__ float4 wtab[];
  const int hm = a.hmax, side = 2 * hm + 1, col = hm + 1;
  for (int k = threadIdx.x; k < col * side * col; k += kEwThreads) {
    const int hz = k % col, hy = (k / col) % side - hm, hx = k / (col * side);
    const int h2i = hx * hx + hy * hy + hz * hz;
    auto weight = [&](float fz) {
      const float fx = (float)hx, fy = (float)hy, h2 = (float)h2i;
      float kc = a.kcoef;
      if (QUAD) {
        const float hSh = fx * (a.GS[0] * fx + a.GS[3] * fy + a.GS[4] * fz) +
                          fy * (a.GS[3] * fx + a.GS[1] * fy + a.GS[5] * fz) +
                          fz * (a.GS[4] * fx + a.GS[5] * fy + a.GS[2] * fz);
        kc = __builtin_fmaf(a.qcoef, hSh, kc);
      }
      return 2.f * kc * expf(-a.kdecay * h2) / h2;  // both h and -h
    };
    float wp = 0.f, wm = 0.f;
    if (h2i > 0 && h2i <= a.hmax2) {
      if (hx > 0 || hy > 0) {
        wp = weight((float)hz);
        if (hz > 0) wm = weight(-(float)hz);
      } else if (hy == 0) {
        wp = weight((float)hz);
      }
    }
    wtab[k] = make_float4(wp + wm, wp - wm, (float)hz * (wp - wm), (float)hz * (wp + wm));
  }
  __syncthreads();
  const int64_t slot = (int64_t)blockIdx.x * kEwThreads + threadIdx.x;
  const int part = P == 1 ? 0 : (int)(threadIdx.x & (P - 1));
  const bool real = slot / P < a.n_targets;
  const int64_t f = real ? slot / P : a.n_targets - 1;  // (whole wavefronts search together)
  const int task = task_of(a, f);
  const int k = (int)(f - dev::gld(a.ioff + task));
  const int32_t* tw = reinterpret_cast<const int32_t*>(a.tasks + task);
  const int id = dev::gld(tw) + k;
  const int pos = (a.ibeg ? dev::gld(a.ibeg + task) : dev::gld(tw)) + k;
  const float4 x = dev::gld(a.rec + pos);
  float r[3] = {x.x - a.c[0], x.y - a.c[1], x.z - a.c[2]};
#pragma unroll
  for (int d = 0; d < 3; ++d) r[d] -= a.L * rintf(r[d] * a.inv_L);
  const float al = a.alpha, sp = 1.1283791670955126f * al;  // 2 alpha / sqrt(pi)
  const float al2 = al * al, k2 = 2.f * al2 * sp, k3 = 4.f * al2 * al2 * sp;  // (2 alpha^2)^l / (alpha sqrt(pi))
  const float tr = a.GS[0] + a.GS[1] + a.GS[2];
  float ax = 0.f, ay = 0.f, az = 0.f;
  // an image at s with -B_1 = kf, B_2, B_3
  auto add = [&](float sx, float sy, float sz, float kf, float b2, float b3) {
    float cf = a.GM * kf;
    if (QUAD) {
      const float Sx = __builtin_fmaf(a.GS[4], sz, __builtin_fmaf(a.GS[3], sy, a.GS[0] * sx));
      const float Sy = __builtin_fmaf(a.GS[5], sz, __builtin_fmaf(a.GS[1], sy, a.GS[3] * sx));
      const float Sz = __builtin_fmaf(a.GS[2], sz, __builtin_fmaf(a.GS[5], sy, a.GS[4] * sx));
      const float sSs = __builtin_fmaf(sz, Sz, __builtin_fmaf(sy, Sy, sx * Sx));
      cf = __builtin_fmaf(0.5f, __builtin_fmaf(tr, b2, -sSs * b3), cf);
      ax = __builtin_fmaf(b2, Sx, ax);
      ay = __builtin_fmaf(b2, Sy, ay);
      az = __builtin_fmaf(b2, Sz, az);
    }
    ax = __builtin_fmaf(cf, sx, ax);
    ay = __builtin_fmaf(cf, sy, ay);
    az = __builtin_fmaf(cf, sz, az);
  };
  auto image = [&](float nx, float ny, float nz) {
    const float sx = __builtin_fmaf(nx, a.L, r[0]), sy = __builtin_fmaf(ny, a.L, r[1]), sz = __builtin_fmaf(nz, a.L, r[2]);
    const float s2 = __builtin_fmaf(sz, sz, __builtin_fmaf(sy, sy, sx * sx));
    float ri = __builtin_amdgcn_rsqf(s2);
    ri = __builtin_fmaf(0.5f * ri, __builtin_fmaf(-s2 * ri, ri, 1.f), ri);
    const float xs = al * (s2 * ri), is2 = ri * ri;
    const float e = exp_neg(xs * xs);
    const float b1 = e * __builtin_fmaf(erfcx_pos(xs), ri, sp) * is2;
    float b2 = 0.f, b3 = 0.f;
    if (QUAD) {
      b2 = __builtin_fmaf(k2, e, 3.f * b1) * is2;
      b3 = __builtin_fmaf(k3, e, 5.f * b2) * is2;
    }
    add(sx, sy, sz, -b1, b2, b3);
  };
  if (P == 1) {
    for (int nx = -a.nrep; nx <= a.nrep; ++nx)
      for (int ny = -a.nrep; ny <= a.nrep; ++ny)
        for (int nz = -a.nrep; nz <= a.nrep; ++nz)
          if (nx != 0 || ny != 0 || nz != 0) image((float)nx, (float)ny, (float)nz);
  } else {
    // images part, part + P, ... of those but the central one
    const int w = 2 * a.nrep + 1, all = w * w * w;
    for (int m = part; m < all - 1; m += P) {
      const int q = m + (2 * m >= all - 1 ? 1 : 0);
      image((float)(q / (w * w) - a.nrep), (float)(q / w % w - a.nrep), (float)(q % w - a.nrep));
    }
  }
  if (part == P - 1) {  // the central copy's direct pull, taken out
    const float d2c = -4.f * sp * al2 * al2, d3c = 2.f * d2c * al2;  // -(2/sqrt(pi)) 2^l alpha^{2l+1}
    const float s2 = __builtin_fmaf(r[2], r[2], __builtin_fmaf(r[1], r[1], r[0] * r[0]));
    const float s = sqrtf(s2);
    const float xs = al * s, x2 = xs * xs;
    float kf, b2 = 0.f, b3 = 0.f;
    if (xs < 1.f) {
      kf = k2 * erf_series_1(x2);
    } else {
      kf = erff(xs) / (s2 * s) - sp * expf(-xs * xs) / s2;
    }
    if (QUAD) {
      if (xs < 1.f) {
        b2 = d2c * erf_series_2(x2);
        b3 = d3c * erf_series_3(x2);
      } else {
        const float e = expf(-x2), is2 = 1.f / s2;
        b2 = __builtin_fmaf(k2, e, -3.f * kf) * is2;
        b3 = __builtin_fmaf(k3, e, 5.f * b2) * is2;
      }
    }
    add(r[0], r[1], r[2], kf, b2, b3);
  }
  float bx = 0.f, by = 0.f, bz = 0.f;
  // (cosine, sine) of one step of each component, and of h_x steps
  const float ux = 2.f * (r[0] * a.inv_L), uy = 2.f * (r[1] * a.inv_L), uz = 2.f * (r[2] * a.inv_L);
  const float c1x = cospif(ux), s1x = sinpif(ux), c1y = cospif(uy), s1y = sinpif(uy), c1z = cospif(uz), s1z = sinpif(uz);
  auto turn = [](float& c, float& s, float c1, float s1) {
    const float t = __builtin_fmaf(c, c1, -s * s1);
    s = __builtin_fmaf(s, c1, c * s1);
    c = t;
  };
  float cx = 1.f, sx = 0.f;
  for (int k = 0; k < part; ++k) turn(cx, sx, c1x, s1x);
  for (int hx = part; hx <= hm; hx += P) {
    float cy = 1.f, sy = 0.f;
    for (int hy = 0; hx * hx + hy * hy <= a.hmax2; ++hy) {
      // E of (hx, hy), and of (hx, -hy) where that is another column of the half-space
      const float cc = cx * cy, ss = sx * sy, sc = sx * cy, cs = cx * sy;
      const bool both = hx > 0 && hy > 0;
      const float ec = cc - ss, es = sc + cs, fc = cc + ss, fs = sc - cs;
      const float4* up = wtab + (hx * side + hm + hy) * col;
      const float4* dn = wtab + (hx * side + hm - hy) * col;
      float A = up[0].x * es, B = both ? dn[0].x * fs : 0.f;
      float cz = 1.f, sz = 0.f;
      for (int hz = 1; hx * hx + hy * hy + hz * hz <= a.hmax2; ++hz) {
        turn(cz, sz, c1z, s1z);
        const float4 w = up[hz];
        const float p = es * cz, q = ec * sz;
        A = __builtin_fmaf(w.x, p, __builtin_fmaf(w.y, q, A));
        bz = __builtin_fmaf(w.z, p, __builtin_fmaf(w.w, q, bz));
        if (both) {
          const float4 v = dn[hz];
          const float p2 = fs * cz, q2 = fc * sz;
          B = __builtin_fmaf(v.x, p2, __builtin_fmaf(v.y, q2, B));
          bz = __builtin_fmaf(v.z, p2, __builtin_fmaf(v.w, q2, bz));
        }
      }
      bx = __builtin_fmaf((float)hx, A + B, bx);
      by = __builtin_fmaf((float)hy, A - B, by);
      turn(cy, sy, c1y, s1y);
    }
#pragma unroll
    for (int q = 0; q < P; ++q) turn(cx, sx, c1x, s1x);
  }
  float vx = ax + bx, vy = ay + by, vz = az + bz;
  if (P > 1) {
    static_assert(P == 1 || P == 4, "sums over the lanes of a quad");
    auto quad_sum = [](float v) {
      v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xb1, 0xf, 0xf, true));  // lanes 1 0 3 2
      v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4e, 0xf, 0xf, true));  // lanes 2 3 0 1
      return v;
    };
    vx = quad_sum(vx);
    vy = quad_sum(vy);
    vz = quad_sum(vz);
  }
  if (!real || part != 0) return;
  float4* dst = a.acc + id;
  const float4 o = dev::gld(dst);
  dev::gst(dst, make_float4(o.x + vx, o.y + vy, o.z + vz, o.w));
}

// Targets from which a lane has one of its own.  Measured with 26 images, 73 vectors and second moments, and with 124
// images, 46 vectors and none (us, with 5 for the clearing of the output): 32,768 targets: 14.0 and 18.6 with
// four lanes a target, 15.0 and 25.5 with one; 65,536: 16.4 and 28.4 against 15.3 and 26.1.
constexpr int64_t kEwaldSplit = 50000;

template <bool QUAD>
hipError_t launch(const EwaldArgs& a, hipStream_t s) {
  const size_t lds = sizeof(float4) * (size_t)(a.hmax + 1) * (size_t)(2 * a.hmax + 1) * (size_t)(a.hmax + 1);
  const int P = a.n_targets < kEwaldSplit ? 4 : 1;
  const unsigned g = (unsigned)((a.n_targets * P + kEwThreads - 1) / kEwThreads);
  if (P == 4) hipLaunchKernelGGL((k_ewald<QUAD, 4>), dim3(g), dim3(kEwThreads), lds, s, a);
  else hipLaunchKernelGGL((k_ewald<QUAD, 1>), dim3(g), dim3(kEwThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ewald(const EwaldArgs& a, hipStream_t s) {
  if (a.n_targets <= 0 || a.n_tasks <= 0) return hipSuccess;
  return a.quad ? launch<true>(a, s) : launch<false>(a, s);
}

}  // namespace gc
