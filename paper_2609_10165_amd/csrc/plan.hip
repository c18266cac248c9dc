// plan.hip -- building ghost-cell plans on the GPU.
//
// Pipeline (one launch per stage, all instances of a batch together):
//   classify      every cell: inside test at its centre (Sec. 3.1), and
//                 whether a face neighbour has the other class; far-field
//                 segments are settled by a radial bound and written as
//                 16-byte constant stores
//   scan/compact  interface cells in linear-index order
//   geometry      closest point, analytic normal, psi; ghost tags for CGC,
//                 CGC_ES and HGC (Eq. HGC_criterion with Eq. delta_n); the
//                 ghosts in linear-index order, and their cell table
//   deps          stencil code (e = sgn n, multipliers r), validation, and
//                 ghost-to-ghost dependencies (Sec. 3.2)
//   levels        layering and canonical order (level, linear index); a
//                 cycle's strongly connected groups become coupled units
//   finalize      canonical structure-of-arrays for the apply kernels
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>

#include "gcr_impl.hpp"

namespace gcr {


// --------------------------------------------------------------------------
// closest point and normal
// --------------------------------------------------------------------------

// The contour point C(s) = (s^2, +-y_t(s^2)) (s >= 0 upper, s < 0 lower
// surface), its derivative D and second derivative E in s.
__device__ __forceinline__ void naca_point(double t, double s, double C[2], double D[2],
                                           double E[2]) {
  double s2 = s * s, sg = s < 0.0 ? -1.0 : 1.0;
  double poly = 0.1260 * s2 + 0.3516 * s2 * s2 - 0.2843 * s2 * s2 * s2 + 0.1036 * s2 * s2 * s2 * s2;
  double dpoly = s * (2.0 * 0.1260 + s2 * (4.0 * 0.3516 + s2 * (-6.0 * 0.2843 + s2 * 8.0 * 0.1036)));
  double d2poly = 2.0 * 0.1260 + s2 * (12.0 * 0.3516 + s2 * (-30.0 * 0.2843 + s2 * 56.0 * 0.1036));
  C[0] = s2;
  C[1] = 5.0 * t * (0.2969 * s - sg * poly);
  D[0] = 2.0 * s;
  D[1] = 5.0 * t * (0.2969 - sg * dpoly);
  E[0] = 2.0;
  E[1] = -5.0 * t * sg * d2poly;
}

__device__ bool project(const ShapeD& s, int dim, const double x[3], bool solid, double n[3],
                        double& psi) {
  double v[3] = {x[0] - s.c[0], x[1] - s.c[1], dim == 3 ? x[2] - s.c[2] : 0.0};
  n[2] = 0.0;
  if (s.kind == kSphere) {
    double rho2 = v[0] * v[0] + v[1] * v[1];
    if (dim == 3) rho2 += v[2] * v[2];
    double rho = sqrt(rho2);
    if (rho == 0.0) return false;
    for (int i = 0; i < dim; ++i) n[i] = v[i] / rho;
    psi = s.r0 - rho;
    return true;
  }
  double S[3] = {0.0, 0.0, 0.0};
  bool ok = false;
  if (s.kind == kStar2D) {
    // Gauss-Newton on a fixed chart of directions u(a) ~ w0 + a t0
    double rho = sqrt(v[0] * v[0] + v[1] * v[1]);
    if (rho == 0.0) return false;
    double w0[2] = {v[0] / rho, v[1] / rho}, t0[2] = {-w0[1], w0[0]};
    double a = 0.0, last = 1.0;
    int good = 0;
    for (int it = 0; it < 80 && good < 2; ++it) {
      double q0 = w0[0] + a * t0[0], q1 = w0[1] + a * t0[1];
      double nv = sqrt(q0 * q0 + q1 * q1);
      double u0 = q0 / nv, u1 = q1 / nv, r, r1;
      star_r(s, u0, u1, r, r1);
      double fac = (-u1 * t0[0] + u0 * t0[1]) / nv;
      double J0 = fac * (r1 * u0 - r * u1), J1 = fac * (r1 * u1 + r * u0);
      double R0 = s.c[0] + r * u0 - x[0], R1 = s.c[1] + r * u1 - x[1];
      double da = -(J0 * R0 + J1 * R1) / (J0 * J0 + J1 * J1);
      a += da;
      last = fabs(da);
      good = last < 1e-15 ? good + 1 : 0;
    }
    ok = good >= 2 || last < 1e-13;
    double q0 = w0[0] + a * t0[0], q1 = w0[1] + a * t0[1];
    double nv = sqrt(q0 * q0 + q1 * q1);
    double u0 = q0 / nv, u1 = q1 / nv, r, r1;
    if (!ok) {
      // Gauss-Newton leaves out the curvature term, so it crawls (or
      // wanders) where the point is nearly as deep as the boundary's radius
      // of curvature: a second-layer candidate inside a tight bend.  Newton
      // on the polar angle from where it stopped, with that term (f = |X -
      // x|^2 / 2, f' = R.X', f'' = X'.X' + R.X''), taking the Gauss-Newton
      // step wherever f'' is not positive.
      double th = atan2(u1, u0);
      good = 0;
      last = 1.0;
      for (int it = 0; it < 60 && good < 2; ++it) {
        double sn, cs, r2;
        sincos(th, &sn, &cs);
        star_r2(s, cs, sn, r, r1, r2);
        const double D1x = r1 * cs - r * sn, D1y = r1 * sn + r * cs;
        const double D2x = (r2 - r) * cs - 2.0 * r1 * sn, D2y = (r2 - r) * sn + 2.0 * r1 * cs;
        const double Rx = s.c[0] + r * cs - x[0], Ry = s.c[1] + r * sn - x[1];
        const double g1 = Rx * D1x + Ry * D1y;
        double g2 = D1x * D1x + D1y * D1y + Rx * D2x + Ry * D2y;
        if (!(g2 > 0.0)) g2 = D1x * D1x + D1y * D1y;
        const double dth = -g1 / g2;
        th += dth;
        last = fabs(dth);
        good = last < 1e-15 ? good + 1 : 0;
      }
      ok = good >= 2 || last < 1e-13;
      sincos(th, &u1, &u0);
    }
    star_r(s, u0, u1, r, r1);
    S[0] = s.c[0] + r * u0;
    S[1] = s.c[1] + r * u1;
    // tangent dX/dtheta = r' u + r u_perp; outward normal = tangent turned clockwise
    double T0 = r1 * u0 - r * u1, T1 = r1 * u1 + r * u0;
    double tn = sqrt(T0 * T0 + T1 * T1);
    n[0] = T1 / tn;
    n[1] = -T0 / tn;
  } else if (s.kind == kShStar) {
    double rho = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    if (rho == 0.0) return false;
    double w0[3] = {v[0] / rho, v[1] / rho, v[2] / rho};
    int ax = 0;
    if (fabs(w0[1]) < fabs(w0[ax])) ax = 1;
    if (fabs(w0[2]) < fabs(w0[ax])) ax = 2;
    double t1[3] = {0.0, 0.0, 0.0};
    t1[ax] = 1.0;
    double dd = w0[ax];
    for (int i = 0; i < 3; ++i) t1[i] -= dd * w0[i];
    double tl = sqrt(t1[0] * t1[0] + t1[1] * t1[1] + t1[2] * t1[2]);
    for (int i = 0; i < 3; ++i) t1[i] /= tl;
    double t2[3] = {w0[1] * t1[2] - w0[2] * t1[1], w0[2] * t1[0] - w0[0] * t1[2],
                    w0[0] * t1[1] - w0[1] * t1[0]};
    double p1 = 0.0, p2 = 0.0, last = 1.0;
    int good = 0;
    for (int it = 0; it < 80 && good < 2; ++it) {
      double q[3], u[3], r, g[3];
      for (int i = 0; i < 3; ++i) q[i] = w0[i] + p1 * t1[i] + p2 * t2[i];
      double nv = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
      for (int i = 0; i < 3; ++i) u[i] = q[i] / nv;
      sh_r(s, u, r, g);
      double ut1 = u[0] * t1[0] + u[1] * t1[1] + u[2] * t1[2];
      double ut2 = u[0] * t2[0] + u[1] * t2[1] + u[2] * t2[2];
      double J1[3], J2[3], R[3];
      double du1[3], du2[3];
      for (int i = 0; i < 3; ++i) {
        du1[i] = (t1[i] - ut1 * u[i]) / nv;
        du2[i] = (t2[i] - ut2 * u[i]) / nv;
      }
      double dr1 = g[0] * du1[0] + g[1] * du1[1] + g[2] * du1[2];
      double dr2 = g[0] * du2[0] + g[1] * du2[1] + g[2] * du2[2];
      for (int i = 0; i < 3; ++i) {
        J1[i] = dr1 * u[i] + r * du1[i];
        J2[i] = dr2 * u[i] + r * du2[i];
        R[i] = s.c[i] + r * u[i] - x[i];
      }
      double a11 = 0, a12 = 0, a22 = 0, b1 = 0, b2 = 0;
      for (int i = 0; i < 3; ++i) {
        a11 += J1[i] * J1[i];
        a12 += J1[i] * J2[i];
        a22 += J2[i] * J2[i];
        b1 -= J1[i] * R[i];
        b2 -= J2[i] * R[i];
      }
      double det = a11 * a22 - a12 * a12;
      double d1 = (b1 * a22 - b2 * a12) / det, d2 = (a11 * b2 - a12 * b1) / det;
      p1 += d1;
      p2 += d2;
      last = fabs(d1) + fabs(d2);
      good = last < 1e-15 ? good + 1 : 0;
    }
    ok = good >= 2 || last < 1e-13;
    double q[3], u[3], r, g[3];
    for (int i = 0; i < 3; ++i) q[i] = w0[i] + p1 * t1[i] + p2 * t2[i];
    double nv = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
    for (int i = 0; i < 3; ++i) u[i] = q[i] / nv;
    sh_r(s, u, r, g);
    for (int i = 0; i < 3; ++i) {
      S[i] = s.c[i] + r * u[i];
      n[i] = u[i] - g[i] / r;   // gradient of |y - c| - r(direction)
    }
    double nl = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    for (int i = 0; i < 3; ++i) n[i] /= nl;
  } else if (s.kind == kAirfoil) {
    double dx = (x[0] - s.c[0]) / s.chord, dy = (x[1] - s.c[1]) / s.chord;
    double b0 = s.ca * dx - s.sa * dy, b1 = s.sa * dx + s.ca * dy;
    double xc = b0 < 0.0 ? 0.0 : (b0 > 1.0 ? 1.0 : b0);
    double sp = sqrt(xc);
    double best = 1e300, bs = 0.0;
    ok = true;
    for (int br = 0; br < 2; ++br) {
      double lo = br == 0 ? 0.0 : -1.0, hi = br == 0 ? 1.0 : 0.0;
      double sv = br == 0 ? sp : -sp;
      if (sv == 0.0) sv = br == 0 ? 1e-3 : -1e-3;
      double last = 1.0;
      // Newton on the squared distance along the contour parameter, clamped
      // to the branch; the Gauss-Newton step where the curvature term makes
      // the second derivative non-positive
      for (int it = 0; it < 200 && last > 1e-15; ++it) {
        double C[2], D[2], E[2];
        naca_point(s.thick, sv, C, D, E);
        const double r0 = C[0] - b0, r1 = C[1] - b1;
        const double dd = D[0] * D[0] + D[1] * D[1];
        double h = dd + r0 * E[0] + r1 * E[1];
        if (!(h > 0.0)) h = dd;
        double ns = sv - (r0 * D[0] + r1 * D[1]) / h;
        ns = ns < lo ? lo : (ns > hi ? hi : ns);
        last = fabs(ns - sv);
        sv = ns;
      }
      if (last > 1e-12) ok = false;
      double C[2], D[2], E[2];
      naca_point(s.thick, sv, C, D, E);
      double d2 = (C[0] - b0) * (C[0] - b0) + (C[1] - b1) * (C[1] - b1);
      if (d2 < best) {
        best = d2;
        bs = sv;
      }
    }
    double C[2], D[2], E[2], nb[2];
    naca_point(s.thick, bs, C, D, E);
    if (fabs(bs) >= 1.0) {
      // trailing-edge corner: the normal is the direction from the corner
      double e0 = b0 - C[0], e1 = b1 - C[1];
      double el = sqrt(e0 * e0 + e1 * e1);
      nb[0] = (solid ? -e0 : e0) / el;
      nb[1] = (solid ? -e1 : e1) / el;
    } else {
      // contour is clockwise in s: outward normal = tangent turned counter-clockwise
      double dl = sqrt(D[0] * D[0] + D[1] * D[1]);
      nb[0] = -D[1] / dl;
      nb[1] = D[0] / dl;
    }
    n[0] = s.ca * nb[0] + s.sa * nb[1];
    n[1] = -s.sa * nb[0] + s.ca * nb[1];
    S[0] = s.c[0] + s.chord * (s.ca * C[0] + s.sa * C[1]);
    S[1] = s.c[1] + s.chord * (-s.sa * C[0] + s.ca * C[1]);
  } else {
    return false;
  }
  double d2 = 0.0;
  for (int i = 0; i < dim; ++i) d2 += (x[i] - S[i]) * (x[i] - S[i]);
  psi = solid ? sqrt(d2) : -sqrt(d2);
  return ok;
}

// --------------------------------------------------------------------------
// 2. scans and compactions
// --------------------------------------------------------------------------

__global__ void k_zero_words(int32_t* __restrict__ a, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0;
}

// excl[i] = sum cnt[0..i), excl[n] = total.  If list is given, the indices
// i with cnt[i] > 0 are written to it in ascending order and their number
// to nlist[0]: each count carries a flag in bits 31 and up, so one scan
// yields both (their sum stays below 2^31).  Tiles of 8 values per thread.
constexpr int kScanT = 8;
constexpr int64_t kScanHi = int64_t(1) << 31;

__device__ __forceinline__ void scan_load(const int32_t* __restrict__ cnt, int64_t n, int64_t b,
                                          int v[kScanT]) {
  const bool vec = (reinterpret_cast<uintptr_t>(cnt) & 15) == 0;
  if (vec && b + kScanT <= n) {
    const int4 a = *reinterpret_cast<const int4*>(cnt + b);
    const int4 c = *reinterpret_cast<const int4*>(cnt + b + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
  } else {
#pragma unroll
    for (int q = 0; q < kScanT; ++q) v[q] = b + q < n ? cnt[b + q] : 0;
  }
}

// the packed sum of a thread's values
__device__ __forceinline__ int64_t scan_sum(const int v[kScanT]) {
  int64_t sum = 0;
#pragma unroll
  for (int q = 0; q < kScanT; ++q) sum += v[q] + (v[q] > 0 ? kScanHi : 0);
  return sum;
}

// the values from b on, `run` the packed sum before them
__device__ __forceinline__ void scan_store(const int v[kScanT], int64_t n, int64_t b, int64_t run,
                                           int64_t* excl, int32_t* __restrict__ list) {
#pragma unroll
  for (int q = 0; q < kScanT; ++q) {
    if (b + q < n) {
      excl[b + q] = run & (kScanHi - 1);
      if (list && v[q] > 0) list[run >> 31] = (int32_t)(b + q);
    }
    run += v[q] + (v[q] > 0 ? kScanHi : 0);
  }
}

template <bool Others>
__device__ __forceinline__ int64_t scanned(const int64_t* p) {
  return Others ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}

// Offsets of the instances from the scan of their chunks, and what follows
// from them: off[i] = excl[start[i]]; with hoff, the instances' cell tables
// too (a power of two, at least 64 and twice the interface cells: at most half
// full).  The offsets, the listed chunks and the band segments go to the host
// as well (pinned memory), so nothing is copied back or up between the halves
// of a build.  By the last workgroup of the scan to finish; where there are
// others, what they stored is read past its own caches.
template <int BS, bool Others>
__device__ __forceinline__ void instance_offsets(const ScanOffsets& O, const int64_t* excl,
                                                 int32_t nlisted, int64_t* sh) {
  int64_t carry = 0;
  for (int i0 = 0; i0 <= O.ninst; i0 += BS) {
    const int i = i0 + (int)threadIdx.x;
    int64_t at = 0, size = 0;
    if (i <= O.ninst) {
      at = scanned<Others>(excl + O.start[i]);
      O.off[i] = at;
      O.host_off[i] = at;
    }
    if (!O.hoff) continue;
    if (i < O.ninst) {
      const int64_t twice = 2 * (scanned<Others>(excl + O.start[i + 1]) - at);
      size = 64;
      while (size < twice) size <<= 1;
      O.hmask[i] = (uint32_t)(size - 1);
    }
    int64_t tot;
    const int64_t before = carry + block_excl_scan<BS>(size, &tot, sh);
    if (i <= O.ninst) O.hoff[i] = before;
    carry += tot;
  }
  if (!O.hoff) return;
  if (threadIdx.x < 64) {
    int v = 0;
    for (int q = threadIdx.x; q < kBandStripes; q += 64) v += O.nband[q * 16];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if (threadIdx.x == 0) {
      O.host_counts[0] = nlisted;
      O.host_counts[1] = v;
    }
  }
}

// Elements before workgroup b's own `tot`, for workgroups numbered in the
// order they started (a single-pass scan with look-back, Merrill and Garland,
// 2016, the look-back by the whole workgroup): each posts its count, sums those posted before it, BS at
// a time, back to the nearest that has posted its sum, and posts its own sum.
// Workgroups wait only for ones that started earlier and post their counts
// without waiting, so every wait ends.  (Called by all BS threads.)  The
// numbers come from one counter, about 20 ns each across the chip, so where
// there would be more than a few hundred workgroups they are larger instead.
constexpr unsigned long long kPostCount = 1ull << 62, kPostSum = 2ull << 62;
template <int BS>
__device__ __forceinline__ int64_t posted_before(unsigned long long* __restrict__ posted, int b,
                                                 int64_t tot) {
  __shared__ int64_t s_sum[BS / 64];
  __shared__ int s_end[BS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid == 0)
    __hip_atomic_store(&posted[b], (b == 0 ? kPostSum : kPostCount) | (unsigned long long)tot,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int64_t before = 0;
  for (int top = b; top > 0; top -= BS) {
    const int j = top - 1 - tid;
    unsigned long long v = kPostSum;   // (before the first: nothing)
    if (j >= 0)
      while ((v = __hip_atomic_load(&posted[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
      }
    const unsigned long long sums = __ballot((v & kPostSum) != 0);
    const int end = sums ? __ffsll(sums) - 1 : 64;
    int64_t x = lane <= end ? (int64_t)(v & (kPostCount - 1)) : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if (lane == 0) {
      s_sum[wv] = x;
      s_end[wv] = end;
    }
    __syncthreads();
    bool found = false;
    for (int w = 0; w < BS / 64 && !found; ++w) {
      before += s_sum[w];
      found = s_end[w] < 64;
    }
    __syncthreads();
    if (found) break;
  }
  if (tid == 0 && b > 0)
    __hip_atomic_store(&posted[b], kPostSum | (unsigned long long)(before + tot), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  return before;
}

// Short inputs: the whole scan by one workgroup, and the offsets if asked for.
__global__ __launch_bounds__(1024) void k_scan(const int32_t* __restrict__ cnt, int64_t n,
                                               int64_t* excl, int32_t* __restrict__ list,
                                               int32_t* nlist, ScanOffsets O) {
  __shared__ int64_t sh[17];
  int64_t carry = 0;
  for (int64_t t0 = 0; t0 < n; t0 += 1024 * kScanT) {
    const int64_t b = t0 + (int64_t)threadIdx.x * kScanT;
    int v[kScanT];
    scan_load(cnt, n, b, v);
    int64_t tot;
    const int64_t before = block_excl_scan<1024>(scan_sum(v), &tot, sh);
    scan_store(v, n, b, carry + before, excl, list);
    carry += tot;
  }
  if (threadIdx.x == 0) {
    excl[n] = carry & (kScanHi - 1);
    if (nlist) nlist[0] = (int32_t)(carry >> 31);
  }
  if (!O.off) return;
  __syncthreads();   // the scan's values, before they are read back
  instance_offsets<1024, false>(O, excl, (int32_t)(carry >> 31), sh);
}

// Longer ones: a tile per workgroup, the sums before it from what the
// workgroups post (posted: [tiles], then the numbers started and finished,
// from zero).  32,768 chunks of a 512^3 grid: 7.1 us in one launch, in three
// (totals, their scan, the tiles again) 15 and their gaps.
__global__ __launch_bounds__(256) void k_scan_tiles(const int32_t* __restrict__ cnt, int64_t n,
                                                    int64_t* excl, int32_t* __restrict__ list,
                                                    int32_t* nlist,
                                                    unsigned long long* __restrict__ posted,
                                                    ScanOffsets O) {
  __shared__ int64_t sh[5];
  __shared__ int s_b, s_nlist;
  if (threadIdx.x == 0) s_b = (int)atomicAdd(&posted[gridDim.x], 1ull);
  __syncthreads();
  const int t = s_b;
  const int64_t b = ((int64_t)t * 256 + threadIdx.x) * kScanT;
  int v[kScanT];
  scan_load(cnt, n, b, v);
  int64_t tot;
  const int64_t rank = block_excl_scan<256>(scan_sum(v), &tot, sh);
  const int64_t before = posted_before<256>(posted, t, tot);
  scan_store(v, n, b, before + rank, excl, list);
  if (t == (int)gridDim.x - 1 && threadIdx.x == 0) {
    excl[n] = (before + tot) & (kScanHi - 1);
    if (nlist) nlist[0] = (int32_t)((before + tot) >> 31);
  }
  if (!O.off) return;   // uniform
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) {
    s_b = atomicAdd(&posted[gridDim.x + 1], 1ull) == gridDim.x - 1;
    __threadfence();
    if (s_b) s_nlist = __hip_atomic_load(nlist, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (s_b) instance_offsets<256, true>(O, excl, s_nlist, sh);   // uniform
}

// One workgroup takes 8,192 values about as fast as four launched with their
// posts (4 us); `posted`: scan_words(n) zeroed words.
constexpr int64_t kScanAlone = 1024 * kScanT, kScanTile = 256 * kScanT;
int64_t scan_words(int64_t n) { return n <= kScanAlone ? 0 : (n + kScanTile - 1) / kScanTile + 2; }
void launch_scan(const int32_t* cnt, int64_t n, int64_t* excl, int32_t* list, int32_t* nlist,
                 unsigned long long* posted, hipStream_t st, const ScanOffsets* O) {
  const ScanOffsets o = O ? *O : ScanOffsets{};
  if (n <= kScanAlone)
    k_scan<<<1, 1024, 0, st>>>(cnt, n, excl, list, nlist, o);
  else
    k_scan_tiles<<<(unsigned)((n + kScanTile - 1) / kScanTile), 256, 0, st>>>(cnt, n, excl, list,
                                                                             nlist, posted, o);
}

// Fresh cells of a moved body (Sec. 7.1: a moving boundary exposes fresh
// fluid cells): cells whose centre was solid before the move (tag 1 or 2)
// and is fluid after it (tag 0 or -2); uncovered ones were not ghosts before
// (tag 1), so no value was ever reconstructed there.  Tags (their
// arrays are 256-byte aligned) are not read where both plans settled their
// span to the same class (each of its cells lies on that side of both
// boundaries).  One launch counts, a tile or several to a workgroup; in the next
// each workgroup sums the counts before its own, and lists, reading again only
// where there are fresh cells.  No workgroup waits for another: the counts lie
// in scratch of the plan, which calls on two streams may share.  A call at 64^3
// 12.5 us, 256^3 14.2, 400^3 30, 1024^3 232; with a launch between that scans
// the counts 15, 23, 50, 660; in one pass of workgroups that post their counts
// to each other, behind a launch that clears them, 16, 14.7, 33.5, 406.
__device__ __forceinline__ uint32_t fresh_bits(const int8_t* __restrict__ a,
                                               const int8_t* __restrict__ b, int64_t base,
                                               int64_t n, int& unc) {
  uint32_t m = 0;
  unc = 0;
  int8_t ta[kSeg], tb[kSeg];
  if (base + kSeg <= n) {
    *reinterpret_cast<uint4*>(ta) = *reinterpret_cast<const uint4*>(a + base);
    *reinterpret_cast<uint4*>(tb) = *reinterpret_cast<const uint4*>(b + base);
  } else {
    for (int q = 0; q < kSeg; ++q) {
      ta[q] = base + q < n ? a[base + q] : 0;
      tb[q] = base + q < n ? b[base + q] : 0;
    }
  }
#pragma unroll
  for (int q = 0; q < kSeg; ++q)
    if ((ta[q] == 1 || ta[q] == 2) && (tb[q] == 0 || tb[q] == -2)) {
      m |= 1u << q;
      unc += ta[q] == 1;
    }
  return m;
}

// A workgroup takes `tiles` tiles in turn, the next one's spans read ahead.
// count [workgroups]: a workgroup's fresh cells, the uncovered ones from bit 31
// on (not read for a grid of one, which the listing launch alone takes).
constexpr int kFreshBS = 1024;   // (a wave's part of a tile is a span)
constexpr int64_t kFreshTile = (int64_t)kFreshBS * kSeg;
// Workgroups at most, as each sums the counts before its own and an empty one
// costs its start too: what the chip holds at once where that leaves no more
// than two tiles to each (256^3: 14.2 us a call, one tile each 16.6), else four
// times that (1024^3, us a call with 1024, 2048 and 4096: 296, 232, 344; 400^3:
// 38, 30, 35).
constexpr int64_t kFreshGroups = 2048, kFreshRound = 512;
template <bool List>
__global__ __launch_bounds__(kFreshBS) void k_fresh(const int8_t* __restrict__ a,
                                                    const int8_t* __restrict__ b,
                                                    const int8_t* __restrict__ sa,
                                                    const int8_t* __restrict__ sb, int64_t n,
                                                    int tiles, int64_t* __restrict__ count,
                                                    int64_t* __restrict__ counts,
                                                    int32_t* __restrict__ list, int64_t cap) {
  __shared__ int64_t sh[kFreshBS / 64 + 1];
  const int g = (int)blockIdx.x;
  int64_t base = (int64_t)g * tiles * kFreshTile + (int64_t)threadIdx.x * kSeg;
  int8_t x = 0, y = 0;
  auto spans = [&](int64_t at) {
    x = at < n ? sa[at / (64 * kSeg)] : 0;
    y = at < n ? sb[at / (64 * kSeg)] : 0;
  };
  spans(base);
  int64_t first = 0, sum = 0;
  if (List && gridDim.x > 1) {
    const int64_t own = count[g];
    const bool last = g == (int)gridDim.x - 1;
    if (own == 0 && !last) return;   // uniform
    int64_t v = 0;
    for (int j = threadIdx.x; j < g; j += kFreshBS) v += count[j];
    (void)block_excl_scan<kFreshBS>(v, &first, sh);
    if (last && threadIdx.x == 0) {
      counts[0] = (first + own) & (kScanHi - 1);
      counts[1] = (first + own) >> 31;
    }
    first &= kScanHi - 1;
  }
  for (int t = 0; t < tiles; ++t, base += kFreshTile) {
    const bool read = x < 0 || x != y;
    if (t + 1 < tiles) spans(base + kFreshTile);
    int unc = 0;
    const uint32_t m = read ? fresh_bits(a, b, base, n, unc) : 0u;
    const int64_t mine = __popc(m) | (int64_t)unc << 31;
    sum += mine;
    if (!List || (gridDim.x > 1 && !__syncthreads_or(m != 0))) continue;   // uniform
    int64_t tot;
    int64_t pos = first + (block_excl_scan<kFreshBS>(mine, &tot, sh) & (kScanHi - 1));
    for (uint32_t w = m; w; w &= w - 1, ++pos)
      if (pos < cap) list[pos] = (int32_t)(base + __ffs(w) - 1);
    first += tot & (kScanHi - 1);
    if (gridDim.x == 1 && threadIdx.x == 0) {   // (one tile)
      counts[0] = tot & (kScanHi - 1);
      counts[1] = tot >> 31;
    }
  }
  if (!List) {
    int64_t tot;
    (void)block_excl_scan<kFreshBS>(sum, &tot, sh);
    if (threadIdx.x == 0) count[g] = tot;
  }
}

extern "C" gcr_status gcr_plan_fresh_cells(const gcr_plan* a, const gcr_plan* b, int64_t* counts,
                                           int32_t* list, int64_t cap, void* stream) {
  if (!plan_ok(a) || !plan_ok(b) || !counts || cap < 0 || (cap > 0 && !list)) return GCR_E_ARG;
  if (a->dim != b->dim || a->ncell != b->ncell) return GCR_E_ARG;
  for (int ax = 0; ax < 3; ++ax)
    if (a->inst.g.n[ax] != b->inst.g.n[ax] || a->inst.g.lo[ax] != b->inst.g.lo[ax] ||
        a->inst.g.h[ax] != b->inst.g.h[ax])
      return GCR_E_ARG;
  hipStream_t st = (hipStream_t)stream;
  const int64_t n = a->ncell, ntiles = (n + kFreshTile - 1) / kFreshTile;
  const int64_t most = ntiles <= 2 * kFreshRound ? kFreshRound : kFreshGroups;
  const int tiles = (int)((ntiles + most - 1) / most);
  const unsigned groups = (unsigned)((ntiles + tiles - 1) / tiles);
  int64_t* const count = static_cast<int64_t*>(
      plan_scratch(const_cast<gcr_plan*>(b), 6, sizeof(int64_t) * groups));
  if (!count) return GCR_E_NOMEM;
  const int64_t room = list ? cap : 0;
  if (groups > 1)
    k_fresh<false><<<groups, kFreshBS, 0, st>>>(a->tags, b->tags, a->span, b->span, n, tiles, count,
                                                counts, list, room);
  k_fresh<true><<<groups, kFreshBS, 0, st>>>(a->tags, b->tags, a->span, b->span, n, tiles, count,
                                             counts, list, room);
  GCR_HIP(hipGetLastError());
  return GCR_OK;
}

// Second ghost layer (Sec. 7.1): the solid cells within R_i cells along each
// axis i of a solid interface cell, R_i = floor((1.5 + sqrt(d)/2) w_max /
// w_min_i) + 1 (w_max the largest cell width, w_min_i the smallest along i;
// h_max / h_i on a uniform grid; set per instance on the host), get the
// candidate mark 0x20.  Every cell with psi <= 1.5 delta n is among them: a
// walk from it through its foot point reaches a fluid centre within that
// box (delta n <= w_max, psi 1-Lipschitz), and the last solid cell before it
// is a solid interface cell.
//
// Around a sphere that lies inside the grid with that walk's room to spare
// (l2tight, set on the host) the walk needs less than the box: beyond the
// foot point it stays outside the ball, so its end, D = (1.5 + sqrt(d)/2) w
// from the candidate's centre, is fluid, w the largest width of the cells
// it can meet.  Those lie within R of the interface cell x it crosses, so w
// is taken over that range instead of the grid, and along each axis the
// candidate's centre is within D of x's own interval.  l2_reach finds that
// interval of indices (a few face reads); with R = 7 (widths 2.6 : 1) it is
// 5 cells an axis at the body instead of 15, with R = 3 it is 5 instead of
// 7.  Bodies of other kinds, and spheres the grid cuts, keep the box.
//
// kL2Split workgroups per chunk of the interface chunk list (striding over it):
// each lists the chunk's solid interface cells in LDS, in index order, and
// takes every kL2Split-th batch of kL2Batch of them (at a sphere's poles a
// chunk holds over a thousand, a dozen times the mean, and one workgroup took
// them in 114 us).  A thread finds one cell's reach, then the workgroup walks
// the (cell, row of its box) items, a row's tags read eight at a time (any
// alignment) and kFly rows in flight per thread before any mark is set.
// Bound by the rows' loads: they overlap heavily and hit in cache.  190^3
// stretched by 1.01 a cell: 1459 -> 49 us; 256^3: 89 -> 21 us (one load per
// box cell before, the box for every body, one workgroup a chunk).
constexpr double kL2Slack = 1.0 + 1e-9;   // dwarfs the rounding of the reach
constexpr int kL2Batch = 64, kL2Split = 8, kL2Grid = 2048;

// faces i - kL2Win .. i + 1 + kL2Win of a stretched axis, read together (a
// loop that stops at a face would pay a round trip a step)
constexpr int kL2Win = 8;
__device__ __forceinline__ void l2_faces(const double* f, int n, int i,
                                         double w[2 * kL2Win + 2]) {
#pragma unroll
  for (int q = 0; q < 2 * kL2Win + 2; ++q) w[q] = f[min(max(i - kL2Win + q, 0), n)];
}

// largest width along axis a of the cells at most R from cell i
__device__ __forceinline__ double l2_width(const GridD& g, int a, int i, int R) {
  if (!g.face[a]) return g.h[a];
  double f[2 * kL2Win + 2], w = 0.0;
  l2_faces(g.face[a], g.n[a], i, f);
#pragma unroll
  for (int q = 0; q <= 2 * kL2Win; ++q)   // (cells off the grid: zero width)
    if (abs(q - kL2Win) <= R) w = fmax(w, f[q + 1] - f[q]);
  for (int q = kL2Win + 1; q <= R; ++q) {
    if (i - q >= 0) w = fmax(w, width(g, a, i - q));
    if (i + q < g.n[a]) w = fmax(w, width(g, a, i + q));
  }
  return w;
}

// [lo, hi]: indices along axis a whose cell centres lie within D of cell
// i's own interval, at most R cells away and inside the grid
__device__ __forceinline__ void l2_reach(const GridD& g, int a, int i, int R, double D, int& lo,
                                         int& hi) {
  const int n = g.n[a];
  if (!g.face[a]) {
    const int r = min(R, (int)floor(D / g.h[a] + 0.5));
    lo = max(i - r, 0);
    hi = min(i + r, n - 1);
    return;
  }
  double f[2 * kL2Win + 2];
  l2_faces(g.face[a], n, i, f);
  const double f0 = f[kL2Win], f1 = f[kL2Win + 1];
  int dn = 0, up = 0;   // centres move away monotonically: the reach is a run
#pragma unroll
  for (int q = 1; q <= kL2Win; ++q) {
    if (q <= R && i - q >= 0 && f0 - 0.5 * (f[kL2Win - q] + f[kL2Win - q + 1]) <= D) dn = q;
    if (q <= R && i + q < n && 0.5 * (f[kL2Win + q] + f[kL2Win + q + 1]) - f1 <= D) up = q;
  }
  if (dn == kL2Win)
    while (dn < R && i - dn - 1 >= 0 && f0 - centre(g, a, i - dn - 1) <= D) ++dn;
  if (up == kL2Win)
    while (up < R && i + up + 1 < n && centre(g, a, i + up + 1) - f1 <= D) ++up;
  lo = i - dn;
  hi = i + up;
}

__global__ __launch_bounds__(256) void k_l2_mark(const Inst* __restrict__ insts, int ninst,
                                                 const int64_t* __restrict__ chunk_start,
                                                 const int32_t* __restrict__ chunk_list,
                                                 const int32_t* __restrict__ nlist,
                                                 int8_t* __restrict__ tags,
                                                 int32_t* __restrict__ dirty,
                                                 int32_t* __restrict__ dlist,
                                                 int32_t* __restrict__ ndirty) {
  __shared__ uint16_t s_cell[kChunk];       // cells within the chunk
  __shared__ int s_at[kL2Batch];            // first cell of the box of each cell of the batch
  __shared__ uint8_t s_len[3][kL2Batch];    // its size along each axis
  __shared__ int s_w[3];
  __shared__ int64_t sh[5];
  for (int it = blockIdx.x; it < nlist[0]; it += gridDim.x) {
    const int64_t chunk = chunk_list[it];
    const int ii = find_inst(chunk_start, ninst, chunk);
    const Inst& I = insts[ii];
    if (!I.layer2) continue;
    const GridD g = I.g;
    const int8_t* T = tags + I.cell_off;
    const int64_t base = (chunk - I.chunk_off) * kChunk;
    int n;
    {
      // 16 cells a thread, one 16-byte load
      const int t0 = (int)threadIdx.x * kSeg;
      uint32_t mask = 0;
      if (base + t0 + kSeg <= g.ncell) {
        const uint4 w = *reinterpret_cast<const uint4*>(T + base + t0);
        const uint32_t q[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int b = 0; b < kSeg; ++b)
          if (((q[b >> 2] >> (8 * (b & 3))) & 0x41u) == 0x41u) mask |= 1u << b;
      } else {
        for (int b = 0; b < kSeg; ++b)
          if (base + t0 + b < g.ncell && (T[base + t0 + b] & 0x41) == 0x41) mask |= 1u << b;
      }
      // in index order, the same list in every workgroup of the chunk (a mark
      // of another one leaves these two bits as they are)
      int64_t tot;
      int at = (int)block_excl_scan<256>(__popc(mask), &tot, sh);
      n = (int)tot;
      for (; mask; mask &= mask - 1) s_cell[at++] = (uint16_t)(t0 + __ffs(mask) - 1);
    }
    const int R[3] = {I.l2r[0], I.l2r[1], I.l2r[2]};   // 0 beyond the grid's dimension
    const bool tight = I.l2tight != 0;
    const double len = 1.5 + 0.5 * sqrt((double)g.dim);
    for (int b0 = (int)blockIdx.y * kL2Batch; b0 < n; b0 += (int)gridDim.y * kL2Batch) {
      __syncthreads();   // the list is whole; the previous batch's boxes are done
      const int nb = min(kL2Batch, n - b0);
      if (threadIdx.x < 3) s_w[threadIdx.x] = 1;
      __syncthreads();
      if ((int)threadIdx.x < nb) {
        int ijk[3], lo[3], hi[3];
        unlinear(g, (int)(base + s_cell[b0 + threadIdx.x]), ijk[0], ijk[1], ijk[2]);
        double D = 0.0;
        if (tight) {
          double w = 0.0;
#pragma unroll
          for (int a = 0; a < 3; ++a)
            if (a < g.dim) w = fmax(w, l2_width(g, a, ijk[a], R[a]));
          D = len * w * kL2Slack;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          lo[a] = max(ijk[a] - R[a], 0);
          hi[a] = min(ijk[a] + R[a], g.n[a] - 1);
          if (tight && a < g.dim) l2_reach(g, a, ijk[a], R[a], D, lo[a], hi[a]);
          s_len[a][threadIdx.x] = (uint8_t)(hi[a] - lo[a] + 1);   // <= 2 * 64 + 1
          atomicMax(&s_w[a], hi[a] - lo[a] + 1);
        }
        s_at[threadIdx.x] = linear(g, lo[0], lo[1], lo[2]);
      }
      __syncthreads();
      const int P = (s_w[0] + 7) / 8, rows = s_w[1] * s_w[2];   // pieces of a row, rows of a box
      const int per = P * rows, items = nb * per;
      constexpr int kFly = 4;
      for (int i0 = threadIdx.x; i0 < items; i0 += 256 * kFly) {
        int at[kFly];
        unsigned long long m[kFly];
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
          const int it = i0 + u * 256;
          at[u] = 0;
          m[u] = 0ull;
          if (it >= items) continue;
          const int c = it / per;
          int o = it - c * per;
          const int p = o % P;
          o /= P;
          const int dj = o % s_w[1], dk = o / s_w[1];
          const int nx = (int)s_len[0][c] - 8 * p;
          if (nx <= 0 || dj >= s_len[1][c] || dk >= s_len[2][c]) continue;
          at[u] = s_at[c] + 8 * p + g.n[0] * (dj + g.n[1] * dk);
          unsigned long long v = 0ull;
          if ((int64_t)at[u] + 8 <= g.ncell) {
            __builtin_memcpy(&v, T + at[u], 8);
          } else {   // the grid's last cells
            for (int q = 0; q < min(nx, 8); ++q)
              v |= (unsigned long long)(uint8_t)T[at[u] + q] << (8 * q);
          }
          // bytes equal to 1 (plain solid, not yet marked) among the row's
          const unsigned long long x = v ^ 0x0101010101010101ull, l7 = 0x7f7f7f7f7f7f7f7full;
          m[u] = ~(((x & l7) + l7) | x | l7);
          if (nx < 8) m[u] &= (1ull << (8 * nx)) - 1ull;
        }
        // a byte store, as every writer of a cell here stores the same value
        // (1 -> 0x21) and no other kernel runs
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
          if (!m[u]) continue;
          if (dirty) {
            // a re-plan counts marks in the listed chunks only: list those of
            // the first and last cell marked (this workgroup's own is listed)
            const int c0 = at[u] + (__ffsll((long long)m[u]) - 1) / 8;
            const int c1 = at[u] + (63 - __clzll((long long)m[u])) / 8;
            for (int64_t ch = I.chunk_off + c0 / kChunk; ch <= I.chunk_off + c1 / kChunk; ++ch)
              if (ch != chunk && dirty[ch] == 0 && atomicExch(&dirty[ch], 1) == 0)
                dlist[atomicAdd(ndirty, 1)] = (int32_t)ch;
          }
          for (; m[u]; m[u] &= m[u] - 1ull)
            tags[I.cell_off + at[u] + (__ffsll((long long)m[u]) - 1) / 8] = 0x21;
        }
      }
    }
    __syncthreads();   // the list is reused by the next chunk
  }
}

// per chunk: cells with an interface or candidate mark, for every chunk
// (list null) or the chunks of list[0, *nlist) (the classified ones and
// those a candidate mark reached; the others hold none)
__device__ __forceinline__ void count_marks_chunk(int64_t chunk, const Inst* __restrict__ insts,
                                                  int ninst,
                                                  const int64_t* __restrict__ chunk_start,
                                                  const int8_t* __restrict__ tags,
                                                  int32_t* __restrict__ chunk_cnt) {
  __shared__ int s;
  const int ii = find_inst(chunk_start, ninst, chunk);
  const Inst& I = insts[ii];
  if (threadIdx.x == 0) s = 0;
  __syncthreads();
  const int64_t base = (chunk - I.chunk_off) * kChunk + (int64_t)threadIdx.x * kSeg;
  int n = 0;
  if (base + kSeg <= I.g.ncell) {
    const uint4 w = *reinterpret_cast<const uint4*>(tags + I.cell_off + base);
    const uint32_t q[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t m = q[b] & 0x60606060u;   // per byte: bit 0 set iff 0x20 or 0x40 is
      n += __popc(((m >> 5) | (m >> 6)) & 0x01010101u);
    }
  } else {
    for (int b = 0; b < kSeg; ++b)
      if (base + b < I.g.ncell && (tags[I.cell_off + base + b] & 0x60)) ++n;
  }
  if (n) atomicAdd(&s, n);
  __syncthreads();
  if (threadIdx.x == 0) chunk_cnt[chunk] = s;
}

__global__ __launch_bounds__(256) void k_count_marks(const Inst* __restrict__ insts, int ninst,
                                                     const int64_t* __restrict__ chunk_start,
                                                     const int8_t* __restrict__ tags,
                                                     int32_t* __restrict__ chunk_cnt,
                                                     const int32_t* __restrict__ list,
                                                     const int32_t* __restrict__ nlist) {
  if (!list) {   // every chunk, one workgroup each
    count_marks_chunk(blockIdx.x, insts, ninst, chunk_start, tags, chunk_cnt);
    return;
  }
  const int nit = nlist[0];
  for (int it = blockIdx.x; it < nit; it += gridDim.x) {
    count_marks_chunk(list[it], insts, ninst, chunk_start, tags, chunk_cnt);
    __syncthreads();   // s is reused by the next chunk
  }
}

__global__ __launch_bounds__(256) void k_compact_iface(const Inst* __restrict__ insts,
                                                       const int32_t* __restrict__ chunk_inst,
                                                       const int8_t* __restrict__ tags,
                                                       const int32_t* __restrict__ chunk_cnt,
                                                       const int64_t* __restrict__ chunk_excl,
                                                       const int32_t* __restrict__ chunk_list,
                                                       int32_t* __restrict__ if_cell,
                                                       unsigned long long* __restrict__ htab,
                                                       int64_t nhash,
                                                       unsigned long long* __restrict__ posted,
                                                       int64_t nposted) {
  // for k_geometry: the cell -> ghost tables emptied, its counts cleared
  const int64_t z0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t z = z0; z < nhash; z += (int64_t)gridDim.x * blockDim.x) htab[z] = ~0ull;
  for (int64_t z = z0; z < nposted; z += (int64_t)gridDim.x * blockDim.x) posted[z] = 0ull;
  const int64_t chunk = chunk_list[blockIdx.x];   // chunks holding listed cells
  __shared__ int64_t sh[5];
  const int ii = chunk_inst[chunk];
  const Inst& I = insts[ii];
  const int64_t base64 = (chunk - I.chunk_off) * kChunk + (int64_t)threadIdx.x * kSeg;
  uint32_t mask = 0;
  int base = 0;
  if (base64 < I.g.ncell) {
    base = (int)base64;
    const int nvalid = (int)min((int64_t)kSeg, I.g.ncell - base64);
    const int8_t* src = tags + I.cell_off + base;
    if (nvalid == kSeg) {
      const uint4 w = *reinterpret_cast<const uint4*>(src);
      const uint32_t q[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int b = 0; b < kSeg; ++b)
        if ((q[b >> 2] >> (8 * (b & 3))) & 0x60u) mask |= 1u << b;
    } else {
      for (int b = 0; b < nvalid; ++b)
        if (src[b] & 0x60) mask |= 1u << b;
    }
  }
  int64_t tot;
  int64_t pos = chunk_excl[chunk] + block_excl_scan<256>(__popc(mask), &tot, sh);
  while (mask) {
    int b = __ffs(mask) - 1;
    mask &= mask - 1;
    if_cell[pos++] = base + b;
  }
}

// --------------------------------------------------------------------------
// 3. geometry and ghost tags
// --------------------------------------------------------------------------

// The instance of element x of a batch, for lanes whose elements ascend from
// the wave's first, x0: a wave compares 64 offsets at once (find_inst's chain
// of loads once instead of log2 times), then each lane steps on.
__device__ __forceinline__ int find_inst_wave(const int64_t* __restrict__ off, int ninst, int64_t x0,
                                              int64_t x) {
  const int lane = threadIdx.x & 63;
  int i = 0;
  for (int k = 0; k < ninst - 1; k += 64) {
    const int m = __popcll(__ballot(k + lane < ninst - 1 && off[k + lane + 1] <= x0));
    i += m;
    if (m < 64) break;
  }
  while (i < ninst - 1 && off[i + 1] <= x) ++i;
  return i;
}

__device__ __forceinline__ uint32_t table_slot(int c, uint32_t mask) {
  const uint32_t h = (uint32_t)c * 2654435761u;
  return (h ^ (h >> 15)) & mask;
}

// enters (cell c, value v); the table is at most half full
__device__ __forceinline__ uint32_t table_insert(unsigned long long* t, uint32_t mask, int c,
                                                 uint32_t v) {
  const unsigned long long entry = ((unsigned long long)(uint32_t)c << 32) | v;
  uint32_t h = table_slot(c, mask);
  while (atomicCAS(&t[h], ~0ull, entry) != ~0ull) h = (h + 1) & mask;
  return h;
}

// Distance, normal and ghost decision of every interface cell, and the ghosts
// in linear order at once: their positions from the counts that the
// workgroups post to each other (posted: [workgroups], then the number
// started), so that one launch does what four did (the cells' arrays written,
// counted, scanned, read back) and the ghosts enter the cell table too.
// Bound by the latency of the projection and of the insertion.  With the
// statistics folded and the results stored by k_finalize, a build went from 14
// launches and a copy after the compaction to 4: 128^2 circle 174 -> 117 us
// for the whole build, fill and read-out, 64 stars 483 -> 375, 512^3 sphere
// 349 -> 316.
// Workgroups of 256 up to this many interface cells, of 1024 beyond (see
// posted_before), which wait for the slowest of more projections but are
// numbered sooner.  Spheres, with 256 / 1024: 1,332 cells 9.6 / 11.3 us, 33,435
// 11.8 / 13.5, 54,759 13.8 / 16.1, 85,532 16.8 / 15.2, 219,077 33.0 / 20.7.
constexpr int64_t kGeometrySmall = 65536;

template <int BS>
__global__ __launch_bounds__(BS) void k_geometry(
    const Inst* __restrict__ insts, int ninst, const int64_t* __restrict__ if_off,
    const int32_t* __restrict__ if_cell, int8_t* __restrict__ tags, int64_t cap,
    unsigned long long* __restrict__ posted, const int64_t* __restrict__ hoff,
    const uint32_t* __restrict__ hmask, unsigned long long* __restrict__ htab,
    int64_t* __restrict__ g_off, int32_t* __restrict__ g_cell, double* __restrict__ g_psi,
    double* __restrict__ g_n, uint8_t* __restrict__ g_ext, uint32_t* __restrict__ g_slot,
    int32_t* __restrict__ flow, InstInfo* __restrict__ info) {
  __shared__ int s_b;
  __shared__ int64_t sh[BS / 64 + 1];
  if (threadIdx.x == 0) s_b = (int)atomicAdd(&posted[gridDim.x], 1ull);
  __syncthreads();
  const int b = s_b;
  const int64_t nif = if_off[ninst], e0 = (int64_t)b * BS, e = e0 + threadIdx.x;
  const bool valid = e < nif;
  const int ii = find_inst_wave(if_off, ninst, e0 + (threadIdx.x & ~63), min(e, nif - 1));
  int c = 0;
  double n[3] = {0.0, 0.0, 0.0}, psi = 0.0;
  bool ghost = false, ext = false;
  if (valid) {
    const Inst& I = insts[ii];
    const GridD& g = I.g;
    c = if_cell[e];
    int8_t* tp = tags + I.cell_off + c;
    const int8_t t0 = *tp;
    const bool solid = (t0 & 1) != 0;
    const bool iface = (t0 & 0x40) != 0;   // else a second-layer candidate
    int i, j, k;
    unlinear(g, c, i, j, k);
    double x[3] = {centre(g, 0, i), centre(g, 1, j), g.dim == 3 ? centre(g, 2, k) : 0.0};
    bool ok = project(I.s, g.dim, x, solid, n, psi);
    if (!ok) atomicOr(&info[ii].err, kErrGeometry);
    // Eq. delta_n with the cell's own widths
    const int ijk[3] = {i, j, k};
    double sum = 0.0;
    for (int a = 0; a < g.dim; ++a) {
      const double w = width(g, a, ijk[a]);
      sum += (n[a] / w) * (n[a] / w);
    }
    double dn = 1.0 / sqrt(sum);
    if (iface) {
      if (I.scheme == kHGC) ghost = solid ? (psi <= dn / 2.0) : (-psi < dn / 2.0);
      else ghost = solid;
    }
    // Sec. 7.1: a second layer adds the solid cells with psi <= 1.5 delta n,
    // reconstructed on the extended stencil
    ext = I.layer2 && solid && !ghost && psi <= 1.5 * dn;
    ghost = ghost || ext;
    *tp = ghost ? (solid ? 2 : -2) : (solid ? 1 : 0);
    if (g.dim == 2) n[2] = 0.0;   // the third normal component of 2D ghosts
  }
  int64_t tot;
  const int64_t rank = block_excl_scan<BS>(ghost ? 1 : 0, &tot, sh);
  const int64_t pos = posted_before<BS>(posted, b, tot) + rank;
  if (ghost) {
    g_ext[pos] = ext ? 1 : 0;
    g_cell[pos] = c;
    g_psi[pos] = psi;
    for (int a = 0; a < 3; ++a) g_n[a * cap + pos] = n[a];
    g_slot[pos] = table_insert(htab + hoff[ii], hmask[ii], c, (uint32_t)pos);
  }
  // offsets of the instances that start here, and of those past the last
  // interface cell
  if (valid)
    for (int i = ii; i >= 0 && if_off[i] == e; --i) g_off[i] = pos;
  if (e == nif - 1)
    for (int i = ninst; i >= 0 && if_off[i] == nif; --i) g_off[i] = pos + (ghost ? 1 : 0);
  if (e == 0) flow[0] = flow[1] = flow[2] = 0;   // of the whole-GPU layering
}

// --------------------------------------------------------------------------
// 4. stencils and dependencies
// --------------------------------------------------------------------------

__device__ __forceinline__ void atomic_max_nonneg(unsigned long long* a, double v) {
  if (v > 0.0) atomicMax(a, (unsigned long long)__double_as_longlong(v));
}

// Statistics of a wave's ghosts of one instance (k_deps): largest alpha and
// multiplier per axis, ghosts on the fluid side.
struct FinPart {
  double am[3];
  int32_t rm[3];
  int32_t fl;
  int32_t inst;
  int32_t pad;
};

// Stencils and the ghosts they read.  A ghost's corners are taken side by side
// (their tags, then the first slots probed in the table, then the rest), so
// the chain tag -> slot is waited for once: the 512^3 sphere's 74,000 ghosts
// take 26 us, one corner after the other 34.  The table holds positions among
// all ghosts here.
__global__ __launch_bounds__(256) void k_deps(const Inst* __restrict__ insts, int ninst,
                                              const int64_t* __restrict__ g_off,
                                              const int32_t* __restrict__ g_cell,
                                              const double* __restrict__ g_psi,
                                              const double* __restrict__ g_n, int64_t cap,
                                              const uint8_t* __restrict__ g_ext,
                                              const int8_t* __restrict__ tags,
                                              const unsigned long long* __restrict__ htab,
                                              const int64_t* __restrict__ hoff,
                                              const uint32_t* __restrict__ hmask,
                                              uint32_t* __restrict__ g_code,
                                              int32_t* __restrict__ deps,
                                              int32_t* __restrict__ lev,
                                              InstInfo* __restrict__ info,
                                              FinPart* __restrict__ part) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, ng = g_off[ninst];
  if ((int64_t)blockIdx.x * blockDim.x >= ng) return;   // uniform
  const bool valid = e < ng;
  const int lane = threadIdx.x & 63;
  const int ii = find_inst_wave(g_off, ninst, e - lane, min(e, ng - 1));
  double am[3] = {0.0, 0.0, 0.0};
  int rm[3] = {0, 0, 0}, fl = 0;
  if (valid) {
    const Inst& I = insts[ii];
    const GridD& g = I.g;
    const int c = g_cell[e];
    const double psi = g_psi[e];
    double n[3];
    int r[3] = {1, 1, 1};
    for (int a = 0; a < 3; ++a) n[a] = g_n[a * cap + e];
    int i, j, k;
    unlinear(g, c, i, j, k);
    if (I.scheme == kCGC_ES || g_ext[e]) {
      // Eq. stencil_anisotropic: r_i = max(1, ceil(2 |x_1 - x_s|_i / dx_i)),
      // dx_i the ghost cell's own width
      const int gi[3] = {i, j, k};
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (a >= g.dim) break;
        double d = psi * n[a];
        double q = 2.0 * fabs(d) / width(g, a, gi[a]);
        int ri = (int)ceil(q);
        r[a] = ri < 1 ? 1 : ri;
        if (r[a] > 15) {
          atomicOr(&info[ii].err, kErrUnsupported);
          r[a] = 15;
        }
      }
    }
    const uint32_t code = make_code(n, r, g.dim);
    uint32_t ghosts = 0;   // corners that are ghosts
    lev[e] = 0;   // k_levels_flow: no level yet
    const int8_t* T = tags + I.cell_off;
    const unsigned long long* const tab = htab + hoff[ii];
    const uint32_t mask = hmask[ii], skip = code_skip(code);
    const int np = (1 << g.dim) - 1;
    int q[8];
    int8_t t[8];
    unsigned long long en[8];
    bool out = false;
#pragma unroll
    for (int m = 1; m < 8; ++m) {
      const bool use = m <= np && !(m & skip), in = use && corner_in_grid(g, code, i, j, k, m);
      out = out || (use && !in);
      q[m] = in ? c + corner_offset(g, code, m) : -1;
      t[m] = 0;
      if (in) t[m] = T[q[m]];
    }
#pragma unroll
    for (int m = 1; m < 8; ++m) {
      out = out || t[m] == 1;
      en[m] = ~0ull;
      if (t[m] == 2 || t[m] == -2) en[m] = tab[table_slot(q[m], mask)];
    }
    if (out) atomicOr(&info[ii].err, kErrStencil);
#pragma unroll
    for (int m = 1; m < 8; ++m) {
      if (m > np) break;
      // (linear probing; an empty slot ends every probe)
      for (uint32_t h = table_slot(q[m], mask); en[m] != ~0ull && (int)(en[m] >> 32) != q[m];
           en[m] = tab[h])
        h = (h + 1) & mask;
      const int32_t d = en[m] == ~0ull ? -1 : (int32_t)(en[m] & 0xffffffffu);
      deps[(int64_t)(m - 1) * cap + e] = d;
      if (d >= 0) ghosts |= 1u << m;
    }
    g_code[e] = code | ghosts << 20;
    double Xs[3];
    stencil_span(g, code, c, Xs);
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (a < g.dim) {
        am[a] = fmax(0.0, psi * n[a] / Xs[a]);
        rm[a] = code_r(code, a);
      }
    fl = psi < 0.0 ? 1 : 0;
  }
  // statistics: the wave's first instance in its record, others (the wave
  // where they meet) by one lane's atomics
  bool first = true;
  for (unsigned long long todo = __ballot(valid); todo;) {   // uniform
    const int i0 = __shfl(ii, __ffsll(todo) - 1);
    const bool mine = valid && ii == i0;
    todo &= ~__ballot(mine);
    double a3[3];
    int r3[3], f = mine ? fl : 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      a3[a] = mine ? am[a] : 0.0;
      r3[a] = mine ? rm[a] : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        a3[a] = fmax(a3[a], __shfl_xor(a3[a], o));
        r3[a] = max(r3[a], __shfl_xor(r3[a], o));
      }
      f += __shfl_xor(f, o);
    }
    if (lane == 0) {
      if (first) {
        FinPart R;
        for (int a = 0; a < 3; ++a) {
          R.am[a] = a3[a];
          R.rm[a] = r3[a];
        }
        R.fl = f;
        R.inst = i0;
        R.pad = 0;
        part[e >> 6] = R;
      } else {
        for (int a = 0; a < 3; ++a) {
          atomic_max_nonneg(&info[i0].max_alpha_bits[a], a3[a]);
          if (r3[a]) atomicMax(&info[i0].rmax[a], r3[a]);
        }
        if (f) atomicAdd(&info[i0].nfluid, f);
      }
    }
    first = false;
  }
}

// For the layerings that push along reverse edges: the number of ghosts
// each ghost reads, and of those that read it (rcnt starts at zero).
__global__ __launch_bounds__(256) void k_rcount(const Inst* __restrict__ insts,
                                                const int64_t* __restrict__ g_off, int ninst,
                                                int64_t cap, const int32_t* __restrict__ deps,
                                                int32_t* __restrict__ rcnt,
                                                uint8_t* __restrict__ dcnt) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= g_off[ninst]) return;
  const int np = (1 << insts[find_inst(g_off, ninst, e)].g.dim) - 1;
  int nd = 0;
  for (int m = 0; m < np; ++m) {
    const int32_t d = deps[(int64_t)m * cap + e];
    if (d < 0) continue;
    atomicAdd(&rcnt[d], 1);   // reverse edge d -> e
    ++nd;
  }
  dcnt[e] = (uint8_t)nd;
}

// Reverse edges of the dependency graph as CSR over all ghosts (linear
// order): out[e] = first reader of ghost e, out[ng] = number of edges (posted
// as in k_scan_tiles).  The counts past the ghost count are zero, so scanning
// the interface capacity gives the same offsets up to the ghost count.
__global__ __launch_bounds__(256) void k_iscan(const int32_t* __restrict__ in, int64_t n,
                                               unsigned long long* __restrict__ posted,
                                               int32_t* __restrict__ out) {
  __shared__ int64_t sh[5];
  __shared__ int s_b;
  if (threadIdx.x == 0) s_b = (int)atomicAdd(&posted[gridDim.x], 1ull);
  __syncthreads();
  const int t = s_b;
  const int64_t b = ((int64_t)t * 256 + threadIdx.x) * kScanT;
  int v[kScanT];
  scan_load(in, n, b, v);
  int64_t sum = 0;
#pragma unroll
  for (int q = 0; q < kScanT; ++q) sum += v[q];
  int64_t tot;
  const int64_t rank = block_excl_scan<256>(sum, &tot, sh);
  int64_t run = posted_before<256>(posted, t, tot) + rank;
#pragma unroll
  for (int q = 0; q < kScanT; ++q) {
    if (b + q < n) out[b + q] = (int32_t)run;
    run += v[q];
  }
  if (b < n && b + kScanT >= n) out[n] = (int32_t)run;   // the thread holding the last value
}

__global__ __launch_bounds__(256) void k_rfill(const Inst* __restrict__ insts,
                                               const int64_t* __restrict__ g_off, int ninst,
                                               int64_t cap, const int32_t* __restrict__ deps,
                                               const int32_t* __restrict__ off,
                                               int32_t* __restrict__ fillc,
                                               int32_t* __restrict__ radj) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= g_off[ninst]) return;
  const int ii = find_inst(g_off, ninst, e);
  const int np = (1 << insts[ii].g.dim) - 1;
  for (int m = 0; m < np; ++m) {
    const int32_t d = deps[(int64_t)m * cap + e];
    if (d >= 0) radj[off[d] + atomicAdd(&fillc[d], 1)] = (int32_t)e;
  }
}

// --------------------------------------------------------------------------
// 6. canonical arrays
// --------------------------------------------------------------------------

// hist (null: perm holds them): the canonical positions are found here, tile
// by tile of the whole-GPU layering (k_levels_flow; the workgroup's 256
// ghosts are its tile): hist[tile][level] is the position of the tile's
// first ghost of that level, its rank among the tile's comes from ballots.
__device__ __forceinline__ int tile_position(const int32_t* __restrict__ lev,
                                             const int32_t* __restrict__ hist, int64_t e, int64_t n,
                                             int32_t* __restrict__ perm) {
  __shared__ int s_wc[4][kWideLevels];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int t = threadIdx.x; t < 4 * kWideLevels; t += 256) s_wc[t / kWideLevels][t % kWideLevels] = 0;
  __syncthreads();
  const bool valid = e < n;
  const int l = valid ? lev[e] - 1 : 0;
  unsigned long long mk = __ballot(valid);
  static_assert(kWideLevels <= 128, "a level index fits 7 ballots");
#pragma unroll
  for (int bit = 0; bit < 7; ++bit) {
    const bool on = (l >> bit) & 1;
    const unsigned long long bb = __ballot(valid && on);
    mk &= on ? bb : ~bb;
  }
  const int rank = __popcll(mk & ((1ull << lane) - 1ull));
  if (valid && rank == 0) s_wc[wv][l] = __popcll(mk);
  __syncthreads();
  if (!valid) return -1;
  int pos = hist[(e >> 8) * kWideLevels + l] + rank;
  for (int w = 0; w < wv; ++w) pos += s_wc[w][l];
  perm[e] = pos;
  return pos;
}

// What the host reads of a build, in pinned memory: of each instance its
// info, first ghost, level offsets and units' levels, as many as there are.
struct BuildResult {
  InstInfo* info;
  int64_t* g_off;
  int32_t* lev_off;    // [ninst][kMaxLevels + 1]
  int32_t* unit_lev;   // [ninst][kMaxUnits]
};

// Workgroup ii < ninst: the instance's unit members from linear-order to
// canonical positions, and its results to the host, the waves' statistics
// (k_deps) folded into its info there (max, max, sum: the order does not
// matter).  Run again after a second layering, it leaves an instance that was
// finished before as it is: the members are mapped once (info.layered), and
// the device's info stays without the waves' sums.
__device__ __forceinline__ void finish_instance(int ii, int ninst, const int64_t* __restrict__ g_off,
                                                const int32_t* __restrict__ perm,
                                                InstInfo* __restrict__ info,
                                                int32_t* __restrict__ unit_mem,
                                                const int32_t* __restrict__ unit_cnt,
                                                const int32_t* __restrict__ unit_lev,
                                                const int32_t* __restrict__ lev_off,
                                                const FinPart* __restrict__ part,
                                                const BuildResult& out) {
  const int tid = threadIdx.x;
  const int nu = min(max(info[ii].nunits, 0), kMaxUnits), nl = min(max(info[ii].nlev, 0), kMaxLevels);
  int32_t* um = unit_mem + (int64_t)ii * kMaxUnits * kMaxUnit;
  const int32_t* uc = unit_cnt + (int64_t)ii * kMaxUnits;
  const int nmap = info[ii].layered == kLayeredMapped ? 0 : nu;
  for (int t = tid; t < nmap * kMaxUnit; t += blockDim.x)
    if (t % kMaxUnit < uc[t / kMaxUnit]) um[t] = perm[um[t]];
  for (int t = tid; t <= nl; t += blockDim.x)
    out.lev_off[(int64_t)ii * (kMaxLevels + 1) + t] = lev_off[(int64_t)ii * (kMaxLevels + 1) + t];
  for (int t = tid; t < nu; t += blockDim.x)
    out.unit_lev[(int64_t)ii * kMaxUnits + t] = unit_lev[(int64_t)ii * kMaxUnits + t];
  double am[3] = {0.0, 0.0, 0.0};
  int rm[3] = {0, 0, 0}, fl = 0;
  const int64_t b = g_off[ii], e = g_off[ii + 1];
  if (e > b)
    for (int64_t w = (b >> 6) + tid; w <= (e - 1) >> 6; w += blockDim.x) {
      const FinPart r = part[w];
      if (r.inst != ii) continue;
      for (int a = 0; a < 3; ++a) {
        am[a] = fmax(am[a], r.am[a]);
        rm[a] = max(rm[a], r.rm[a]);
      }
      fl += r.fl;
    }
  __shared__ double s_am[3][4];
  __shared__ int s_rm[3][4], s_fl[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      am[a] = fmax(am[a], __shfl_xor(am[a], o));
      rm[a] = max(rm[a], __shfl_xor(rm[a], o));
    }
    fl += __shfl_xor(fl, o);
  }
  if ((tid & 63) == 0) {
    for (int a = 0; a < 3; ++a) {
      s_am[a][tid >> 6] = am[a];
      s_rm[a][tid >> 6] = rm[a];
    }
    s_fl[tid >> 6] = fl;
  }
  __syncthreads();
  if (tid != 0) return;
  InstInfo I = info[ii];
  for (int w = 0; w < 4; ++w) {
    for (int a = 0; a < 3; ++a) {
      const unsigned long long bits = (unsigned long long)__double_as_longlong(s_am[a][w]);
      if (bits > I.max_alpha_bits[a]) I.max_alpha_bits[a] = bits;   // non-negative: bit order
      I.rmax[a] = max(I.rmax[a], s_rm[a][w]);
    }
    I.nfluid += s_fl[w];
  }
  out.info[ii] = I;
  if (I.layered) info[ii].layered = kLayeredMapped;
  out.g_off[ii] = b;
  if (ii == ninst - 1) out.g_off[ninst] = e;
}

__global__ __launch_bounds__(256) void k_finalize(
    const Inst* __restrict__ insts, int ninst, const int64_t* __restrict__ g_off, int64_t cap,
    const int32_t* __restrict__ g_cell, const double* __restrict__ g_psi,
    const double* __restrict__ g_n, const uint32_t* __restrict__ g_code,
    const uint32_t* __restrict__ g_slot,
    const int32_t* __restrict__ deps, int32_t* __restrict__ cgi,
    const int32_t* __restrict__ lev, const int32_t* __restrict__ blk_idx,
    int32_t* __restrict__ perm, const int32_t* __restrict__ hist, int32_t* __restrict__ cell,
    double* __restrict__ delta,
    double* __restrict__ nrm, double* __restrict__ psi, uint32_t* __restrict__ code,
    int32_t* __restrict__ level, int32_t* __restrict__ blk, const int64_t* __restrict__ hoff,
    unsigned long long* __restrict__ htab, InstInfo* __restrict__ info,
    int32_t* __restrict__ unit_mem, const int32_t* __restrict__ unit_cnt,
    const int32_t* __restrict__ unit_lev, const int32_t* __restrict__ lev_off,
    const FinPart* __restrict__ part, BuildResult out) {
  if ((int)blockIdx.x < ninst)
    finish_instance(blockIdx.x, ninst, g_off, perm, info, unit_mem, unit_cnt, unit_lev, lev_off,
                    part, out);
  const int64_t e0 = (int64_t)blockIdx.x * blockDim.x, e = e0 + threadIdx.x;
  const int64_t ng_all = g_off[ninst];
  if (e0 >= ng_all) return;   // uniform
  const int ii = find_inst_wave(g_off, ninst, e0 + (threadIdx.x & ~63), min(e, ng_all - 1));
  int pl = -1;
  if (hist) {   // (a batch of one; uniform)
    if (info[0].layered) pl = tile_position(lev, hist, e, ng_all, perm);
  } else if (e < ng_all) {
    pl = perm[e];
  }
  if (e >= ng_all || pl < 0 || pl >= g_off[ii + 1] - g_off[ii]) return;   // (the build failed earlier)
  const int64_t p = g_off[ii] + pl;
  const double ps = g_psi[e];
  const uint32_t cd = g_code[e];
  const int c = g_cell[e];
  cell[p] = c;
  psi[p] = ps;
  code[p] = cd;
  level[p] = lev[e];
  blk[p] = blk_idx[e];
  for (int a = 0; a < 3; ++a) {
    const double na = g_n[a * cap + e];
    nrm[a * cap + p] = na;
    delta[a * cap + p] = ps * na;
  }
  // the cell table from positions among all ghosts to canonical ones
  htab[hoff[ii] + g_slot[e]] = ((unsigned long long)(uint32_t)c << 32) | (uint32_t)pl;
  if (cgi && insts[ii].g.dim == 2) {
    // the corners' ghosts, by position (the graph's edges in this order)
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      const int32_t d = deps[(int64_t)(k - 1) * cap + e];
      cgi[(int64_t)(k - 1) * cap + p] = (k & code_skip(cd)) ? -2 : d < 0 ? -1 : perm[d];
    }
  }
}

// --------------------------------------------------------------------------
// 7. cell -> ghost hash tables (open addressing, at most half full)
// --------------------------------------------------------------------------

__global__ void k_hash_clear(unsigned long long* __restrict__ t, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) t[i] = ~0ull;
}

// --------------------------------------------------------------------------
// host orchestration
// --------------------------------------------------------------------------

static double factorial(int n) {
  double f = 1.0;
  for (int i = 2; i <= n; ++i) f *= (double)i;
  return f;
}

constexpr int kMaxL2Radius = 64;   // second-layer candidate box half-width, cells

static gcr_status make_shape(const gcr_shape& gs, int dim, ShapeD* out);
static void set_l2tight(Inst* I);

static gcr_status make_inst(const gcr_grid& gg, const gcr_shape& gs, int scheme, Inst* I) {
  std::memset(I, 0, sizeof(Inst));
  if (gg.dim != 2 && gg.dim != 3) return GCR_E_ARG;
  const int base = scheme & ~kLayer2;
  if (base < 0 || base > 2) return GCR_E_ARG;
  int64_t ncell = 1;
  for (int a = 0; a < gg.dim; ++a) {
    if (gg.n[a] < 1) return GCR_E_ARG;
    if (gg.faces[a]) {
      for (int64_t q = 0; q < gg.n[a]; ++q)
        if (!(gg.faces[a][q + 1] > gg.faces[a][q]) || !std::isfinite(gg.faces[a][q]) ||
            !std::isfinite(gg.faces[a][q + 1]))
          return GCR_E_ARG;
    } else if (!(gg.h[a] > 0.0) || !std::isfinite(gg.lo[a])) {
      return GCR_E_ARG;
    }
    ncell *= gg.n[a];
    if (ncell >= (int64_t(1) << 31)) return GCR_E_UNSUPPORTED;
  }
  I->g.dim = gg.dim;
  for (int a = 0; a < 3; ++a) {
    I->g.n[a] = a < gg.dim ? (int)gg.n[a] : 1;
    I->g.lo[a] = a < gg.dim ? gg.lo[a] : 0.0;
    I->g.h[a] = a < gg.dim ? gg.h[a] : 1.0;
    // a stretched axis: the caller's faces for now; build_batch puts a
    // device copy here before the instance table is uploaded
    I->g.face[a] = a < gg.dim ? gg.faces[a] : nullptr;
    if (I->g.face[a]) {
      I->g.lo[a] = gg.faces[a][0];
      I->g.h[a] = (gg.faces[a][gg.n[a]] - gg.faces[a][0]) / (double)gg.n[a];
    }
  }
  I->g.ncell = ncell;
  set_division(&I->g);
  I->scheme = base;
  I->layer2 = (scheme & kLayer2) ? 1 : 0;
  if (I->layer2) {
    // second-layer candidate box: every solid cell with psi <= 1.5 delta n
    // has a fluid centre within (1.5 + sqrt(d)/2) w_max of its own (delta n
    // <= w_max, the largest cell width), which lies at most
    // floor(D / w_min_a) + 1 cells away along axis a (w_min_a the smallest
    // width along a)
    double wmax = 0.0, wmin[3] = {0.0, 0.0, 0.0};
    for (int a = 0; a < gg.dim; ++a) {
      wmin[a] = gg.faces[a] ? HUGE_VAL : gg.h[a];
      if (!gg.faces[a]) wmax = std::max(wmax, gg.h[a]);
      else
        for (int64_t q = 0; q < gg.n[a]; ++q) {
          const double w = gg.faces[a][q + 1] - gg.faces[a][q];
          wmax = std::max(wmax, w);
          wmin[a] = std::min(wmin[a], w);
        }
    }
    for (int a = 0; a < 3; ++a) {
      I->l2r[a] = 0;
      if (a >= gg.dim) continue;
      const double r = std::floor((1.5 + 0.5 * std::sqrt((double)gg.dim)) * wmax / wmin[a]) + 1.0;
      // box sizes stay far inside int range; wider boxes mean a grid
      // stretched beyond any use near the body
      if (!(r <= (double)kMaxL2Radius)) return GCR_E_UNSUPPORTED;
      I->l2r[a] = (int)r;
    }
    I->l2walk = (1.5 + 0.5 * std::sqrt((double)gg.dim)) * wmax;
  }
  const gcr_status st = make_shape(gs, gg.dim, &I->s);
  set_l2tight(I);
  return st;
}

// Whether the second layer's candidates lie within the walk of their foot
// points (k_l2_mark): a sphere inside the grid with the walk's length to
// spare on every side, so that no walk meets the grid's edge.
static void set_l2tight(Inst* I) {
  I->l2tight = 0;
  if (!I->layer2 || I->s.kind != kSphere) return;
  for (int a = 0; a < I->g.dim; ++a) {
    const double need = I->s.r0 + 2.0 * I->l2walk;
    const double lo = I->g.lo[a], hi = lo + I->g.h[a] * (double)I->g.n[a];
    if (!(I->s.c[a] - need > lo) || !(I->s.c[a] + need < hi)) return;
  }
  I->l2tight = 1;
}

// The device description of body gs in dim dimensions (Sec. 7: the bodies
// of the test cases), with its culling bounds.
static gcr_status make_shape(const gcr_shape& gs, int dim, ShapeD* out) {
  ShapeD s;
  std::memset(&s, 0, sizeof(s));
  s.kind = gs.kind;
  for (int a = 0; a < 3; ++a) s.c[a] = a < dim ? gs.center[a] : 0.0;
  s.r0 = gs.r0;
  if (gs.kind == kSphere) {
    if (!(gs.r0 > 0.0)) return GCR_E_ARG;
    for (int a = 0; a < 3; ++a) s.cull_c[a] = s.c[a];
    s.rmin = s.rmax = gs.r0;
  } else if (gs.kind == kStar2D) {
    if (dim != 2 || !(gs.r0 > 0.0) || gs.ncoef < 0 || 2 * gs.ncoef > kMaxCoef) return GCR_E_ARG;
    if (gs.ncoef > 0 && !gs.coef) return GCR_E_ARG;
    s.ncoef = gs.ncoef;
    double sa = 0.0;
    for (int q = 0; q < 2 * gs.ncoef; ++q) {
      s.coef[q] = gs.coef[q];
      sa += std::fabs(gs.coef[q]);
    }
    for (int a = 0; a < 3; ++a) s.cull_c[a] = s.c[a];
    s.rmin = std::max(0.0, gs.r0 * (1.0 - sa));
    s.rmax = gs.r0 * (1.0 + sa);
    // |d/dt (A cos kt + B sin kt)| <= k sqrt(A^2 + B^2)
    double lip = 0.0;
    for (int k = 0; k < gs.ncoef; ++k)
      lip += (double)k * std::hypot(gs.coef[2 * k], gs.coef[2 * k + 1]);
    s.lip = gs.r0 * lip;
  } else if (gs.kind == kShStar) {
    int L = (int)std::lround(std::sqrt((double)gs.ncoef)) - 1;
    if (dim != 3 || !(gs.r0 > 0.0) || L < 0 || (L + 1) * (L + 1) != gs.ncoef || L > 8 ||
        !gs.coef)
      return GCR_E_ARG;
    s.ncoef = gs.ncoef;
    s.L = L;
    double sa = 0.0;
    for (int l = 0; l <= L; ++l)
      for (int m = -l; m <= l; ++m) {
        int am = m < 0 ? -m : m;
        double N = am == 0 ? 1.0 : std::sqrt(2.0 * factorial(l - am) / factorial(l + am));
        s.coef[l * l + l + m] = gs.coef[l * l + l + m] * N;
        sa += std::fabs(gs.coef[l * l + l + m]);   // |Y_lm| <= 1 (Schmidt)
      }
    for (int a = 0; a < 3; ++a) s.cull_c[a] = s.c[a];
    s.rmin = std::max(0.0, gs.r0 * (1.0 - sa));
    s.rmax = gs.r0 * (1.0 + sa);
    // on a great circle Y_lm is a trigonometric polynomial of degree <= l
    // with |Y_lm| <= 1, so (Bernstein) its derivative is at most l
    double lip = 0.0;
    for (int l = 1; l <= L; ++l)
      for (int m = -l; m <= l; ++m) lip += (double)l * std::fabs(gs.coef[l * l + l + m]);
    s.lip = gs.r0 * lip;
  } else if (gs.kind == kAirfoil) {
    if (dim != 2 || !(gs.chord > 0.0) || !(gs.thickness > 0.0) || gs.thickness > 0.5)
      return GCR_E_ARG;
    s.chord = gs.chord;
    s.thick = gs.thickness;
    s.ca = std::cos(gs.incidence);
    s.sa = std::sin(gs.incidence);
    // mid-chord in world coordinates; the section lies within 0.51 chords of it
    s.cull_c[0] = s.c[0] + gs.chord * (s.ca * 0.5);
    s.cull_c[1] = s.c[1] + gs.chord * (-s.sa * 0.5);
    s.rmin = 0.0;
    s.rmax = 0.51 * gs.chord;
  } else {
    return GCR_E_ARG;
  }
  *out = s;
  return GCR_OK;
}

BatchData::~BatchData() {
  for (void* p : owned) pool_free(p);
}

template <class T>
static T* own(BatchData& B, size_t n) {
  // bump allocation from pooled chunks of at least 4 MiB (a build makes a
  // few pool calls instead of one per array); 256-byte aligned
  constexpr size_t kArena = size_t(4) << 20;
  const size_t bytes = ((sizeof(T) * (n ? n : 1)) + 255) & ~size_t(255);
  if (bytes > B.arena_left) {
    const size_t chunk = std::max(bytes, kArena);
    char* c = static_cast<char*>(pool_alloc(chunk));
    if (!c) return nullptr;
    B.owned.push_back(c);
    if (bytes >= kArena) return reinterpret_cast<T*>(c);   // a chunk of its own
    B.arena_cur = c;
    B.arena_left = chunk;
  }
  T* p = reinterpret_cast<T*>(B.arena_cur);
  B.arena_cur += bytes;
  B.arena_left -= bytes;
  return p;
}

gcr_status status_from_err(uint32_t err) {
  if (err & kErrGeometry) return GCR_E_GEOMETRY;
  if (err & kErrCycle) return GCR_E_CYCLE;
  if (err & kErrStencil) return GCR_E_STENCIL;
  if (err & kErrDegenerate) return GCR_E_DEGENERATE;
  if (err & kErrUnsupported) return GCR_E_UNSUPPORTED;
  return GCR_OK;
}

static inline unsigned blocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// stage timing (process-wide switch, per-thread results)
static std::atomic<int> g_profiling{0};
static thread_local float g_stage_ms[kStages] = {};

// Brings the calling thread's table of thread-local storage up to date.
// Libraries loaded after a thread started (this one and those HIP loads) leave
// every access of the thread to such storage elsewhere, several per PyTorch or
// HIP call, on the dynamic linker's slow path until it touches the storage of
// the one loaded last.  Measured after the first plan of a process, without
// and with this: torch.empty 1.33 and 1.08 us, a small torch kernel launch 5.1
// and 4.3 us.
void touch_thread_storage() {
  volatile float* p = g_stage_ms;
  p[0] = p[0];
}

struct StageEvents {
  hipEvent_t ev[12] = {};
  bool on = false;
  explicit StageEvents(bool enable) : on(enable) {
    if (on)
      for (auto& e : ev)
        if (hipEventCreate(&e) != hipSuccess) on = false;
  }
  void mark(int i, hipStream_t st) {
    if (on) (void)hipEventRecord(ev[i], st);
  }
  hipEvent_t event(int i) const { return on ? ev[i] : nullptr; }
  void collect(double call_ms) {
    if (!on) return;
    // stages 0..7 as documented; 8..10 split stage 0 into the span pass,
    // the store pass (k_classify) and the interface marks (k_band_iface);
    // 11 is the stream's wait for the host between the two halves (the
    // first synchronisation and the sizing); 12 the call's host time
    // (stage 4, the ghosts' compaction, is part of stage 3 now)
    constexpr int kEv = kStages - 1;
    const int a[kEv] = {0, 1, 3, 4, 5, 5, 7, 8, 0, 10, 11, 2};
    const int b[kEv] = {1, 2, 4, 5, 5, 7, 8, 9, 10, 11, 1, 3};
    g_stage_ms[kEv] = (float)call_ms;
    for (int s = 0; s < kEv; ++s) {
      float ms = 0.f;
      if (a[s] != b[s] && hipEventElapsedTime(&ms, ev[a[s]], ev[b[s]]) != hipSuccess) ms = -1.f;
      g_stage_ms[s] = ms;
    }
  }
  ~StageEvents() {
    if (on)
      for (auto& e : ev) (void)hipEventDestroy(e);
  }
};

void set_profiling(int mask) { g_profiling.store(mask & 3); }
int profiling_mask() { return g_profiling.load(); }

static std::atomic<int64_t> g_wide_min{0};   // 0: the default
void set_wide_layering(int64_t v) { g_wide_min.store(v > 0 ? v : 0); }
int64_t wide_layering_min() {
  const int64_t v = g_wide_min.load();
  return v ? v : kWideMinInterface;
}
static std::atomic<int> g_wave_res{kWaveResidual};
void set_wave_residual(int v) { g_wave_res.store(v < 0 ? 0 : (v > kWaveResidual ? kWaveResidual : v)); }
int wave_residual() { return g_wave_res.load(); }
bool wide_layering_forced() { return g_wide_min.load() != 0; }
void last_build_times(float* ms) {
  for (int s = 0; s < kStages; ++s) ms[s] = g_stage_ms[s];
}

template <class T>
static T* own_solo(BatchData& B, size_t n) {
  // a pool allocation of its own (so that a re-plan can take it over)
  T* p = static_cast<T*>(pool_alloc(sizeof(T) * (n ? n : 1)));
  if (p) B.owned.push_back(p);
  return p;
}

static gcr_status build_core(const std::shared_ptr<BatchData>& B, hipStream_t st,
                             BatchData* prev, std::shared_ptr<BatchData>* out);

gcr_status build_batch(int ninst, const gcr_grid* grids, const gcr_shape* shapes,
                       const int32_t* schemes, hipStream_t st, std::shared_ptr<BatchData>* out) {
  if (ninst < 1 || !grids || !shapes || !schemes || !out) return GCR_E_ARG;
  auto B = std::make_shared<BatchData>();
  B->ninst = ninst;
  B->inst.resize(ninst);
  for (int i = 0; i < ninst; ++i) {
    gcr_status s = make_inst(grids[i], shapes[i], schemes[i], &B->inst[i]);
    if (s != GCR_OK) return s;
  }
  // stretched axes: device copies of the faces (pageable sources, consumed
  // when each copy returns)
  for (int i = 0; i < ninst; ++i)
    for (int a = 0; a < 3; ++a) {
      const double* hf = B->inst[i].g.face[a];
      if (!hf) continue;
      const int64_t nf = (int64_t)B->inst[i].g.n[a] + 1;
      double* df = own<double>(*B, nf);
      if (!df) return GCR_E_NOMEM;
      GCR_HIP(hipMemcpyAsync(df, hf, sizeof(double) * nf, hipMemcpyHostToDevice, st));
      B->inst[i].g.face[a] = df;
    }
  return build_core(B, st, nullptr, out);
}

gcr_status build_update(BatchData& prev, const gcr_shape& shape, bool incremental,
                        hipStream_t st, std::shared_ptr<BatchData>* out) {
  if (prev.ninst != 1 || !out) return GCR_E_UNSUPPORTED;
  ShapeD sd;
  const gcr_status s = make_shape(shape, prev.inst[0].g.dim, &sd);
  if (s != GCR_OK) return s;
  return build_update(prev, sd, incremental, st, out);
}

gcr_status build_update(BatchData& prev, const ShapeD& shape, bool incremental, hipStream_t st,
                        std::shared_ptr<BatchData>* out) {
  if (prev.ninst != 1 || !out) return GCR_E_UNSUPPORTED;
  auto B = std::make_shared<BatchData>();
  B->ninst = 1;
  B->inst.resize(1);
  Inst I = prev.inst[0];
  I.s = shape;
  set_l2tight(&I);
  // the stretched faces: device copies of the previous plan's
  for (int a = 0; a < 3; ++a) {
    if (!I.g.face[a]) continue;
    const int64_t nf = (int64_t)I.g.n[a] + 1;
    double* df = own<double>(*B, nf);
    if (!df) return GCR_E_NOMEM;
    GCR_HIP(hipMemcpyAsync(df, I.g.face[a], sizeof(double) * nf, hipMemcpyDeviceToDevice, st));
    I.g.face[a] = df;
  }
  B->inst[0] = I;
  return build_core(B, st, incremental ? &prev : nullptr, out);
}

// The levels and canonical arrays, from the ghosts in linear order and their
// dependencies, layered as `how` says: by one workgroup per instance pulling,
// by the whole GPU, or by the layerings that push along reverse edges, which
// take every graph the others leave.  A second call for instances that the
// first left does no harm to the others: the push layerings pass them by
// (info.layered), k_finalize stores the same again, and of those left it has
// stored nothing (their cell tables hold linear-order indices as before).
enum Layering { kLayerPull, kLayerFlow, kLayerPush };
static gcr_status build_levels(BatchData& D, hipStream_t st, int ninst, int64_t nif,
                               int64_t max_if, Layering how, const FinPart* part,
                               const BuildResult& out, StageEvents& T) {
  const int64_t cap = D.cap;
  int32_t* hist = nullptr;
  // ghost count unknown on the host: launch over the interface capacity
  if (how == kLayerPush) {
    k_zero_words<<<blocks(2 * cap, 256), 256, 0, st>>>(D.d_rcnt, 2 * cap);
    k_rcount<<<blocks(nif, 256), 256, 0, st>>>(D.d_inst, D.d_g_off, ninst, cap, D.d_deps,
                                                D.d_rcnt, D.d_dcnt);
    // reverse-edge offsets, over the interface capacity
    const int64_t ntiles = (cap + kScanTile - 1) / kScanTile;
    unsigned long long* const posted = own<unsigned long long>(D, ntiles + 1);
    if (!posted) return GCR_E_NOMEM;
    k_zero_words<<<blocks(2 * (ntiles + 1), 256), 256, 0, st>>>(reinterpret_cast<int32_t*>(posted),
                                                                2 * (ntiles + 1));
    k_iscan<<<(unsigned)ntiles, 256, 0, st>>>(D.d_rcnt, cap, posted, D.d_roff);
    k_rfill<<<blocks(nif, 256), 256, 0, st>>>(D.d_inst, D.d_g_off, ninst, cap, D.d_deps,
                                               D.d_roff, D.d_rcnt + cap, D.d_radj);
  }
  T.mark(7, st);
  {
    LevelsArgs L;
    L.insts = D.d_inst;
    L.g_off = D.d_g_off;
    L.deps = D.d_deps;
    L.cap = cap;
    L.lev = D.d_lev;
    L.blk_idx = D.d_blk_idx;
    L.perm = D.d_perm;
    L.lev_off = D.d_lev_off;
    L.unit_mem = D.d_unit_mem;
    L.unit_cnt = D.d_unit_cnt;
    L.unit_lev = D.d_unit_lev;
    L.reach = D.d_reach;
    L.listA = D.d_listA;
    L.dcnt = D.d_dcnt;
    L.roff = D.d_roff;
    L.radj = D.d_radj;
    L.cnt = D.d_cnt;
    L.bits = D.d_bits;
    L.info = D.d_info;
    L.flow = L.hist = nullptr;
    L.cur_cap = 0;
    L.wave_res = wave_residual();
    if (how == kLayerFlow) {
      L.flow = D.d_rcnt;   // (cleared by k_geometry)
      hist = L.hist = own<int32_t>(D, (size_t)kWideLevels * (cap / 256 + 1));
      if (!L.hist) return GCR_E_NOMEM;
    }
    bool all_2d = true;
    for (const Inst& I : D.inst) all_2d = all_2d && I.g.dim == 2;
    const gcr_status ls = how == kLayerFlow   ? launch_levels_flow(L, max_if, st)
                          : how == kLayerPull ? launch_levels_pull(L, ninst, max_if, all_2d, st)
                                              : launch_levels(L, ninst, max_if, st);
    if (ls != GCR_OK) return ls;
  }
  T.mark(8, st);
  const unsigned nfb = std::max(blocks(nif, 256), (unsigned)ninst);
  k_finalize<<<nfb, 256, 0, st>>>(
      D.d_inst, ninst, D.d_g_off, cap, D.d_g_cell, D.d_g_psi, D.d_g_n, D.d_g_code, D.d_g_slot,
      D.d_deps, hist ? nullptr : D.d_cgi, D.d_lev, D.d_blk_idx, D.d_perm, hist, D.d_cell,
      D.d_delta, D.d_nrm, D.d_psi, D.d_code, D.d_level, D.d_blk, D.d_hoff, D.d_htab, D.d_info,
      D.d_unit_mem, D.d_unit_cnt, D.d_unit_lev, D.d_lev_off, part, out);
  T.mark(9, st);
  return GCR_OK;
}

// The build proper: B holds its instances (device faces in place); with
// prev, a re-plan of prev's single instance that takes over its tags.
static gcr_status build_core(const std::shared_ptr<BatchData>& B, hipStream_t st,
                             BatchData* prev, std::shared_ptr<BatchData>* out) {
  const auto t_call = std::chrono::steady_clock::now();
  touch_thread_storage();
  const int ninst = B->ninst;
  std::vector<int64_t> chunk_start(ninst + 1);
  int64_t cells = 0, chunks = 0;
  for (int i = 0; i < ninst; ++i) {
    Inst& I = B->inst[i];
    I.cell_off = cells;
    cells += (I.g.ncell + 255) / 256 * 256;
    I.chunk_off = chunks;
    I.nchunk = (I.g.ncell + kChunk - 1) / kChunk;
    chunk_start[i] = chunks;
    chunks += I.nchunk;
  }
  chunk_start[ninst] = chunks;
  B->ncells_total = cells;
  B->nchunks = chunks;
  BatchData& D = *B;
  // the small per-instance tables that cross between host and device live in
  // one device block with the layout of the pinned staging block, so each
  // transfer is one contiguous copy:
  //   R1 up:   instances | chunk starts | info (zeroed)
  //   stored by k_finalize at the end:    info | g_off | lev_off | unit_lev
  //   stored by the scans halfway: if_off | chunk-list and band counts | interface offsets
  //   device only: hash offsets | hash masks
  // each region 256-byte aligned
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t o_inst = 0, o_cs = o_inst + al(sizeof(Inst) * ninst);
  const size_t o_info = o_cs + al(8 * (ninst + 1));
  const size_t o_go = o_info + al(sizeof(InstInfo) * ninst);
  const size_t o_lo = o_go + al(8 * (ninst + 1));
  const size_t o_ul = o_lo + al(4 * (size_t)ninst * (kMaxLevels + 1));
  const size_t o_if = o_ul + al(4 * (size_t)ninst * kMaxUnits);
  const size_t o_nl = o_if + al(8 * (ninst + 1));   // chunk-list count, band stripes
  const size_t o_io = o_nl + al(64 + 64 * kBandStripes);
  const size_t o_ho = o_io + al(8 * (ninst + 1));
  const size_t o_hm = o_ho + al(8 * (ninst + 1));
  const size_t stage_bytes = o_hm + al(4 * ninst);
  char* tb = own<char>(D, stage_bytes);
  if (!tb) return GCR_E_NOMEM;
  D.d_inst = reinterpret_cast<Inst*>(tb + o_inst);
  D.d_chunk_start = reinterpret_cast<int64_t*>(tb + o_cs);
  D.d_info = reinterpret_cast<InstInfo*>(tb + o_info);
  D.d_g_off = reinterpret_cast<int64_t*>(tb + o_go);
  D.d_lev_off = reinterpret_cast<int32_t*>(tb + o_lo);
  D.d_unit_lev = reinterpret_cast<int32_t*>(tb + o_ul);
  D.d_if_off = reinterpret_cast<int64_t*>(tb + o_if);
  D.d_nchunk_list = reinterpret_cast<int32_t*>(tb + o_nl);
  D.d_nband = reinterpret_cast<int32_t*>(tb + o_nl + 64);
  D.d_iface_off = reinterpret_cast<int64_t*>(tb + o_io);
  D.d_hoff = reinterpret_cast<int64_t*>(tb + o_ho);
  D.d_hmask = reinterpret_cast<uint32_t*>(tb + o_hm);
  if (prev) {
    // the previous plan's tags, which the classification below updates
    if (prev->ninst != 1 || prev->nchunks != chunks || !prev->d_tags) return GCR_E_UNSUPPORTED;
    auto it = std::find(prev->owned.begin(), prev->owned.end(), (void*)prev->d_tags);
    if (it == prev->owned.end()) return GCR_E_UNSUPPORTED;
    prev->owned.erase(it);
    D.owned.push_back(prev->d_tags);
    D.d_tags = prev->d_tags;
    prev->d_tags = nullptr;
  } else {
    // a single instance's tags on their own, for a later re-plan to take over
    D.d_tags = ninst == 1 ? own_solo<int8_t>(D, cells) : own<int8_t>(D, cells);
  }
  D.d_chunk_cnt = own<int32_t>(D, chunks);
  D.d_dirty = own<int32_t>(D, chunks);
  D.d_dirty_list = own<int32_t>(D, chunks);
  D.d_ndirty = own<int32_t>(D, 1);
  if (!D.d_dirty || !D.d_dirty_list || !D.d_ndirty) return GCR_E_NOMEM;
  D.d_span = own<int8_t>(D, chunks * (kChunk / (64 * kSeg)));
  D.d_chunk_list = own<int32_t>(D, chunks);
  D.d_band = own<int32_t>(D, chunks * 8);   // band mask of each chunk (4 x 64 bits)
  D.d_chunk_inst = own<int32_t>(D, chunks);
  D.d_chunk_excl = own<int64_t>(D, chunks + 1);
  // what the scans' workgroups post: of the store pass's list, of the chunk
  // counts, and of those with the second layer's marks
  const int64_t words = scan_words(chunks);
  D.d_scan_tmp = own<unsigned long long>(D, 3 * words);
  D.d_unit_mem = own<int32_t>(D, (size_t)ninst * kMaxUnits * kMaxUnit);
  D.d_unit_cnt = own<int32_t>(D, (size_t)ninst * kMaxUnits);
  D.d_reach = own<uint32_t>(D, (size_t)ninst * kMaxResidual * (kMaxResidual / 32));
  if (!D.d_tags || !D.d_chunk_cnt || !D.d_chunk_excl || !D.d_scan_tmp || !D.d_span ||
      !D.d_chunk_list || !D.d_band || !D.d_chunk_inst || !D.d_unit_mem || !D.d_unit_cnt ||
      !D.d_reach)
    return GCR_E_NOMEM;
  bool any_layer2 = false, any_2d = false, any_3d = false;
  for (int i = 0; i < ninst; ++i) {
    any_layer2 = any_layer2 || D.inst[i].layer2;
    any_2d = any_2d || D.inst[i].g.dim == 2;
    any_3d = any_3d || D.inst[i].g.dim == 3;
  }
  PinnedStage PS;
  PS.st = st;
  PS.p = (char*)pinned_alloc(stage_bytes);
  if (!PS.p) return GCR_E_NOMEM;
  std::memcpy(PS.p + o_inst, D.inst.data(), sizeof(Inst) * ninst);
  std::memcpy(PS.p + o_cs, chunk_start.data(), 8 * (ninst + 1));
  std::memset(PS.p + o_info, 0, o_go - o_info);
  PS.pending = true;
  GCR_HIP(hipMemcpyAsync(tb, PS.p, o_go, hipMemcpyHostToDevice, st));   // R1

  StageEvents T((g_profiling.load() & 1) != 0);
  T.mark(0, st);
  ClassifyWork W{D.d_dirty, D.d_dirty_list, D.d_ndirty, D.d_chunk_excl, D.d_scan_tmp, 3 * words,
                 !any_3d};
  ClassifyUpdate U{};
  if (prev) {
    U.span_prev = prev->d_span;
    U.ghost_prev = prev->d_g_cell;
    U.ng_prev = prev->d_g_cell ? prev->g_off[1] : 0;
  }
  launch_classify(D.d_inst, ninst, D.d_chunk_start, chunks, D.d_span, D.d_chunk_inst, D.d_tags,
                  D.d_chunk_cnt, D.d_band, D.d_nband, T.event(10), T.event(11), st, W,
                  prev ? &U : nullptr);
  T.mark(1, st);
  ScanOffsets O{};
  O.start = D.d_chunk_start;
  O.ninst = ninst;
  O.nband = D.d_nband;
  if (any_layer2) {
    // interface counts of the instances, then the second-layer candidates
    // join the list: mark, recount every chunk, scan again
    O.off = D.d_iface_off;
    O.host_off = reinterpret_cast<int64_t*>(PS.p + o_io);
    launch_scan(D.d_chunk_cnt, chunks, D.d_chunk_excl, D.d_chunk_list, D.d_nchunk_list,
                D.d_scan_tmp + words, st, &O);
    // with a chunk list, marks outside it extend it, and the count covers
    // the list; else every chunk is counted
    const bool listed = prev || !W.every_chunk;
    k_l2_mark<<<dim3((unsigned)std::min<int64_t>(chunks, kL2Grid), kL2Split), 256, 0, st>>>(
        D.d_inst, ninst, D.d_chunk_start, D.d_chunk_list, D.d_nchunk_list, D.d_tags,
        listed ? D.d_dirty : nullptr, D.d_dirty_list, D.d_ndirty);
    k_count_marks<<<(unsigned)(listed ? std::min<int64_t>(chunks, kListGrid) : chunks), 256, 0,
                    st>>>(D.d_inst, ninst, D.d_chunk_start, D.d_tags, D.d_chunk_cnt,
                          listed ? D.d_dirty_list : nullptr, D.d_ndirty);
  }
  O.off = D.d_if_off;
  O.host_off = reinterpret_cast<int64_t*>(PS.p + o_if);
  O.hoff = D.d_hoff;
  O.hmask = D.d_hmask;
  O.host_counts = reinterpret_cast<int32_t*>(PS.p + o_nl);
  launch_scan(D.d_chunk_cnt, chunks, D.d_chunk_excl, D.d_chunk_list, D.d_nchunk_list,
              D.d_scan_tmp + 2 * words, st, &O);
  T.mark(2, st);
  GCR_HIP(hipGetLastError());
  GCR_HIP(hipStreamSynchronize(st));
  D.if_off.assign(O.host_off, O.host_off + ninst + 1);
  D.iface_off = D.if_off;   // interface cells alone (second-layer candidates excluded)
  if (any_layer2) std::memcpy(D.iface_off.data(), PS.p + o_io, 8 * (ninst + 1));
  const int32_t nlist = O.host_counts[0];
  D.nband = O.host_counts[1];
  const int64_t nif = D.if_off[ninst];
  const int64_t cap = std::max<int64_t>(nif, 1);
  D.nif = nif;
  D.cap = cap;
  // cell -> ghost tables: at most half full (ghosts <= interface cells);
  // keyed to linear-order ghost indices while the plan is built, remapped
  // to canonical positions once those are known (instance_offsets' sizes)
  D.hoff.assign(ninst + 1, 0);
  D.hmask.assign(ninst, 0);
  for (int i = 0; i < ninst; ++i) {
    int64_t size = 64;
    while (size < 2 * (D.if_off[i + 1] - D.if_off[i])) size <<= 1;
    D.hmask[i] = (uint32_t)(size - 1);
    D.hoff[i + 1] = D.hoff[i] + size;
  }
  D.d_htab = own<unsigned long long>(D, D.hoff[ninst]);
  if (!D.d_htab) return GCR_E_NOMEM;
  const int64_t nblk = (nif + 255) / 256;
  D.d_if_cell = own<int32_t>(D, cap);
  unsigned long long* const posted = own<unsigned long long>(D, nblk + 1);
  D.d_g_cell = own<int32_t>(D, cap);
  D.d_g_ext = own<uint8_t>(D, cap);
  D.d_g_psi = own<double>(D, cap);
  D.d_g_n = own<double>(D, 3 * cap);
  D.d_g_code = own<uint32_t>(D, cap);
  D.d_g_slot = own<uint32_t>(D, cap);
  D.d_deps = own<int32_t>(D, 7 * cap);
  D.d_lev = own<int32_t>(D, cap);
  D.d_blk_idx = own<int32_t>(D, cap);
  D.d_perm = own<int32_t>(D, cap);
  D.d_cell = own<int32_t>(D, cap);
  D.d_delta = own<double>(D, 3 * cap);
  D.d_nrm = own<double>(D, 3 * cap);
  D.d_psi = own<double>(D, cap);
  D.d_code = own<uint32_t>(D, cap);
  D.d_level = own<int32_t>(D, cap);
  D.d_blk = own<int32_t>(D, cap);
  if (any_2d) D.d_cgi = own<int32_t>(D, 3 * cap);
  D.d_listA = own<int32_t>(D, cap);
  D.d_rcnt = own<int32_t>(D, 2 * cap + 1);   // counts, then fill pointers; before, LevelsArgs::flow
  D.d_roff = own<int32_t>(D, cap + 1);
  D.d_dcnt = own<uint8_t>(D, cap);
  D.d_radj = own<int32_t>(D, 7 * cap);
  D.d_cnt = own<uint32_t>(D, (cap >> 2) + ninst + 2);
  D.d_bits = own<uint32_t>(D, (cap >> 5) + ninst + 2);
  if (!D.d_listA || !D.d_rcnt || !D.d_roff || !D.d_radj || !D.d_cnt || !D.d_bits || !D.d_dcnt)
    return GCR_E_NOMEM;
  if (!D.d_if_cell || !posted || !D.d_g_cell || !D.d_g_ext || !D.d_g_psi || !D.d_g_n ||
      !D.d_g_code || !D.d_g_slot || !D.d_deps || !D.d_lev ||
      !D.d_blk_idx || !D.d_perm || !D.d_cell || !D.d_delta || !D.d_nrm || !D.d_psi ||
      !D.d_code || !D.d_level || !D.d_blk || (any_2d && !D.d_cgi))
    return GCR_E_NOMEM;
  T.mark(3, st);
  const BuildResult out_host{reinterpret_cast<InstInfo*>(PS.p + o_info),
                             reinterpret_cast<int64_t*>(PS.p + o_go),
                             reinterpret_cast<int32_t*>(PS.p + o_lo),
                             reinterpret_cast<int32_t*>(PS.p + o_ul)};
  Layering how = kLayerPush;
  FinPart* part = nullptr;
  if (nif > 0) {
    k_compact_iface<<<(unsigned)nlist, 256, 0, st>>>(D.d_inst, D.d_chunk_inst, D.d_tags,
                                                     D.d_chunk_cnt, D.d_chunk_excl, D.d_chunk_list,
                                                     D.d_if_cell, D.d_htab, D.hoff[ninst], posted, nblk + 1);
    T.mark(4, st);
    auto geometry = [&](auto kernel, unsigned bs) {
      kernel<<<blocks(nif, bs), bs, 0, st>>>(
          D.d_inst, ninst, D.d_if_off, D.d_if_cell, D.d_tags, cap, posted, D.d_hoff, D.d_hmask,
          D.d_htab, D.d_g_off, D.d_g_cell, D.d_g_psi, D.d_g_n, D.d_g_ext, D.d_g_slot, D.d_rcnt,
          D.d_info);
    };
    if (nif <= kGeometrySmall) geometry(k_geometry<256>, 256);
    else geometry(k_geometry<1024>, 1024);
    T.mark(5, st);
    int64_t max_if = 0;
    for (int i = 0; i < ninst; ++i) max_if = std::max(max_if, D.if_off[i + 1] - D.if_off[i]);
    // a plan alone: the whole GPU for large 3D bodies (in 2D, where concave
    // bodies have cycles and chains are long, only when asked for)
    const bool flow = ninst == 1 && max_if >= wide_layering_min() &&
                      (any_3d || wide_layering_forced());
    how = flow ? kLayerFlow : levels_pull(max_if) ? kLayerPull : kLayerPush;
    part = own<FinPart>(D, (cap + 63) / 64);
    if (!part) return GCR_E_NOMEM;
    k_deps<<<blocks(nif, 256), 256, 0, st>>>(D.d_inst, ninst, D.d_g_off, D.d_g_cell, D.d_g_psi,
                                              D.d_g_n, cap, D.d_g_ext, D.d_tags, D.d_htab,
                                              D.d_hoff, D.d_hmask, D.d_g_code, D.d_deps, D.d_lev,
                                              D.d_info, part);
    const gcr_status s = build_levels(D, st, ninst, nif, max_if, how, part, out_host, T);
    if (s != GCR_OK) return s;
  } else {
    k_hash_clear<<<blocks(D.hoff[ninst], 256), 256, 0, st>>>(D.d_htab, D.hoff[ninst]);
    for (int i = 4; i <= 9; ++i) T.mark(i, st);
    GCR_HIP(hipMemsetAsync(D.d_g_off, 0, sizeof(int64_t) * (ninst + 1), st));
    GCR_HIP(hipMemsetAsync(D.d_lev_off, 0, sizeof(int32_t) * ninst * (kMaxLevels + 1), st));
    GCR_HIP(hipMemcpyAsync(PS.p + o_info, tb + o_info, o_go - o_info, hipMemcpyDeviceToHost, st));
    std::memset(out_host.g_off, 0, sizeof(int64_t) * (ninst + 1));
    for (int i = 0; i < ninst; ++i) out_host.lev_off[(size_t)i * (kMaxLevels + 1)] = 0;
  }
  GCR_HIP(hipGetLastError());
  D.g_off.resize(ninst + 1);
  D.info.resize(ninst);
  for (;;) {
    GCR_HIP(hipStreamSynchronize(st));
    std::memcpy(D.g_off.data(), PS.p + o_go, 8 * (ninst + 1));
    std::memcpy(D.info.data(), PS.p + o_info, sizeof(InstInfo) * ninst);
    bool again = false;
    for (int i = 0; i < ninst && how != kLayerPush; ++i)
      again = again || (!D.info[i].layered && !D.info[i].err && D.g_off[i + 1] > D.g_off[i]);
    if (!again) break;
    // graphs that these layerings leave (deeper than their tables, a unit
    // beyond the solver's size, a cycle in a large 3D one): those once more,
    // a cycle by the pull form where it fits
    int64_t max_if = 0;
    for (int i = 0; i < ninst; ++i) max_if = std::max(max_if, D.if_off[i + 1] - D.if_off[i]);
    how = how == kLayerFlow && levels_pull(max_if) ? kLayerPull : kLayerPush;
    const gcr_status s = build_levels(D, st, ninst, nif, max_if, how, part, out_host, T);
    if (s != GCR_OK) return s;
  }
  PS.pending = false;
  // each instance's level offsets and units' levels, one after another
  D.lev_at.resize(ninst);
  D.unit_at.resize(ninst);
  D.lev_off.clear();
  D.unit_lev.clear();
  for (int i = 0; i < ninst; ++i) {
    const int32_t* const lo = out_host.lev_off + (size_t)i * (kMaxLevels + 1);
    const int32_t* const ul = out_host.unit_lev + (size_t)i * kMaxUnits;
    D.lev_at[i] = D.lev_off.size();
    D.unit_at[i] = D.unit_lev.size();
    if (D.info[i].err) continue;   // (the build fails below)
    D.lev_off.insert(D.lev_off.end(), lo, lo + D.info[i].nlev + 1);
    D.unit_lev.insert(D.unit_lev.end(), ul, ul + D.info[i].nunits);
  }
  T.collect(std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_call)
                .count());
  D.flow_order = how == kLayerFlow;
  D.ng_total = D.g_off[ninst];
  for (int i = 0; i < ninst; ++i) {
    gcr_status s = status_from_err(D.info[i].err);
    if (s != GCR_OK) return s;
  }
  GCR_HIP(hipGetLastError());
  *out = B;
  return GCR_OK;
}

void make_plan_view(const std::shared_ptr<BatchData>& B, int i, gcr_plan* p) {
  const BatchData& D = *B;
  p->batch = B;
  p->index = i;
  p->inst = D.inst[i];
  p->dim = p->inst.g.dim;
  p->ncell = p->inst.g.ncell;
  p->goff = D.g_off[i];
  p->ng = D.g_off[i + 1] - D.g_off[i];
  p->nif = D.iface_off[i + 1] - D.iface_off[i];
  p->stride = D.cap;
  p->info = D.info[i];
  p->nlev = p->info.nlev;
  p->lev_off.assign(D.lev_off.begin() + D.lev_at[i],
                    D.lev_off.begin() + D.lev_at[i] + p->nlev + 1);
  p->tags = D.d_tags + p->inst.cell_off;
  p->span = D.d_span + p->inst.chunk_off * (kChunk / (64 * kSeg));
  const int64_t o = p->goff;
  if (D.d_cell) {
    p->cell = D.d_cell + o;
    for (int a = 0; a < 3; ++a) {
      p->delta[a] = D.d_delta + a * D.cap + o;
      p->nrm[a] = D.d_nrm + a * D.cap + o;
    }
    p->psi = D.d_psi + o;
    p->code = D.d_code + o;
    p->level = D.d_level + o;
    p->blk = D.d_blk + o;
    // (the whole-GPU layering finds the positions too late for the table)
    p->cgi = p->dim == 2 && !D.flow_order && D.d_cgi ? D.d_cgi + o : nullptr;
  }
  p->fill_fault = &D.d_info[i].fill_fault;
  p->unit_mem = D.d_unit_mem + (int64_t)i * kMaxUnits * kMaxUnit;
  p->unit_cnt = D.d_unit_cnt + (int64_t)i * kMaxUnits;
  p->d_lev_off = D.d_lev_off + (int64_t)i * (kMaxLevels + 1);
  p->unit_lev = D.d_unit_lev + (int64_t)i * kMaxUnits;
  p->unit_lev_host.assign(D.unit_lev.begin() + D.unit_at[i],
                          D.unit_lev.begin() + D.unit_at[i] + p->info.nunits);
  p->htab = D.d_htab + D.hoff[i];
  p->hmask = D.hmask[i];
}

}  // namespace gcr
