// Obstacle and segment geometry of the exploration kernels, in explicitly rounded
// binary64 operations (the library's definitions are in include/pirrt.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pirrt {

struct ObsView {
  int32_t n;
  const int32_t* kind;
  const double* centre;
  const double* size;
};

template <int D>
__device__ __forceinline__ bool point_blocked(const double* x, const ObsView& ob) {
  for (int o = 0; o < ob.n; ++o) {
    const double* c = ob.centre + (int64_t)o * D;
    const double* s = ob.size + (int64_t)o * D;
    if (ob.kind[o] == 0) {
      double d2 = 0.0;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const double e = x[k] - c[k];
        d2 = __dadd_rn(d2, __dmul_rn(e, e));
      }
      if (d2 <= __dmul_rn(s[0], s[0])) return true;
    } else {
      bool inside = true;
#pragma unroll
      for (int k = 0; k < D; ++k)
        if (fabs(x[k] - c[k]) > s[k]) inside = false;
      if (inside) return true;
    }
  }
  return false;
}

template <int D>
__device__ __forceinline__ bool hits_sphere(const double* a, const double* b, const double* c, double rad) {
  double ee = 0.0, ce = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const double e = b[k] - a[k];
    ee = __dadd_rn(ee, __dmul_rn(e, e));
    ce = __dadd_rn(ce, __dmul_rn(c[k] - a[k], e));
  }
  double t = ee > 0.0 ? __ddiv_rn(ce, ee) : 0.0;
  if (t < 0.0) t = 0.0;
  if (t > 1.0) t = 1.0;
  double q2 = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const double q = __dadd_rn(a[k], __dmul_rn(t, b[k] - a[k])) - c[k];
    q2 = __dadd_rn(q2, __dmul_rn(q, q));
  }
  return q2 <= __dmul_rn(rad, rad);
}

template <int D>
__device__ __forceinline__ bool hits_box(const double* a, const double* b, const double* c, const double* half) {
  double lo_t = 0.0, hi_t = 1.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const double lo = c[k] - half[k], hi = c[k] + half[k];
    const double e = b[k] - a[k];
    if (e == 0.0) {
      if (a[k] < lo || a[k] > hi) return false;
      continue;
    }
    double t_lo = __ddiv_rn(lo - a[k], e), t_hi = __ddiv_rn(hi - a[k], e);
    if (t_lo > t_hi) {
      const double s = t_lo;
      t_lo = t_hi;
      t_hi = s;
    }
    if (t_lo > lo_t) lo_t = t_lo;
    if (t_hi < hi_t) hi_t = t_hi;
    if (lo_t > hi_t) return false;
  }
  return true;
}

template <int D>
__device__ __forceinline__ bool segment_blocked(const double* a, const double* b, const ObsView& ob) {
  for (int o = 0; o < ob.n; ++o) {
    const double* c = ob.centre + (int64_t)o * D;
    const double* s = ob.size + (int64_t)o * D;
    const bool hit = ob.kind[o] == 0 ? hits_sphere<D>(a, b, c, s[0]) : hits_box<D>(a, b, c, s);
    if (hit) return true;
  }
  return false;
}

template <int D>
__device__ __forceinline__ double dist2(const double* a, const double* b) {
  double d2 = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const double e = a[k] - b[k];
    d2 = __dadd_rn(d2, __dmul_rn(e, e));
  }
  return d2;
}

// Bounding spheres of the first kNearMax obstacles in LDS, in binary32: most obstacles
// are far from a point or a short segment, and one distance to the centre settles that
// for a seventh of the exact test's operations.  A segment of points in the unit cube
// meets an obstacle only if its midpoint lies within the obstacle's bounding radius plus
// half its length of the centre; the binary32 distance (centres within [-4, 4]: off by
// less than 1e-6 a coordinate) is compared with 2e-5 to spare.  Obstacles that are not
// ruled out, and those past kNearMax, take the exact test.  With 40 spheres in 6D the
// exact tests of a batch's rows took 61 us for 1,000 rows and 1.13 ms for 200,000 (a
// chain of obstacle loads and divisions per candidate), with the filter 25 us and 0.39 ms;
// the sampler's candidates 17 -> 6 us a batch.
constexpr int kNearMax = 128;

template <int D>
struct NearObstacles {
  float centre[kNearMax][D];
  float radius[kNearMax];

  __device__ __forceinline__ void load(const ObsView& ob) {  // every thread of the workgroup; a barrier follows
    const int m = ob.n < kNearMax ? ob.n : kNearMax;
    for (int o = threadIdx.x; o < m; o += blockDim.x) {
      double r2 = 0.0;
      bool in = true;
      for (int k = 0; k < D; ++k) {
        const double c = ob.centre[(int64_t)o * D + k], s = ob.size[(int64_t)o * D + k];
        centre[o][k] = (float)c;
        in = in && fabs(c) <= 4.0;
        if (ob.kind[o] != 0 || k == 0) r2 += s * s;
      }
      radius[o] = in && r2 <= 16.0 ? (float)sqrt(r2) * 1.00001f + 2e-5f : __int_as_float(0x7f800000);
    }
  }

  // Bit i: obstacle o0 + i may meet the segment of half length `reach` around x.
  __device__ __forceinline__ uint64_t near(const ObsView& ob, int o0, const float* x, float reach) const {
    const int m = ob.n < kNearMax ? ob.n : kNearMax;
    const int end = o0 + 64 < m ? o0 + 64 : m;
    uint64_t bits = 0;
    for (int o = o0; o < end; ++o) {
      float d2 = 0.0f;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const float e = x[k] - centre[o][k];
        d2 = __fmaf_rn(e, e, d2);
      }
      const float r = radius[o] + reach;
      if (!(d2 > r * r)) bits |= 1ull << (o - o0);
    }
    return bits;
  }

  __device__ __forceinline__ bool point_blocked(const double* x, const ObsView& ob) const {
    float xf[D];
#pragma unroll
    for (int k = 0; k < D; ++k) xf[k] = (float)x[k];
    for (int o0 = 0; o0 < ob.n; o0 += 64) {
      if (o0 >= kNearMax) return pirrt::point_blocked<D>(x, rest(ob));
      for (uint64_t b = near(ob, o0, xf, 0.0f); b; b &= b - 1)
        if (pirrt::point_blocked<D>(x, one(ob, o0 + __ffsll((long long)b) - 1))) return true;
    }
    return false;
  }

  // d2: the squared length of the segment
  __device__ __forceinline__ bool segment_blocked(const double* a, const double* b, double d2, const ObsView& ob) const {
    float x[D];
#pragma unroll
    for (int k = 0; k < D; ++k) x[k] = 0.5f * ((float)a[k] + (float)b[k]);
    const float reach = 0.50001f * sqrtf((float)d2) + 1e-6f;
    for (int o0 = 0; o0 < ob.n; o0 += 64) {
      if (o0 >= kNearMax) return pirrt::segment_blocked<D>(a, b, rest(ob));
      for (uint64_t m = near(ob, o0, x, reach); m; m &= m - 1)
        if (pirrt::segment_blocked<D>(a, b, one(ob, o0 + __ffsll((long long)m) - 1))) return true;
    }
    return false;
  }

 private:
  static __device__ __forceinline__ ObsView one(const ObsView& ob, int o) {
    return ObsView{1, ob.kind + o, ob.centre + (int64_t)o * D, ob.size + (int64_t)o * D};
  }
  static __device__ __forceinline__ ObsView rest(const ObsView& ob) {
    return ObsView{ob.n - kNearMax, ob.kind + kNearMax, ob.centre + (int64_t)kNearMax * D,
                   ob.size + (int64_t)kNearMax * D};
  }
};

}  // namespace pirrt
