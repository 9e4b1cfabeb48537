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

}  // namespace pirrt
