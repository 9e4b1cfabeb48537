// Radius neighbours of a range of points (Extend's connection step, Sec. III): for every
// new point v, the earlier points u with 0 < |x_u - x_v|^2 <= r^2 whose segment is free.
//
// The distance test of all pairs is a contraction: with f16 roundings y of the scaled
// points 64 (x - 1/2),
//   y_u . y_v - |y_u|^2 / 2 - |y_v|^2 / 2 + T / 2  =  (T - |y_u - y_v|^2) / 2,
// so one v_mfma_f32_32x32x16_f16 decides 32 x 32 pairs: eight coordinates (zero padded),
// the two half norms as a high and a low f16 part each, against ones.  A non-negative
// result makes the pair a candidate.  T covers the radius plus every rounding:
//   - a coordinate of [0, 1] scales into [-32, 32], where an f16 is within 2^-7 of it
//     (2^-13 before scaling), so two points' distance moves by at most 2 sqrt(D) 2^-13;
//     the norms are those of the rounded points, exactly;
//   - the norms' two parts and the binary32 accumulation of 16 products of at most
//     512 D + T / 2 are off by less than 0.004 D + 2^-18 T (each 16 2^-23 of the
//     largest term, four times over).
// So every true neighbour is a candidate, and about 4% (6D, 100k points) of the
// candidates are not neighbours.  The exact binary64 test, the segment test and the
// ascending order of a row follow per row (k_search_finish), over some sixty candidates
// instead of all earlier points.  The points must lie in [0, 1]^D (the scene's cube);
// otherwise the caller's all-pairs search in binary64 does the whole job.
//
// Measured (all rows of 200,000 6D points / 1,000 new points against 100,000): the
// all-pairs search took 26.3 ms / 1.97 ms in its two passes (binary64 VALU bound, and one
// workgroup per 256 rows and 8,192 points leaves the chip idle in the second case), the
// candidates 1.44 ms / 19 us (the matrix instruction and the maximum over its results:
// about 180 cycles a tile).
#include <cmath>

#include "internal.h"
#include "search.h"

namespace pirrt {

namespace {

constexpr int kThreads = 256;
constexpr int kStage = 256;  // points staged in LDS together

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Two f16 values in one word (the first in the low half), and back.
__device__ __forceinline__ uint32_t pack2(_Float16 a, _Float16 b) {
  return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}
__device__ __forceinline__ float low_half(uint32_t w) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu));
}
__device__ __forceinline__ float high_half(uint32_t w) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
}

// A record: the eight scaled coordinates, then {-|y|^2/2 (high, low), 1, 1, 0, 0, 0, 0}:
// the K = 16 operand of a row of the first matrix.
template <int D>
__global__ void __launch_bounds__(kThreads) k_search_pack(int64_t first, int64_t n, const double* __restrict__ pts,
                                                          uint4* __restrict__ rec, SearchState* __restrict__ state) {
  const int64_t i = first + (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    state->most = 0;
    state->listed = 0;
    state->wide = 0;
    state->crowded = 0;
    state->nnz = 0;
  }
  if (i >= n) return;
  _Float16 y[8];
  double norm = 0.0;
  bool in = true;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    y[k] = (_Float16)0.0f;
    if (k < D) {
      const double x = pts[i * D + k];
      in = in && x >= 0.0 && x <= 1.0;
      y[k] = (_Float16)(float)((x - 0.5) * 64.0);
      norm += (double)(float)y[k] * (double)(float)y[k];
    }
  }
  const float half = (float)(0.5 * norm);
  const _Float16 hi = (_Float16)half, lo = (_Float16)(half - (float)hi), one = (_Float16)1.0f;
  rec[2 * i] = make_uint4(pack2(y[0], y[1]), pack2(y[2], y[3]), pack2(y[4], y[5]), pack2(y[6], y[7]));
  rec[2 * i + 1] = make_uint4(pack2(-hi, -lo), pack2(one, one), 0u, 0u);
  if (!in) atomicOr(&state->outside, 1);
}

// A wave owns NB blocks of 32 rows, a workgroup 4 NB of them, and takes NU tiles of 32
// earlier points together (NB x NU = 4 independent matrix instructions); the earlier points of the
// workgroup's chunk go through LDS in stages of 256 (8 tiles), the next stage's loads in
// flight.  Lane l holds column l % 32 of a block's result: the two lanes of a row share
// its candidate count in registers, and candidates are written as they are found, in no
// order, with no atomics.  A tile without a candidate (most of them) costs the matrix
// instruction, a three-way maximum over the 16 results' bits and a branch.
// (Two waves per SIMD at least: the compiler then keeps the results in VGPRs, where the
// maximum reads them, instead of accumulation registers.)
template <int NB, int NU>
__global__ void __launch_bounds__(kThreads, 2) k_search(int64_t n_old, int64_t n, int64_t row0, int32_t rows,
                                                     const uint4* __restrict__ rec, float half_t, int32_t nch,
                                                     int64_t chunk, int32_t cap, int32_t* __restrict__ cand,
                                                     int32_t* __restrict__ cnt, SearchState* __restrict__ state) {
  __shared__ uint4 tile[2][2 * kStage];
  if (state->outside) return;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int col = lane & 31, half = lane >> 5;
  // the last rows have the most earlier points: they start first
  const int64_t group = (int64_t)gridDim.x - 1 - blockIdx.x;
  const int64_t r_wg = group * (4 * NB * 32), r_wave = r_wg + (int64_t)wave * (NB * 32);
  const int64_t c = blockIdx.y;
  const int64_t rows_end = r_wg + 4 * NB * 32 < rows ? r_wg + 4 * NB * 32 : rows;
  const int64_t u_begin = c * chunk;
  const int64_t v_end = n_old + row0 + rows_end;  // every u of the workgroup is below it
  const int64_t u_end = u_begin + chunk < v_end ? u_begin + chunk : v_end;
  f16x8 vb[NB];
  int32_t found[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    found[b] = 0;
    int64_t v = n_old + row0 + r_wave + b * 32 + col;
    if (v > n - 1) v = n - 1;
    uint4 w = rec[2 * v + half];
    if (half) {  // the second matrix: ones against the first's norms, (T - |y_v|^2) / 2 against its ones
      const float t = half_t + (low_half(w.x) + high_half(w.x));
      const _Float16 hi = (_Float16)t;
      w.x = w.y;
      w.y = pack2(hi, (_Float16)(t - (float)hi));
    }
    vb[b] = __builtin_bit_cast(f16x8, w);
  }
  uint4 next0 = make_uint4(0u, 0u, 0u, 0u), next1 = next0;
  if (u_begin < u_end) {
    next0 = rec[2 * u_begin + threadIdx.x];
    next1 = rec[2 * u_begin + kThreads + threadIdx.x];
  }
  int buf = 0;
  for (int64_t u0 = u_begin; u0 < u_end; u0 += kStage, buf ^= 1) {
    tile[buf][threadIdx.x] = next0;
    tile[buf][kThreads + threadIdx.x] = next1;
    __syncthreads();  // two buffers: one barrier a stage
    if (u0 + kStage < u_end) {
      next0 = rec[2 * (u0 + kStage) + threadIdx.x];
      next1 = rec[2 * (u0 + kStage) + kThreads + threadIdx.x];
    }
    const int tiles = u_end - u0 < kStage ? (int)((u_end - u0 + 31) / 32) : kStage / 32;
    for (int t0 = 0; t0 < tiles; t0 += NU) {
      f32x16 acc[NU][NB];
#pragma unroll
      for (int j = 0; j < NU; ++j) {
        const f16x8 a = __builtin_bit_cast(f16x8, tile[buf][2 * (32 * (t0 + j) + col) + half]);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          f32x16 zero;
#pragma unroll
          for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
          acc[j][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, vb[b], zero, 0, 0, 0);
        }
      }
#pragma unroll
      for (int jb = 0; jb < NU * NB; ++jb) {
        const int j = jb / NB, b = jb % NB, t = t0 + j;
        if (t >= tiles) break;
        int top = __float_as_int(acc[j][b][0]);
#pragma unroll
        for (int r = 1; r < 16; ++r) {
          const int x = __float_as_int(acc[j][b][r]);
          top = x > top ? x : top;
        }
        if (__ballot(top >= 0) == 0ull) continue;  // no sign bit is clear: no candidate
        uint32_t neg = 0;
#pragma unroll
        for (int r = 15; r >= 0; --r) neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[j][b][r]), 31);
        uint32_t m = ~neg & 0xffffu;  // bit r: result r, point 8 (r / 4) + 4 half + r % 4 of the tile
        const int64_t row = r_wave + b * 32 + col, v = n_old + row0 + row;
        const int64_t ut = u0 + 32 * t;
        if (ut + 32 > v) {  // the last tile of a row: earlier points only
          uint32_t keep = 0;
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (ut + 8 * (r >> 2) + 4 * half + (r & 3) < v) keep |= 1u << r;
          m &= keep;
        }
        const int mine = __popc(m);
        const int other = __shfl_xor(mine, 32, kWave);
        int32_t pos = found[b] + (half ? other : 0);
        found[b] += mine + other;
        if (row < rows) {
          int32_t* list = cand + ((int64_t)row * nch + c) * cap;
          while (m) {
            const int r = __ffs(m) - 1;
            m &= m - 1;
            if (pos < cap) list[pos] = (int32_t)(ut + 8 * (r >> 2) + 4 * half + (r & 3));
            ++pos;
          }
        }
      }
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int64_t row = r_wave + b * 32 + col;
    if (half == 0 && row < rows) {
      cnt[row * nch + c] = found[b];
      if (found[b] > cap) atomicMax(&state->most, found[b]);
    }
  }
}

// One group of 32 lanes per row: gathers the row's candidate lists, tests them exactly
// (binary64 distance, then the segment), and writes the survivors in ascending order of
// the neighbour id (each finds its rank among the row's survivors in LDS) with their
// costs over the row's candidates.
constexpr int kFinLanes = 32;
constexpr int kFinRows = kThreads / kFinLanes;
constexpr int kRankStep = 8;  // ids compared per step of the ranking

template <int D>
__global__ void __launch_bounds__(kThreads) k_search_finish(int64_t n_old, int64_t row0, int32_t rows, double r2,
                                                            const double* __restrict__ pts, ObsView ob, int32_t nch,
                                                            int32_t cap, int32_t crowd, int32_t* __restrict__ cand,
                                                            const int32_t* __restrict__ cnt,
                                                            float* __restrict__ ccost, int32_t* __restrict__ deg,
                                                            SearchState* __restrict__ state) {
  __shared__ int32_t ids[kFinRows][kSearchRowMax + kRankStep];
  __shared__ float cst[kFinRows][kSearchRowMax];
  __shared__ NearObstacles<D> spheres;
  if (state->outside || state->most) return;
  spheres.load(ob);
  const int g = threadIdx.x / kFinLanes, l = threadIdx.x % kFinLanes;
  const int64_t row = (int64_t)blockIdx.x * kFinRows + g;
  const bool live = row < rows;
  // the lists one after the other (a lane per list at a time)
  int total = 0;
  for (int c0 = 0; c0 < nch; c0 += kFinLanes) {
    const int c = c0 + l;
    const int k = live && c < nch ? cnt[row * nch + c] : 0;
    if (k > crowd && !state->crowded) state->crowded = 1;
    int incl = k;
#pragma unroll
    for (int off = 1; off < kFinLanes; off <<= 1) {
      const int y = __shfl_up(incl, off, kFinLanes);
      if (l >= off) incl += y;
    }
    const int at = total + incl - k;
    total += __shfl(incl, kFinLanes - 1, kFinLanes);
    if (nch > 1 && k > 0) {  // (lists are 16 bytes aligned: their room is a multiple of 4)
      const int4* list = reinterpret_cast<const int4*>(cand + (row * nch + c) * cap);
      for (int i = 0; i < k; i += 4) {
        const int4 w = list[i / 4];
        const int32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i + e < k && at + i + e < kSearchRowMax) ids[g][at + i + e] = u[e];
      }
    }
  }
  if (total > kSearchRowMax) {
    if (l == 0) atomicMax(&state->listed, total);
    total = 0;
  }
  int32_t* out = cand + row * nch * cap;
  float* outc = ccost + row * nch * cap;
  if (nch == 1)
    for (int i = l; i < total; i += kFinLanes) ids[g][i] = out[i];
  __syncthreads();  // the obstacles' spheres; from here on a row's LDS traffic stays inside its wave
  const int64_t v = n_old + row0 + row;
  double xv[D];
#pragma unroll
  for (int k = 0; k < D; ++k) xv[k] = live ? pts[v * D + k] : 0.0;
  int kept = 0;
  for (int i0 = 0; __ballot(i0 < total) != 0ull; i0 += kFinLanes) {
    bool ok = i0 + l < total;
    int32_t u = 0;
    float w = 0.0f;
    if (ok) {
      u = ids[g][i0 + l];
      double xu[D];
#pragma unroll
      for (int k = 0; k < D; ++k) xu[k] = pts[(int64_t)u * D + k];
      const double d2 = dist2<D>(xu, xv);
      ok = d2 <= r2 && d2 > 0.0;
      if (ok) {
        w = __double2float_rn(__dsqrt_rn(d2));
        ok = !spheres.segment_blocked(xu, xv, d2, ob);
      }
    }
    const uint32_t bits = (uint32_t)(__ballot(ok) >> (threadIdx.x & 32));
    if (ok) {  // kept <= i0: the survivors overwrite candidates already read
      const int p = kept + __popc(bits & ((1u << l) - 1u));
      ids[g][p] = u;
      cst[g][p] = w;
    }
    kept += __popc(bits);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if (l < kRankStep) ids[g][kept + l] = INT32_MAX;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  for (int i = l; i < kept; i += kFinLanes) {
    const int32_t u = ids[g][i];
    int rank = 0;
    for (int j = 0; j < kept; j += kRankStep)
#pragma unroll
      for (int e = 0; e < kRankStep; ++e) rank += ids[g][j + e] < u;
    out[rank] = u;
    outc[rank] = cst[g][i];
  }
  if (live && l == 0) deg[row] = kept;
}

// The same with a workgroup per row, for rows of hundreds of candidates or more (samples
// crowded along a corridor, connection radii of a good part of the cube).  The survivors of a
// window of ids are bits in LDS, so their order costs a count over its words, whatever their
// number: ranking a row's survivors against each other was most of the time from a thousand
// on, and rows of more than 4,096 candidates went to the all-pairs search after all (all rows of
// 10,000 2D points with 2,548 entries each 5.9 ms; the all-pairs search alone 3.5).
//
// A window is as many chunks of earlier points as fit the bits.  The row's finished ids take the
// place of its candidates: those of chunks [0, c) are no more than these chunks' candidates,
// and a window's are read before its ids are written.
constexpr int kWideThreads = 1024;

template <int D>
__global__ void __launch_bounds__(kWideThreads) k_search_finish_wide(int64_t n, int64_t n_old, int64_t row0, double r2,
                                                                 const double* __restrict__ pts, ObsView ob,
                                                                 int32_t nch, int64_t chunk, int32_t cap,
                                                                 int32_t crowd, int32_t* cand,
                                                                 const int32_t* __restrict__ cnt,
                                                                 float* __restrict__ ccost,
                                                                 int32_t* __restrict__ deg,
                                                                 SearchState* __restrict__ state) {
  __shared__ uint32_t bits[kSearchWindow / 32 + kSearchWindow / 1024];
  __shared__ NearObstacles<D> spheres;
  __shared__ int32_t at[kSearchMaxChunks + 1];
  __shared__ int32_t wsum[kWideThreads / kWave];
  static_assert(kSearchMaxChunks <= kWave, "one wave adds up the lists");
  if (state->outside || state->most) return;
  spheres.load(ob);
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  const int64_t row = blockIdx.x;
  if (wave == 0) {
    const int k = lane < nch ? cnt[row * nch + lane] : 0;
    int incl = k;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int y = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += y;
    }
    if (lane == 0) at[0] = 0;
    if (lane < nch) at[lane + 1] = incl;
    if (__ballot(k > crowd) != 0ull && lane == 0 && !state->crowded) state->crowded = 1;
  }
  __syncthreads();
  auto word = [](int w) { return w + (w >> 5); };  // consecutive words of a thread, other banks
  int32_t* out = cand + row * nch * cap;
  float* outc = ccost + row * nch * cap;
  const int64_t v = n_old + row0 + row;
  // (the rows of the last points have all n to find candidates among)
  if (t == 0 && at[nch] * n > kSearchRowMax * v && state->wide == 0) state->wide = 1;
  double xv[D];
#pragma unroll
  for (int k = 0; k < D; ++k) xv[k] = pts[v * D + k];
  const int per = (int)(kSearchWindow / chunk);
  int kept = 0;
  for (int c0 = 0; c0 < nch && c0 * chunk < v; c0 += per) {
    const int c1 = c0 + per < nch ? c0 + per : nch;
    const int64_t u0 = c0 * chunk, u1 = c1 * chunk < v ? c1 * chunk : v;
    const int words = (int)((u1 - u0 + 31) / 32);
    for (int w = t; w < words; w += kWideThreads) bits[word(w)] = 0u;
    __syncthreads();
    for (int i = at[c0] + t; i < at[c1]; i += kWideThreads) {
      int c = c0;  // the list that holds candidate i
      for (int top = c1; top - c > 1;) {
        const int mid = (c + top) / 2;
        if (at[mid] <= i)
          c = mid;
        else
          top = mid;
      }
      const int32_t u = out[(int64_t)c * cap + (i - at[c])];
      double xu[D];
#pragma unroll
      for (int k = 0; k < D; ++k) xu[k] = pts[(int64_t)u * D + k];
      const double d2 = dist2<D>(xu, xv);
      if (d2 <= r2 && d2 > 0.0 && !spheres.segment_blocked(xu, xv, d2, ob)) {
        const int x = (int)(u - u0);
        atomicOr(&bits[word(x >> 5)], 1u << (x & 31));
      }
    }
    __syncthreads();
    // the window's ids in order: a run of words a thread
    const int each = (words + kWideThreads - 1) / kWideThreads;
    const int w0 = t * each, w1 = w0 + each < words ? w0 + each : words;
    int mine = 0;
    for (int w = w0; w < w1; ++w) mine += __popc(bits[word(w)]);
    int incl = mine;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int y = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += y;
    }
    if (lane == kWave - 1) wsum[wave] = incl;
    __syncthreads();
    int pos = kept + incl - mine, end = kept;
#pragma unroll
    for (int j = 0; j < kWideThreads / kWave; ++j) {
      if (j < wave) pos += wsum[j];
      end += wsum[j];
    }
    for (int w = w0; w < w1; ++w)
      for (uint32_t m = bits[word(w)]; m; m &= m - 1) out[pos++] = (int32_t)(u0 + 32 * w + __ffs(m) - 1);
    __syncthreads();
    for (int i = kept + t; i < end; i += kWideThreads) {
      double xu[D];
#pragma unroll
      for (int k = 0; k < D; ++k) xu[k] = pts[(int64_t)out[i] * D + k];
      outc[i] = __double2float_rn(__dsqrt_rn(dist2<D>(xu, xv)));
    }
    kept = end;
  }
  if (t == 0) deg[row] = kept;
}

// Finished rows into CSR, kCsrRows a workgroup (one where they are long: 181 rows of 10,000
// entries took 920 us at 32).  Up to kPrefixRows rows each workgroup sums the lengths of the
// rows before its own itself (one launch instead of a scan's three); above, `off` holds their
// exclusive sums.
constexpr int32_t kPrefixRows = 16384;

template <int kCsrRows>
__global__ void __launch_bounds__(kThreads) k_search_rows(int32_t rows, int32_t stride, const int32_t* __restrict__ deg,
                                                          const int64_t* __restrict__ off,
                                                          const int32_t* __restrict__ cand,
                                                          const float* __restrict__ ccost, int64_t base,
                                                          int64_t capacity, int64_t* __restrict__ rp,
                                                          int32_t* __restrict__ col, float* __restrict__ cost,
                                                          const SearchState* __restrict__ state,
                                                          SearchState* __restrict__ report) {
  __shared__ int64_t start[kCsrRows + 1];
  __shared__ int64_t part[2][kThreads / kWave];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    report->outside = state->outside;
    report->most = state->most;
    report->listed = state->listed;
    report->wide = state->wide;
    report->crowded = state->crowded;
  }
  if (state->outside || state->most || state->listed) return;
  const int32_t first = blockIdx.x * kCsrRows;
  const int32_t last = first + kCsrRows < rows ? first + kCsrRows : rows;
  int64_t total;
  if (off) {
    if (threadIdx.x <= last - first) start[threadIdx.x] = off[first + threadIdx.x];
    total = off[rows];
  } else {
    int64_t before = 0, all = 0;
    for (int32_t i = threadIdx.x; i < rows; i += kThreads) {
      const int32_t k = deg[i];
      all += k;
      if (i < first) before += k;
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
      before += __shfl_xor(before, o, kWave);
      all += __shfl_xor(all, o, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
      part[0][threadIdx.x / kWave] = before;
      part[1][threadIdx.x / kWave] = all;
    }
    __syncthreads();
    before = part[0][0] + part[0][1] + part[0][2] + part[0][3];
    total = part[1][0] + part[1][1] + part[1][2] + part[1][3];
    if (threadIdx.x < kWave) {
      const int i = first + threadIdx.x;
      const int k = threadIdx.x < kCsrRows && i < rows ? deg[i] : 0;
      int incl = k;
#pragma unroll
      for (int o = 1; o < kCsrRows; o <<= 1) {
        const int y = __shfl_up(incl, o, kWave);
        if ((int)threadIdx.x >= o) incl += y;
      }
      if (threadIdx.x < kCsrRows) start[threadIdx.x] = before + incl - k;
      if (threadIdx.x == kCsrRows - 1) start[kCsrRows] = before + incl;
    }
  }
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) report->nnz = base + total;
  if (base + total > capacity) return;
  if (threadIdx.x < last - first) rp[first + threadIdx.x] = base + start[threadIdx.x];
  if (last == rows && threadIdx.x == 0) rp[rows] = base + total;
  // a group of lanes per row: every row of the workgroup at once
  constexpr int kLanes = kThreads / kCsrRows;
  const int i = threadIdx.x / kLanes;
  if (i >= last - first) return;
  const int64_t from = (int64_t)(first + i) * stride, to = base + start[i];
  const int k = (int)(start[i + 1] - start[i]);
#pragma unroll 4
  for (int j = threadIdx.x % kLanes; j < k; j += kLanes) {
    if (col) col[to + j] = cand[from + j];
    if (cost) cost[to + j] = ccost[from + j];
  }
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per > 0 ? (n + per - 1) / per : 1); }

// The threshold T / 2 of the candidate test, in scaled units (see the top of the file).
float half_threshold(int d, double radius) {
  const double r = (radius < 4.0 ? radius : 4.0) + 2.0 * std::sqrt((double)d) * std::ldexp(1.0, -13) * 1.001;
  const double t = 4096.0 * r * r;
  const double slack = 0.004 * d + t * std::ldexp(1.0, -18);
  return (float)((0.5 * t + slack) * (1.0 + std::ldexp(1.0, -20)));
}

}  // namespace

#define PIRRT_SEARCH_DIM(d, call) \
  switch (d) {                    \
    case 1: call(1); break;       \
    case 2: call(2); break;       \
    case 3: call(3); break;       \
    case 4: call(4); break;       \
    case 5: call(5); break;       \
    case 6: call(6); break;       \
    case 7: call(7); break;       \
    default: call(8); break;      \
  }

void launch_search_pack(int d, int64_t first, int64_t n, const double* pts, uint4* rec, SearchState* state,
                        hipStream_t s) {
#define PACK(D)                                                                                                  \
  hipLaunchKernelGGL(k_search_pack<D>, dim3(blocks_for(n - first, kThreads)), dim3(kThreads), 0, s, first, n, pts, \
                     rec, state)
  PIRRT_SEARCH_DIM(d, PACK)
#undef PACK
}

void launch_search(const SearchArgs& a, hipStream_t s) {
  const float ht = half_threshold(a.d, a.radius);
  // four blocks of rows per wave share each point's load; with few rows one block per
  // wave gives the chip more waves
  if (a.rows >= kSearchWideRows)
    hipLaunchKernelGGL((k_search<4, 1>), dim3(blocks_for(a.rows, 512), (unsigned)a.nch), dim3(kThreads), 0, s, a.n_old, a.n,
                       a.row0, a.rows, a.rec, ht, a.nch, a.chunk, a.cap, a.cand, a.cnt, a.state);
  else
    hipLaunchKernelGGL((k_search<1, 4>), dim3(blocks_for(a.rows, 128), (unsigned)a.nch), dim3(kThreads), 0, s, a.n_old, a.n,
                       a.row0, a.rows, a.rec, ht, a.nch, a.chunk, a.cap, a.cand, a.cnt, a.state);
#define FINISH(D)                                                                                                   \
  hipLaunchKernelGGL(k_search_finish<D>, dim3(blocks_for(a.rows, kFinRows)), dim3(kThreads), 0, s, a.n_old, a.row0, \
                     a.rows, a.radius * a.radius, a.pts, a.obs, a.nch, a.cap, a.crowd, a.cand, a.cnt, a.ccost, a.deg,          \
                     a.state)
#define WIDE(D)                                                                                                      \
  hipLaunchKernelGGL(k_search_finish_wide<D>, dim3((unsigned)a.rows), dim3(kWideThreads), 0, s, a.n, a.n_old, a.row0, \
                     a.radius * a.radius, a.pts, a.obs, a.nch, a.chunk, a.cap, a.crowd, a.cand, a.cnt, a.ccost, a.deg, a.state)
  if (a.wide) {
    PIRRT_SEARCH_DIM(a.d, WIDE)
  } else {
    PIRRT_SEARCH_DIM(a.d, FINISH)
  }
#undef WIDE
#undef FINISH
}

void launch_search_rows(const SearchArgs& a, int64_t base, int64_t capacity, int64_t* row_ptr, int32_t* col,
                        float* cost, int64_t* off, void* scan, hipStream_t s) {
  const int64_t* offs = nullptr;
  if (a.rows > kPrefixRows) {
    scan_i32_to_i64(a.deg, a.rows, off, scan, s);
    offs = off;
  }
#define ROWS(R)                                                                                                     \
  hipLaunchKernelGGL(k_search_rows<R>, dim3(blocks_for(a.rows, R)), dim3(kThreads), 0, s, a.rows, a.nch * a.cap, a.deg, \
                     offs, a.cand, a.ccost, base, capacity, row_ptr + a.row0, col, cost, a.state, a.report)
  if (a.wide)
    ROWS(1);
  else
    ROWS(32);
#undef ROWS
}

}  // namespace pirrt
