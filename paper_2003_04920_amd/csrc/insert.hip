// Inserting a small batch (at most kInsertBlockMax vertices) into a single graph in four
// launches: what store.hip does in a dozen, fused.  A planner's batch of 100 or 1,000
// vertices is bound by the launches and their round trips through memory, not by the
// entries.
//
//   k_insert_prepare : neighbour ids to slots, the new entries of every row counted, the
//                      new vertices' ids.
//   k_insert_offsets : new row offsets (old offset + new entries before the row: every
//                      workgroup sums the counts before its own by itself) and each row's
//                      cursor for the mirrored entries.
//   k_insert_rows    : old rows copied, new rows and their mirrors placed; and of Extend's
//                      local relaxation the part over existing neighbours, whose g is
//                      final, with the entries inside the batch listed.
//   k_insert_policy  : one workgroup finishes the relaxation over the batch's inner edges
//                      in LDS: each new vertex repeats its minimum over its lower
//                      neighbours until a round changes nothing.  An edge always leads to
//                      the higher id, so the fixed point is the serial one.
//
// Batches of 1,000 up to a 6D graph of 30,000 vertices: a dozen kernels of 117 us together
// (the single-workgroup relaxation over whole rows 73 of them) are now four of 45 (8, 8,
// 15 and 14); batches of 100 up to a 2D graph of 10,000: 55 us, now 30.
#include "internal.h"

namespace pirrt {

namespace {

constexpr int kThreads = 256;
constexpr int kRowGW = 8;       // lanes per new row
constexpr int kCopyGW = 32;     // lanes per copied row
constexpr int kOffThreads = 1024;
constexpr int kOffTile = 4 * kOffThreads;

inline unsigned blocks_for(int64_t n, int per_block = kThreads) {
  int64_t b = (n + per_block - 1) / per_block;
  return (unsigned)(b > 0 ? b : 1);
}

__global__ void __launch_bounds__(kThreads) k_insert_prepare(int32_t n_new, int64_t n_old,
                                                             const int64_t* __restrict__ brp,
                                                             const int32_t* __restrict__ bcol,
                                                             int32_t* __restrict__ slot_of, int32_t* __restrict__ ext_of,
                                                             int32_t* __restrict__ bslot, int32_t* __restrict__ add0,
                                                             int32_t* __restrict__ dcount) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = t / kRowGW;
  const int gl = (int)(t % kRowGW);
  if (t == 0) dcount[0] = 0;
  if (i >= n_new) return;
  const int64_t a = brp[i], b = brp[i + 1];
  const int32_t v = (int32_t)(n_old + i);
  if (gl == 0) {
    slot_of[v] = v;
    ext_of[v] = v;
    if (b > a) atomicAdd(&add0[v], (int)(b - a));
  }
  for (int64_t j = a + gl; j < b; j += kRowGW) {
    const int32_t u = bcol[j];
    const int32_t s = u >= n_old ? u : slot_of[u];  // new vertices take the slots of their ids
    bslot[j] = s;
    atomicAdd(&add0[s], 1);
  }
}

__global__ void __launch_bounds__(kOffThreads) k_insert_offsets(int64_t n1, int64_t n_old,
                                                               const int64_t* __restrict__ rp_old,
                                                               const int64_t* __restrict__ brp,
                                                               const int32_t* __restrict__ add0,
                                                               int32_t* __restrict__ add, int64_t* __restrict__ rp_new) {
  __shared__ int64_t wsum[kOffThreads / kWave];
  const int t = threadIdx.x, lane = t & (kWave - 1), wid = t / kWave;
  const int64_t v0 = (int64_t)blockIdx.x * kOffTile;
  // new entries of the rows before this tile
  int64_t before = 0;
  const int4* c4 = reinterpret_cast<const int4*>(add0);
#pragma unroll 4
  for (int64_t q = t; q < v0 / 4; q += kOffThreads) {
    const int4 c = c4[q];
    before += (int64_t)c.x + c.y + c.z + c.w;
  }
  int32_t c[4];
  int64_t mine = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t v = v0 + 4 * t + k;
    c[k] = v < n1 ? add0[v] : 0;
    mine += c[k];
  }
  int64_t incl = mine;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int64_t y = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += y;
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) before += __shfl_xor(before, off, kWave);
  // wave totals of this tile, and of the rows before it
  if (lane == kWave - 1) wsum[wid] = incl;
  __shared__ int64_t bsum[kOffThreads / kWave];
  if (lane == 0) bsum[wid] = before;
  __syncthreads();
  int64_t run = incl - mine;
  for (int w = 0; w < kOffThreads / kWave; ++w) {
    run += bsum[w];
    if (w < wid) run += wsum[w];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t v = v0 + 4 * t + k;
    if (v < n1) {
      const int64_t o = rp_old[v < n_old ? v : n_old];
      rp_new[v] = o + run;
      add[v] = v < n_old ? (int32_t)(rp_old[v + 1] - o) : (int32_t)(brp[v - n_old + 1] - brp[v - n_old]);
      run += c[k];
      if (v == n1 - 1) rp_new[n1] = rp_old[n_old] + run;
    }
  }
}

// Workgroups [0, new_blocks) take the new rows, the others copy the old ones.
__global__ void __launch_bounds__(kThreads) k_insert_rows(int32_t n_new, int64_t n_old, int32_t insert_root,
                                                         unsigned new_blocks, const int64_t* __restrict__ brp,
                                                         const int32_t* __restrict__ bcol,
                                                         const int32_t* __restrict__ bslot,
                                                         const float* __restrict__ bcost,
                                                         const int64_t* __restrict__ rp_old,
                                                         const int32_t* __restrict__ col_old,
                                                         const float* __restrict__ cst_old,
                                                         const int64_t* __restrict__ rp_new,
                                                         int32_t* __restrict__ col_new, float* __restrict__ cst_new,
                                                         int32_t* __restrict__ cursor, int32_t* __restrict__ add0,
                                                         const float* __restrict__ g, uint4* __restrict__ base,
                                                         InsertEdge* __restrict__ inner, int32_t* __restrict__ dcount) {
  if (blockIdx.x >= new_blocks) {
    const int64_t t = (int64_t)(blockIdx.x - new_blocks) * kThreads + threadIdx.x;
    const int64_t v = t / kCopyGW;
    const int gl = (int)(t % kCopyGW);
    if (v >= n_old) return;
    const int64_t a = rp_old[v], b = rp_old[v + 1], dst = rp_new[v];
    if (gl == 0) add0[v] = 0;
    for (int64_t j = a + gl; j < b; j += kCopyGW) {
      col_new[dst + (j - a)] = col_old[j];
      cst_new[dst + (j - a)] = cst_old[j];
    }
    return;
  }
  __shared__ int32_t listed, first;
  if (threadIdx.x == 0) listed = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t i = t / kRowGW;
  const int gl = (int)(t % kRowGW);
  const bool valid = i < n_new;
  const int32_t v = (int32_t)(n_old + i);
  const int64_t a = valid ? brp[i] : 0, b = valid ? brp[i + 1] : 0, dst = valid ? rp_new[v] : 0;
  if (valid && gl == 0) add0[v] = 0;
  uint32_t bv = 0xffffffffu, bc = 0xffffffffu, be = 0xffffffffu;
  int32_t bs = -1;
  int inside = 0;
  for (int64_t j = a + gl; j < b; j += kRowGW) {
    const int32_t s = bslot[j];
    const float c = bcost[j];
    col_new[dst + (j - a)] = s;
    cst_new[dst + (j - a)] = c;
    const int64_t pos = rp_new[s] + atomicAdd(&cursor[s], 1);
    col_new[pos] = v;
    cst_new[pos] = c;
    if (s >= n_old) {
      ++inside;
      continue;
    }
    const uint32_t u = (uint32_t)bcol[j];
    const uint32_t vb = __float_as_uint(add_rn(g[s], c)), cb = __float_as_uint(c);
    if (vb < bv || (vb == bv && (u < be || (u == be && cb < bc)))) {
      bv = vb;
      be = u;
      bc = cb;
      bs = s;
    }
  }
  // the row's best existing neighbour: (value, id) first, then the cost
  const unsigned long long k = ((unsigned long long)bv << 32) | be;
  const unsigned long long km = dpp_group_min_u64<kRowGW>(k);
  const uint32_t cm = dpp_group_min_u32<kRowGW>(k == km ? bc : 0xffffffffu);
  const int grp = (threadIdx.x & (kWave - 1)) / kRowGW;
  const unsigned long long wb = group_bits<kRowGW>(__ballot(k == km && bc == cm), grp);
  const int32_t ws = __shfl(bs, grp * kRowGW + (wb ? __ffsll((long long)wb) - 1 : 0), kWave);
  if (valid && gl == 0) base[i] = make_uint4((uint32_t)(km >> 32), (uint32_t)km, cm, (uint32_t)ws);
  // the entries inside the batch (one reservation a workgroup)
  int32_t at = inside > 0 ? atomicAdd(&listed, inside) : 0;
  __syncthreads();
  if (threadIdx.x == 0) first = listed > 0 ? atomicAdd(&dcount[0], listed) : 0;
  __syncthreads();
  if (inside == 0) return;
  at += first;
  for (int64_t j = a + gl; j < b; j += kRowGW) {
    const int32_t s = bslot[j];
    if (s < n_old) continue;
    if (at < kInsertInner) inner[at] = InsertEdge{(int32_t)i, (int32_t)(s - n_old), bcost[j]};
    ++at;
  }
}

constexpr int kPolThreads = 1024;
constexpr int kPer = kInsertBlockMax / kPolThreads;

__global__ void __launch_bounds__(kPolThreads) k_insert_policy(int32_t n_new, int64_t n_old, int32_t insert_root,
                                                              const uint4* __restrict__ base,
                                                              const InsertEdge* __restrict__ inner,
                                                              const int32_t* __restrict__ dcount,
                                                              int32_t* __restrict__ placed, float* __restrict__ g,
                                                              int32_t* __restrict__ parent,
                                                              float* __restrict__ pcost) {
  extern __shared__ uint32_t lds[];
  uint32_t* val = lds;                                   // [kInsertBlockMax] g of the new vertices (bits)
  int32_t* off = reinterpret_cast<int32_t*>(val + kInsertBlockMax);  // [kInsertBlockMax] first inner edge
  float* ec = reinterpret_cast<float*>(off + kInsertBlockMax);       // [kInsertInner]
  uint16_t* eu = reinterpret_cast<uint16_t*>(ec + kInsertInner);     // [kInsertInner]
  __shared__ int wsum[kPolThreads / kWave];
  __shared__ int moved[3];
  const int t = threadIdx.x, lane = t & (kWave - 1), wid = t / kWave;
  const int32_t E = dcount[0];
  if (E > kInsertInner) {  // too many inner edges: the host takes the level path
    if (t == 0) *placed = 0;
    return;
  }
  for (int i = t; i < kInsertBlockMax; i += kPolThreads) off[i] = 0;
  if (t < 3) moved[t] = 0;
  __syncthreads();
  for (int32_t e = t; e < E; e += kPolThreads) atomicAdd(&off[inner[e].to], 1);
  __syncthreads();
  // thread t's vertices are kPer t .. kPer t + kPer - 1: exclusive sums of the counts
  int cnt[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    cnt[k] = off[kPer * t + k];
    sum += cnt[k];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int y = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += y;
  }
  if (lane == kWave - 1) wsum[wid] = incl;
  __syncthreads();
  int run = incl - sum;
  for (int w = 0; w < wid; ++w) run += wsum[w];
  int at[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    at[k] = run;
    off[kPer * t + k] = run;
    run += cnt[k];
  }
  __syncthreads();
  for (int32_t e = t; e < E; e += kPolThreads) {
    const InsertEdge x = inner[e];
    const int p = atomicAdd(&off[x.to], 1);
    ec[p] = x.cost;
    eu[p] = (uint16_t)x.from;
  }
  uint4 b[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = kPer * t + k;
    b[k] = i < n_new ? base[i] : make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);
    if (n_old + i == insert_root) b[k].x = 0u;
    val[i] = b[k].x < 0x7f800000u ? b[k].x : 0x7f800000u;
  }
  __syncthreads();
  // the minimum over the lower neighbours by (value, id, cost), the existing ones' first
  auto best = [&](int k) {
    uint4 m = b[k];
    if (n_old + kPer * t + k == insert_root) return m;
    for (int p = at[k]; p < at[k] + cnt[k]; ++p) {
      const float c = ec[p];
      const uint32_t u = (uint32_t)n_old + eu[p];
      const uint32_t vb =
          __float_as_uint(add_rn(__uint_as_float(__hip_atomic_load(&val[eu[p]], __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_WORKGROUP)), c));
      const uint32_t cb = __float_as_uint(c);
      if (vb < m.x || (vb == m.x && (u < m.y || (u == m.y && cb < m.z)))) m = make_uint4(vb, u, cb, u);
    }
    return m;
  };
  for (int round = 0;;) {
    int ch = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (cnt[k] == 0) continue;
      const uint4 m = best(k);
      const uint32_t now = m.x < 0x7f800000u ? m.x : 0x7f800000u;
      const int i = kPer * t + k;
      if (now != __hip_atomic_load(&val[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
        __hip_atomic_store(&val[i], now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        ch = 1;
      }
    }
    // one barrier a round: the three flags take turns
    if (ch) __hip_atomic_store(&moved[round], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const int next = round == 2 ? 0 : round + 1, after = next == 2 ? 0 : next + 1;
    __syncthreads();
    const int any = __hip_atomic_load(&moved[round], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (t == 0) __hip_atomic_store(&moved[after], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    round = next;
    if (!any) break;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = kPer * t + k;
    if (i >= n_new) continue;
    const uint4 m = best(k);
    const bool root = n_old + i == insert_root, found = !root && m.x < 0x7f800000u;
    g[n_old + i] = root ? 0.0f : (found ? __uint_as_float(m.x) : pos_inf());
    parent[n_old + i] = found ? (int32_t)m.w : -1;
    pcost[n_old + i] = found ? __uint_as_float(m.z) : 0.0f;
  }
  if (t == 0) *placed = n_new;
}

}  // namespace

hipError_t launch_insert_small(const InsertArgs& a, hipStream_t s) {
  const int64_t n1 = a.n_old + a.n_new;
  hipLaunchKernelGGL(k_insert_prepare, dim3(blocks_for((int64_t)a.n_new * kRowGW)), dim3(kThreads), 0, s, a.n_new,
                     a.n_old, a.brp, a.bcol, a.slot_of, a.ext_of, a.bslot, a.add0, a.dcount);
  hipLaunchKernelGGL(k_insert_offsets, dim3(blocks_for(n1, kOffTile)), dim3(kOffThreads), 0, s, n1, a.n_old, a.rp_old,
                     a.brp, a.add0, a.add, a.rp_new);
  uint4* base = reinterpret_cast<uint4*>(a.scratch);
  InsertEdge* inner = reinterpret_cast<InsertEdge*>(base + kInsertBlockMax);
  const unsigned nb = blocks_for((int64_t)a.n_new * kRowGW);
  const unsigned ob = a.n_old > 0 ? blocks_for(a.n_old * kCopyGW) : 0;
  hipLaunchKernelGGL(k_insert_rows, dim3(nb + ob), dim3(kThreads), 0, s, a.n_new, a.n_old, a.insert_root, nb, a.brp,
                     a.bcol, a.bslot, a.bcost, a.rp_old, a.col_old, a.cst_old, a.rp_new, a.col_new, a.cst_new, a.add,
                     a.add0, a.g, base, inner, a.dcount);
  const size_t lds = 8 * (size_t)kInsertBlockMax + 6 * (size_t)kInsertInner;
  const hipError_t e = hipFuncSetAttribute((const void*)k_insert_policy, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_insert_policy, dim3(1), dim3(kPolThreads), lds, s, a.n_new, a.n_old, a.insert_root, base, inner,
                     a.dcount, a.placed, a.g, a.parent, a.pcost);
  return hipGetLastError();
}

}  // namespace pirrt
