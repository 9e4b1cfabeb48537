// Replan of a mid-sized graph in one launch (Alg. 2; Sec. IV-B, IV-C): a few workgroups
// that stay resident for the whole loop, with one grid barrier per iteration.
//
// At a few thousand vertices the multi-kernel loop is five short launches an iteration
// (about 30 us, whatever the work); the bytes of an iteration would take a tenth of one.
// Here every workgroup keeps the whole vertex state (g, parent, parent-edge cost: 10
// bytes a vertex) in LDS and evaluates the whole tree by itself, so g never crosses a
// workgroup; each owns a range of rows, and all that an iteration exchanges are the
// parents its rows switched:
//
//   Evaluate : thread t repeats g(v) = fl(g(parent) + cost) for vertices t, t + 1024, ...
//              until a whole round changes nothing.  On a tree that fixed point is the
//              root-to-leaf fold, bit for bit, from any starting values; the previous g
//              makes the rounds follow the depth of what changed, not of the tree (three
//              or four rounds an iteration).  (The host says whether the stored policy is
//              known to be a tree: otherwise the first Evaluate starts from +inf, where a
//              cycle of parents stays.  Improve makes no new cycles.)
//   P        : the sign bit of g in LDS, set where fl(g + h) < G, G = g(goal) or +inf.
//   rows     : a group of 8 lanes per owned row reads it once for both steps: the row is
//              in the domain if its vertex or a neighbour is in P (narrowed domain: if a
//              neighbour's offer passes), and the lexicographic minimum of (g(u) + c,
//              caller id, c) is Improve's.  g is only read (Jacobi step).
//   exchange : each workgroup lists its switches in a region of its own; one 64-bit word
//              per iteration counts arrivals and adds up the switches, so the workgroups
//              that wait for it also learn whether to stop; then all read all lists.
//
// The lists have two buffers: a workgroup can be one barrier ahead of another at most, and
// then writes the buffer that the slower one has finished reading.  What crosses
// workgroups inside the launch -- the lists and the words -- is written and read by
// device-scope atomics only, which bypass the L1 and the XCDs' L2s, and every wave waits
// for its stores before its workgroup arrives.  So no cache is written back or
// invalidated, and the adjacency stays in them.
//
// Results: every workgroup has every vertex, so each writes a range of caller ids to the
// caller's arrays, and the one that is done last the counters to host memory; the set-up kernel
// before brings the heuristic into storage order and checks it.  Two launches and one wait a
// call; a check, a gather, a copy-out kernel, three copies and a wait more took 20 us more at
// 2,002 2D vertices.
//
// Residency: nothing is written before all workgroups have met at a gate.  A workgroup
// that waits there too long (others hold the chip) closes the gate; then every workgroup
// leaves, the problem stays active and the host runs the multi-kernel loop.  Past the gate
// all are resident, so every later wait ends.  The wait is far longer than a Replan: workgroups
// that others hold up get their turn within a few Replans' time, and two calls of 15,000 vertices
// fill the chip.  Calls from 1, 2, 3, 4 and 8 threads at once, a handle of that size and a stream
// each, took 0.85, 1.26, 1.61, 1.67 and 2.66 ms on average (the multi-kernel loop 1.18, 1.74, 1.31,
// 2.34 and 2.43), none more than 6.5; beside another stream's element-wise kernels or matrix
// products, back to back, 1.62 and 4.4 ms (3.8 and 5.1).
#include "internal.h"

namespace pirrt {

namespace {

constexpr int kResThreads = 1024;
constexpr int kGW = 8;                          // lanes per row
constexpr int kQ = 2;                           // quads of entries per lane in flight
constexpr int kResRows = kResThreads / kGW;     // rows of one pass
constexpr int kTogether = 4;                    // vertices of a thread evaluated together
constexpr uint32_t kGatePolls = 1u << 14;       // about ten milliseconds
constexpr uint32_t kBarrierPolls = 1u << 24;    // never reached: all workgroups are resident

__device__ __forceinline__ unsigned long long load_agent(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(unsigned long long* p, unsigned long long x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All workgroups meet before anything is written: true once every one is resident, false
// (in all of them) when one gave up waiting.
__device__ __forceinline__ bool gate(ResidentSync* sy, uint32_t W) {
  __shared__ int open;
  if (threadIdx.x == 0) {
    uint32_t st = 0;  // 0 waiting, 1 open, 2 closed
    if (__hip_atomic_fetch_add(&sy->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == W - 1) {
      uint32_t want = 0;
      st = __hip_atomic_compare_exchange_strong(&sy->gate, &want, 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT)
               ? 1u
               : want;
    } else {
      for (uint32_t i = 0; i < kGatePolls; ++i) {
        st = __hip_atomic_load(&sy->gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (st) break;
        __builtin_amdgcn_s_sleep(8);
      }
      if (!st) {
        uint32_t want = 0;
        st = __hip_atomic_compare_exchange_strong(&sy->gate, &want, 2u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT)
                 ? 2u
                 : want;
      }
    }
    open = st == 1u;
  }
  __syncthreads();
  return open != 0;
}

// Grid barrier of iteration `it` that also sums `mine` over the workgroups (the value in
// thread 0); -1 if the wait failed.  The words rotate: word it + 2 is cleared here, when
// nobody polls it any more (all have passed barrier it - 1) and nobody uses it yet.
__device__ __forceinline__ int grid_sum(ResidentSync* sy, uint32_t W, int it, int mine) {
  __shared__ int sum;
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // this wave's stores are done
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long* w = &sy->word[it % 4][0];
    unsigned long long x =
        __hip_atomic_fetch_add(w, ((unsigned long long)(uint32_t)mine << 32) | 1ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT) +
        (((unsigned long long)(uint32_t)mine << 32) | 1ull);
    uint32_t i = 0;
    while ((uint32_t)x != W && i < kBarrierPolls) {
      x = load_agent(w);
      ++i;
    }
    asm volatile("" ::: "memory");
    sum = (uint32_t)x == W ? (int)(x >> 32) : -1;
    if (blockIdx.x == 0) store_agent(&sy->word[(it + 2) % 4][0], 0ull);
  }
  __syncthreads();
  return sum;
}

// K: vertices per thread.  The first 64 entries of a group's row stay in registers.  Slots
// are kept as 16-bit byte offsets into g (4 v).
template <int K, bool kLook>
__global__ void __launch_bounds__(kResThreads) k_replan_resident(ResidentArgs a) {
  constexpr int N = K * kResThreads;
  constexpr uint32_t kNone = N * 4;  // an entry past the end of a row: a slot with g = +inf
  extern __shared__ float g[];       // [N + 64]; the sign bit: the vertex is in P
  float* pc = g + N + 64;            // [N] parent-edge costs
  // [N] parents; the root and vertices without one keep their value: themselves, cost 0
  uint16_t* par = reinterpret_cast<uint16_t*>(pc + N);
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const uint32_t W = gridDim.x;
  if (a.ps->active == 0) return;  // the heuristic was refused
  if (!gate(a.sync, W)) return;
  const int32_t n = a.n, R = a.rows;
  const int32_t first = (int32_t)blockIdx.x * R;
  const int32_t own = first >= n ? 0 : (first + R < n ? R : n - first);
  const int32_t root = a.ps->root, goal = a.ps->goal, cap = a.ps->cap;
  // (a few vertices' loads in flight together, none behind the value of another)
  float hv[K];
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += kTogether) {
    int32_t p[kTogether];
    float c[kTogether], old[kTogether];
#pragma unroll
    for (int j = 0; j < kTogether && k0 + j < K; ++j) {
      const int32_t v = t + (k0 + j) * kResThreads, i = v < n ? v : n - 1;
      p[j] = a.parent[i];
      c[j] = a.pcost[i];
      old[j] = a.g[i];
      hv[k0 + j] = a.h ? a.h[i] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < kTogether && k0 + j < K; ++j) {
      const int32_t v = t + (k0 + j) * kResThreads;
      const bool has = v < n && v != root && p[j] >= 0;
      par[v] = (uint16_t)(4 * (has ? p[j] : v));
      pc[v] = has ? c[j] : 0.0f;
      g[v] = v == root ? 0.0f : (has && a.tree ? old[j] : pos_inf());
    }
  }
  if (t < 64) g[N + t] = pos_inf();
  __shared__ int moved[3];  // whether an Evaluate round changed something; the rounds take turns
  if (t < 3) moved[t] = 0;
  // the group's row
  const int gl = t % kGW, grp = lane / kGW;
  const int4* col4 = reinterpret_cast<const int4*>(a.col);
  const float4* cst4 = reinterpret_cast<const float4*>(a.cst);
  const bool valid = t / kGW < own;
  const int32_t x = first + (valid ? t / kGW : 0);
  const uint32_t ra = valid ? (uint32_t)a.rp[x] : 0u, rb = valid ? (uint32_t)a.rp[x + 1] : 0u;
  const float hx = kLook && a.h && valid ? a.h[x] : 0.0f;
  uint32_t eu[2 * kQ];  // the entries' slots, two a register
  float ec[4 * kQ];     // and costs
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const uint32_t k = (ra >> 2) + gl + q * kGW;
    const bool live = 4 * k < rb;
    const int4 w = live ? col4[k] : make_int4(0, 0, 0, 0);
    const float4 c = live ? cst4[k] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const int32_t u[4] = {w.x, w.y, w.z, w.w};
    const float cc[4] = {c.x, c.y, c.z, c.w};
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = 4 * k + e >= ra && 4 * k + e < rb ? 4u * (uint32_t)u[e] : kNone;
      ec[4 * q + e] = cc[e];
    }
    eu[2 * q] = o[0] | (o[1] << 16);
    eu[2 * q + 1] = o[2] | (o[3] << 16);
  }
  __syncthreads();

  auto at = [&](uint32_t offset) {  // g at a byte offset, with its sign bit
    float* p = static_cast<float*>(__builtin_assume_aligned(reinterpret_cast<char*>(g) + offset, 4));
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  int round = 0;
  auto evaluate = [&]() {
    uint32_t u[(K + 1) / 2];
    float c[K], own_g[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int v = t + k * kResThreads;
      u[k / 2] = (k & 1) ? u[k / 2] | ((uint32_t)par[v] << 16) : par[v];
      c[k] = pc[v];
      own_g[k] = fabsf(at(4 * v));
    }
    for (;;) {
      int ch = 0;
      // a few vertices at a time: their reads are in flight together, and the next ones see
      // what they wrote (parents mostly have lower slots)
#pragma unroll
      for (int k0 = 0; k0 < K; k0 += kTogether) {
        float up[kTogether];
#pragma unroll
        for (int j = 0; j < kTogether && k0 + j < K; ++j)
          up[j] = fabsf(at(((k0 + j) & 1) ? u[(k0 + j) / 2] >> 16 : u[(k0 + j) / 2] & 0xffffu));
#pragma unroll
        for (int j = 0; j < kTogether && k0 + j < K; ++j) {
          const float now = add_rn(up[j], c[k0 + j]);
          if (now != own_g[k0 + j]) {  // (never NaN: values are >= 0, costs finite)
            own_g[k0 + j] = now;
            __hip_atomic_store(&g[t + (k0 + j) * kResThreads], now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            ch = 1;
          }
        }
      }
      // one barrier a round: this round's flag is set before it and read after it, and the
      // flag of the round after next was last read before it
      if (ch) __hip_atomic_store(&moved[round], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      const int next = round == 2 ? 0 : round + 1, after = next == 2 ? 0 : next + 1;
      __syncthreads();
      const int any = __hip_atomic_load(&moved[round], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (t == 0) __hip_atomic_store(&moved[after], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      round = next;
      if (!any) break;  // a whole round changed nothing
    }
  };

  evaluate();
  int32_t iters = 0, status = 0;
  long long chg_sum = 0;
  int sum_p = 0, sum_d = 0;  // per thread: at most one an iteration
  unsigned long long sum_e = 0, sum_pe = 0;
  for (;;) {
    const float G = a.prune ? fabsf(at(4 * goal)) : pos_inf();
    __shared__ int switched;
    if (t == 0) switched = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int v = t + k * kResThreads;
      const float old = g[v], val = fabsf(old);
      const float now = add_rn(val, hv[k]) < G ? -val : val;
      if (__float_as_uint(now) != __float_as_uint(old)) g[v] = now;
    }
    __syncthreads();
    unsigned long long* lists = a.lists + (int64_t)(iters & 1) * W * (R + 1);
    unsigned long long* list = lists + (int64_t)blockIdx.x * (R + 1);
    const float gx = at(4 * x);
    // The least offer g(u) + c of the row (as bits: they are >= 0), and whether a
    // neighbour in P puts x into the domain.
    uint32_t best = 0x7f800000u;
    bool near = false;
    uint32_t any = 0;
    float val[4 * kQ];
#pragma unroll
    for (int e = 0; e < 4 * kQ; ++e) {
      const float gu = at((e & 1) ? eu[e / 2] >> 16 : eu[e / 2] & 0xffffu);
      val[e] = add_rn(fabsf(gu), ec[e]);
      if (kLook)
        near = near || (__float_as_uint(gu) >> 31 && add_rn(val[e], hx) < G);
      else
        any |= __float_as_uint(gu);
      best = __float_as_uint(val[e]) < best ? __float_as_uint(val[e]) : best;
    }
    // entries past the first 64 of the row, from memory
    auto tail = [&](auto&& each) {
      for (uint32_t k = (ra >> 2) + gl + kQ * kGW; 4 * k < rb; k += kGW) {
        const int4 w = col4[k];
        const float4 c = cst4[k];
        const int32_t u[4] = {w.x, w.y, w.z, w.w};
        const float cc[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (4 * k + e < rb) each(4u * (uint32_t)u[e], cc[e]);
      }
    };
    tail([&](uint32_t o, float c) {
      const float gu = at(o), offer = add_rn(fabsf(gu), c);
      if (kLook)
        near = near || (__float_as_uint(gu) >> 31 && add_rn(offer, hx) < G);
      else
        any |= __float_as_uint(gu);
      best = __float_as_uint(offer) < best ? __float_as_uint(offer) : best;
    });
    if (!kLook) near = any >> 31;
    const bool px = __float_as_uint(gx) >> 31;
    const bool in = valid && x != root && (px || group_bits<kGW>(__ballot(near), grp) != 0ull);
    const uint32_t mv = dpp_group_min_u32<kGW>(best);
    const bool sw = in && __uint_as_float(mv) < fabsf(gx);
    if (gl == 0 && valid) {
      if (px) {
        sum_p += 1;
        sum_pe += rb - ra;
      }
      if (in) {
        sum_d += 1;
        sum_e += rb - ra;
      }
    }
    // Which neighbour it is, in waves where a row switches: the lowest (caller id, cost)
    // among the offers equal to the minimum; caller ids are fetched only for real ties.
    if (__ballot(sw) != 0ull) {
      int32_t bo = -1;
      uint32_t bc = 0xffffffffu;
      auto take = [&](uint32_t o, float c, float offer) {
        if (__float_as_uint(offer) != mv) return;
        const uint32_t cb = __float_as_uint(c);
        if (bo >= 0) {
          const int32_t e1 = a.ext_of[o / 4], e0 = a.ext_of[bo / 4];
          if (e1 > e0 || (e1 == e0 && cb >= bc)) return;
        }
        bo = (int32_t)o;
        bc = cb;
      };
      if (sw) {
#pragma unroll
        for (int e = 0; e < 4 * kQ; ++e)
          take((e & 1) ? eu[e / 2] >> 16 : eu[e / 2] & 0xffffu, ec[e], val[e]);
        tail([&](uint32_t o, float c) { take(o, c, add_rn(fabsf(at(o)), c)); });
      }
      const bool tied = bo >= 0;
      const bool multi = __popcll(group_bits<kGW>(__ballot(tied), grp)) > 1;
      const uint32_t e = tied ? (multi ? (uint32_t)a.ext_of[bo / 4] : 0u) : 0xffffffffu;
      const unsigned long long k2 = ((unsigned long long)e << 32) | (tied ? bc : 0xffffffffu);
      const unsigned long long m2 = dpp_group_min_u64<kGW>(k2);
      const unsigned long long wb = group_bits<kGW>(__ballot(tied && k2 == m2), grp);
      if (sw && gl == (wb ? __ffsll((long long)wb) - 1 : 0))
        store_agent(&list[1 + atomicAdd(&switched, 1)],
                    ((unsigned long long)bc << 32) | ((uint32_t)bo << 16) | (4u * (uint32_t)x));
    }
    __syncthreads();
    if (t == 0) store_agent(&list[0], (unsigned long long)(uint32_t)switched);
    const int changed = grid_sum(a.sync, W, iters, switched);
    ++iters;
    if (changed < 0) {  // cannot happen (see the top); the host reports it
      status = 2;
      break;
    }
    chg_sum += changed;
    if (changed == 0) break;
    // 32 threads per list, all of a thread's lists in flight together; the first entries
    // come with the list's length
    constexpr int kLists = kResidentGroups / (kResThreads / 32);
    unsigned long long entry[kLists];
#pragma unroll
    for (int j = 0; j < kLists; ++j) {
      const uint32_t w = t / 32 + j * (kResThreads / 32);
      entry[j] = w < W && t % 32 <= R ? load_agent(&lists[(int64_t)w * (R + 1) + t % 32]) : 0ull;
    }
#pragma unroll
    for (int j = 0; j < kLists; ++j) {
      const uint32_t w = t / 32 + j * (kResThreads / 32);
      const uint32_t len = (uint32_t)__shfl((int)(uint32_t)entry[j], 0, 32);
      for (uint32_t i = t % 32; i <= len; i += 32) {
        if (i >= 32) entry[j] = load_agent(&lists[(int64_t)w * (R + 1) + i]);
        if (i == 0) continue;
        const uint32_t v = ((uint32_t)entry[j] & 0xffffu) / 4;
        par[v] = (uint16_t)((uint32_t)entry[j] >> 16);
        pc[v] = __uint_as_float((uint32_t)(entry[j] >> 32));
      }
    }
    __syncthreads();
    evaluate();
    if (iters >= cap) {
      status = 1;
      break;
    }
  }
  // results: the owned rows' policy and g, the counters into the problem's state
  for (int i = t; i < own; i += kResThreads) {
    const int32_t v = first + i;
    a.g[v] = fabsf(g[v]);
    if (par[v] != 4 * v) {  // parents switch but never go: the others' entries stay as stored
      a.parent[v] = par[v] / 4;
      a.pcost[v] = pc[v];
    }
  }
  // the caller's copy: every workgroup has every vertex, so it takes caller ids in a row
  for (int i = t; i < own; i += kResThreads) {
    const int32_t e = first + i, v = a.slot_of[e];
    if (a.g_out) a.g_out[e] = fabsf(g[v]);
    if (a.parent_out) a.parent_out[e] = par[v] != 4 * v ? a.ext_of[par[v] / 4] : -1;
  }
  // The counters, one addition each a workgroup: with one a wave, some 6,000 to one line, a
  // Replan of one iteration took 105 us at 12,000 vertices and 132 at 15,000 (the loop of
  // launches 98 and 100), now 51 and 61.
  __shared__ unsigned long long sums[4];
  if (t < 4) sums[t] = 0ull;
  __syncthreads();
  unsigned long long sp = (unsigned)sum_p, sd = (unsigned)sum_d;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    sp += __shfl_xor(sp, o, kWave);
    sd += __shfl_xor(sd, o, kWave);
    sum_e += __shfl_xor(sum_e, o, kWave);
    sum_pe += __shfl_xor(sum_pe, o, kWave);
  }
  if (lane == 0) {
    atomicAdd(&sums[0], sp);
    atomicAdd(&sums[1], sd);
    atomicAdd(&sums[2], sum_e);
    atomicAdd(&sums[3], sum_pe);
  }
  __syncthreads();
  if (t != 0) return;
  atomicAdd(&a.ps->sum_P, sums[0]);
  atomicAdd(&a.ps->sum_D, sums[1]);
  atomicAdd(&a.ps->edges, sums[2]);
  atomicAdd(&a.ps->mark_edges, sums[3]);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // they are in
  // the workgroup that is done last has all sums and reports them (all agree on the rest)
  if (__hip_atomic_fetch_add(&a.sync->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != W - 1) return;
  ProblemState q = {};
  q.root = root;
  q.goal = goal;
  q.iterations = iters;
  q.status = status;
  q.cap = cap;
  q.edges = load_agent(&a.ps->edges);
  q.sum_P = load_agent(&a.ps->sum_P);
  q.sum_D = load_agent(&a.ps->sum_D);
  q.mark_edges = load_agent(&a.ps->mark_edges);
  q.changed_total = (unsigned long long)chg_sum;
  *a.ps = q;
  *a.report = q;
}

template <int K>
hipError_t launch_k(const ResidentArgs& a, int W, hipStream_t s) {
  constexpr int N = K * kResThreads;
  static_assert(4 * N < 65536 && 10 * N + 256 <= 160 * 1024 - 512, "16-bit offsets; LDS of a workgroup");
  const size_t lds = 10 * (size_t)N + 256;
  const void* f = a.lookahead ? (const void*)k_replan_resident<K, true> : (const void*)k_replan_resident<K, false>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if (a.lookahead)
    hipLaunchKernelGGL((k_replan_resident<K, true>), dim3(W), dim3(kResThreads), lds, s, a);
  else
    hipLaunchKernelGGL((k_replan_resident<K, false>), dim3(W), dim3(kResThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_replan_resident(ResidentArgs a, hipStream_t s) {
  static_assert(kResidentMax <= 15 * kResThreads && kResidentMax <= kResRows * kResidentGroups, "sizes covered");
  const int W = (a.n + kResRows - 1) / kResRows;  // one row a group
  a.rows = (a.n + W - 1) / W;
  // A thread's vertices, by steps: those it has no use for are evaluated all the same (10,000 2D
  // vertices took 140 us with 15 to a thread, 117 with 10; 5,000 95 with 8, 88 with 5).
  switch ((a.n + kResThreads - 1) / kResThreads) {
    case 1: return launch_k<1>(a, W, s);
    case 2: return launch_k<2>(a, W, s);
    case 3: return launch_k<3>(a, W, s);
    case 4: return launch_k<4>(a, W, s);
    case 5: return launch_k<5>(a, W, s);
    case 6: return launch_k<6>(a, W, s);
    case 7:
    case 8: return launch_k<8>(a, W, s);
    case 9:
    case 10: return launch_k<10>(a, W, s);
    case 11:
    case 12: return launch_k<12>(a, W, s);
  }
  return launch_k<15>(a, W, s);
}

}  // namespace pirrt
