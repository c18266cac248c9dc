// levels.hip -- layering of the ghost dependency graph (Sec. 3.2) and the
// canonical order (level, linear index).
//
// The level of a ghost is the longest dependency path from a ghost that
// reads no ghost.  Three forms, all with that result:
//   k_levels_pull            one workgroup per instance of at most kPullMax
//                            ghosts, every level in LDS; cycles found on the
//                            way
//   k_levels_flow (+ _scan)  one large 3D instance on the whole GPU
//   k_levels_fast, k_levels  one workgroup per instance pushing levels along
//                            reverse edges (a CSR list built by grid-wide
//                            kernels for them alone): batches with larger
//                            instances, and the graphs the others leave
//                            (deeper than their tables, a cycle in an
//                            instance too large for k_levels_pull)
//
// k_levels, the most general: each ghost (or coupled unit) holds a byte
// counter of unplaced ghosts it reads, packed four to a word and kept in LDS
// when the instance fits.  Level k is formed from the dependants of level
// k-1 whose counter drops to zero: they set their bit in a bitmap over the
// linear ghost order, and one workgroup scan over the bitmap words emits them
// in linear-index order with their canonical positions.  The work is
// O(ghosts + edges) plus one bitmap scan per level, independent of the order
// threads run in.  If a level comes out empty while ghosts remain, the
// remaining ghosts hold cycles: their strongly connected groups (from the
// transitive closure of the remaining graph) become coupled units, and the
// layering restarts with each unit as one node, so a unit sits one level
// above the deepest level it needs.
#include <hip/hip_runtime.h>

#include <mutex>

#include "gcr_impl.hpp"

namespace gcr {

__device__ __forceinline__ int64_t find_sorted(const int32_t* a, int64_t lo, int64_t hi, int v) {
  while (lo < hi) {
    int64_t mid = (lo + hi) >> 1;
    int x = a[mid];
    if (x == v) return mid;
    if (x < v) lo = mid + 1; else hi = mid;
  }
  return -1;
}

// byte counters packed four per 32-bit word; a counter never goes below
// zero (one decrement per counted edge) and never exceeds 8 * 7, so no carry
// or borrow crosses into a neighbour
__device__ __forceinline__ void cnt_add(uint32_t* c, int i, uint32_t v) {
  atomicAdd(&c[i >> 2], v << ((i & 3) * 8));
}
__device__ __forceinline__ uint32_t cnt_dec(uint32_t* c, int i) {
  const uint32_t old = atomicSub(&c[i >> 2], 1u << ((i & 3) * 8));
  return (old >> ((i & 3) * 8)) & 0xffu;
}
__device__ __forceinline__ uint32_t cnt_get(const uint32_t* c, int i) {
  return (c[i >> 2] >> ((i & 3) * 8)) & 0xffu;
}

// ---------------------------------------------------------------------------
// Layering of one large instance by the whole GPU, in two launches.
//
// k_levels_flow: a thread holds up to kFlowJ ghosts and polls the levels of
// the ghosts they read (agent scope, the stores and loads go past the XCDs'
// own caches); a ghost whose reads all have a level takes 1 + the highest at
// once.  No round, barrier or list: a level costs one store-to-load trip
// across the chip (about 0.5 us, measured on a chain of 95 levels), where a
// grid barrier a level cost 30-40.
// Reads that have a level are not polled again.  Waves wait only for
// ghosts of the same launch; its at most kFlowGrid workgroups (half of what
// the chip holds) are resident together unless other work fills it.  What it
// does not finish it leaves with info.layered = 0 to the one-workgroup
// layerings: an instance with a cycle, or one starved of its workgroups.
//   - Two ghosts that read each other, the most common cycle by far, are
//     seen as the reads are loaded (the corner is the same for both), and
//     stop every wave at its next look.  Spheres are spared the search: a
//     read leads away from the centre along every axis, so |x - c|_1 grows
//     along a chain, which never closes.
//   - A wave that placed no ghost of its own for kFlowTicks, nor saw a
//     workgroup finish, stops every wave too (a chain of kWideLevels levels
//     takes a third of that), so every wave ends.
// The tiles' counts per level follow.
//
// k_levels_scan: the counts scanned over the tiles of each level, level
// offsets, results.  k_finalize adds each ghost's rank in its tile: the
// stable counting sort of the canonical order.
//
// Bound by the chain of levels and the polls of the ghosts that wait (HBM
// round trips).  512^3 sphere, 74,000 ghosts: 27 us for both against 581 for
// rounds with a grid barrier; 256^3 with a second layer (36,000): 26 against
// 191 for one workgroup in LDS.
constexpr int kFlowJ = 4, kFlowGrid = 1024;
// Polls between two looks at the launch's state: often where a pair may have
// stopped it (64^3 body with cycles: 52 us for both layerings, and 770 more
// when waves only gave up in their own time), less so with more than
// kFlowLookTiles tiles and seldom on a sphere, as every look reads one address
// (sphere of 640^3: 38 us with the first, 34 with the last).
constexpr int kFlowLook = 16, kFlowLookMany = 64, kFlowLookSphere = 256, kFlowLookTiles = 128;
constexpr int64_t kFlowTicks = 20000;   // 200 us of the 100 MHz clock

__device__ __forceinline__ int flow_get(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void flow_put(int32_t* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether a wave that waits may go on.  state: workgroups finished, ghosts
// placed, and whether to stop, of the launch.
struct FlowWait {
  const int look;
  int polls = 0, seen = -1;
  bool moved_since = false;
  int64_t since = 0;
  __device__ __forceinline__ bool go_on(bool moved, int32_t* state) {
    moved_since = moved_since || __ballot(moved) != 0ull;
    if (++polls < look) return true;
    polls = 0;
    // (one answer for the wave)
    const int done = __builtin_amdgcn_readfirstlane(flow_get(state));
    if (__builtin_amdgcn_readfirstlane(flow_get(state + 2)) != 0) return false;
    const int64_t now = wall_clock64();
    if (moved_since || done != seen) {
      moved_since = false;
      seen = done;
      since = now;
    } else if (now - since > kFlowTicks) {
      flow_put(state + 2, 1);
      return false;
    }
    return true;
  }
};

__global__ __launch_bounds__(256) void k_levels_flow(LevelsArgs L) {
  __shared__ int s_hist[kWideLevels];
  __shared__ int s_placed;
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t lo = L.g_off[0];
  const int n = (int)(L.g_off[1] - lo);
  const int ntiles = (n + 255) >> 8, G = (int)gridDim.x;
  const int np = (1 << L.insts[0].g.dim) - 1;
  const bool pairs = L.insts[0].s.kind != kSphere;
  const int look = !pairs ? kFlowLookSphere : ntiles <= kFlowLookTiles ? kFlowLook : kFlowLookMany;
  const int32_t* __restrict__ deps = L.deps + lo;
  int32_t* lev = L.lev + lo;
  if (tid == 0) s_placed = 0;
  __syncthreads();
  int placed = 0;
  if (ntiles <= kFlowJ * G) {
    // the reads without a level, in registers (-1: none, or placed)
    int32_t d[kFlowJ][7];
    int top[kFlowJ];
    uint32_t pend = 0;
#pragma unroll
    for (int j = 0; j < kFlowJ; ++j) {
      const int e = ((int)blockIdx.x + j * G) * 256 + tid;
      top[j] = 0;
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        d[j][q] = -1;
        if (e < n && q < np) {
          const int32_t v = deps[(int64_t)q * L.cap + e];
          if (v >= 0) d[j][q] = (int32_t)(v - lo);
        }
      }
      if (e < n) {
        pend |= 1u << j;
        L.blk_idx[lo + e] = -1;
      }
    }
    if (pairs) {
      bool met = false;
#pragma unroll
      for (int j = 0; j < kFlowJ; ++j)
#pragma unroll
        for (int q = 0; q < 7; ++q)
          if (d[j][q] >= 0)
            met = met || deps[(int64_t)q * L.cap + d[j][q]] - lo == ((int)blockIdx.x + j * G) * 256 + tid;
      if (met) flow_put(L.flow + 2, 1);
    }
    FlowWait W{look};
    while (__ballot(pend != 0) != 0ull) {
      bool moved = false;
#pragma unroll
      for (int j = 0; j < kFlowJ; ++j) {
        if (!((pend >> j) & 1u)) continue;
        int v[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) v[q] = d[j][q] >= 0 ? flow_get(lev + d[j][q]) : 0;
        bool open = false;
#pragma unroll
        for (int q = 0; q < 7; ++q) {
          if (v[q]) d[j][q] = -1;
          top[j] = max(top[j], v[q]);
          open = open || d[j][q] >= 0;
        }
        if (open) continue;
        flow_put(lev + ((int)blockIdx.x + j * G) * 256 + tid, top[j] + 1);
        pend &= ~(1u << j);
        ++placed;
        moved = true;
      }
      if (!W.go_on(moved, L.flow)) break;
    }
  } else {
    // more ghosts than the registers hold: their reads from memory, every time
    for (int t = blockIdx.x; t < ntiles; t += G) {
      const int e = t * 256 + tid;
      if (e >= n) continue;
      L.blk_idx[lo + e] = -1;
      for (int q = 0; q < np && pairs; ++q) {
        const int32_t v = deps[(int64_t)q * L.cap + e];
        if (v >= 0 && deps[(int64_t)q * L.cap + (v - lo)] - lo == e) flow_put(L.flow + 2, 1);
      }
    }
    FlowWait W{look};
    for (bool open = true; __ballot(open) != 0ull;) {
      bool moved = false;
      open = false;
      for (int t = blockIdx.x; t < ntiles; t += G) {
        const int e = t * 256 + tid;
        if (e >= n || flow_get(lev + e) != 0) continue;
        int top = 0;
        bool ready = true;
        for (int q = 0; q < np; ++q) {
          const int32_t v = deps[(int64_t)q * L.cap + e];
          if (v < 0) continue;
          const int l = flow_get(lev + (v - lo));
          top = max(top, l);
          ready = ready && l != 0;
        }
        if (ready) {
          flow_put(lev + e, top + 1);
          ++placed;
          moved = true;
        } else {
          open = true;
        }
      }
      if (!W.go_on(moved, L.flow)) break;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) placed += __shfl_xor(placed, o);
  if (lane == 0 && placed) atomicAdd(&s_placed, placed);
  __syncthreads();
  // a finished (or weary) workgroup: one more for those that wait, and its
  // ghosts, by one atomic (about 20 ns each; with one a wave the 512^3
  // sphere's pass took 31 us instead of 19)
  if (tid == 0 && s_placed)
    atomicAdd(reinterpret_cast<unsigned long long*>(L.flow),
              1ull | (unsigned long long)s_placed << 32);
  // the tiles' counts per level (levels beyond the table: dropped here, and
  // the instance is left to the others, as its counts fall short)
  for (int t = blockIdx.x; t < ntiles; t += G) {
    __syncthreads();
    if (tid < kWideLevels) s_hist[tid] = 0;
    __syncthreads();
    const int e = t * 256 + tid;
    const int l = e < n ? flow_get(lev + e) : 0;
    if (l >= 1 && l <= kWideLevels) atomicAdd(&s_hist[l - 1], 1);
    __syncthreads();
    if (tid < kWideLevels) L.hist[(int64_t)t * kWideLevels + tid] = s_hist[tid];
  }
}

__global__ __launch_bounds__(1024) void k_levels_scan(LevelsArgs L) {
  constexpr int kSeg8 = 1024 / kWideLevels, kU = 20;
  static_assert(kWideLevels == 128, "levels on 128 threads");
  __shared__ int s_sum[kSeg8][kWideLevels];
  __shared__ int s_off[kWideLevels + 1];
  __shared__ int64_t sh[17];
  const int tid = threadIdx.x, l = tid % kWideLevels, seg = tid / kWideLevels;
  const int n = (int)(L.g_off[1] - L.g_off[0]);
  const int ntiles = (n + 255) >> 8;
  const bool whole = L.flow[1] == n;
  const int per = (ntiles + kSeg8 - 1) / kSeg8, t0 = seg * per, t1 = min(ntiles, t0 + per);
  int32_t* h = L.hist + l;
  int sum = 0;
  for (int t = t0; t < t1; t += kU) {
    int v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = t + u < t1 ? h[(int64_t)(t + u) * kWideLevels] : 0;
#pragma unroll
    for (int u = 0; u < kU; ++u) sum += v[u];
  }
  s_sum[seg][l] = sum;
  __syncthreads();
  int tot = 0;
  if (seg == 0)
    for (int q = 0; q < kSeg8; ++q) tot += s_sum[q][l];
  int64_t all;
  const int64_t off = block_excl_scan<1024>(seg == 0 ? tot : 0, &all, sh);
  if (seg == 0) s_off[l] = (int)off;
  // (levels are used without a gap, so the used ones are counted)
  const int nlev = __syncthreads_count(seg == 0 && tot > 0);
  if (!whole || all != n) return;   // uniform: info.layered stays 0
  int run = s_off[l];
  for (int q = 0; q < seg; ++q) run += s_sum[q][l];
  for (int t = t0; t < t1; t += kU) {
    int v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = t + u < t1 ? h[(int64_t)(t + u) * kWideLevels] : 0;
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (t + u < t1) {
        h[(int64_t)(t + u) * kWideLevels] = run;
        run += v[u];
      }
  }
  if (tid <= nlev) L.lev_off[tid] = tid < nlev ? s_off[tid] : n;
  if (tid < 64) {
    int w = 0;
    for (int q = tid; q < kWideLevels; q += 64) {
      int c = 0;
      for (int k = 0; k < kSeg8; ++k) c += s_sum[k][q];
      w = max(w, c);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o));
    if (tid == 0) {
      L.info[0].nlev = nlev;
      L.info[0].maxwidth = w;
      L.info[0].nunits = 0;
      L.info[0].maxunit = 0;
      L.info[0].layered = 1;
    }
  }
}

gcr_status launch_levels_flow(const LevelsArgs& L, int64_t max_n, hipStream_t st) {
  const int64_t tiles = std::max<int64_t>(1, (max_n + 255) >> 8);
  k_levels_flow<<<(unsigned)std::min<int64_t>(tiles, kFlowGrid), 256, 0, st>>>(L);
  k_levels_scan<<<1, 1024, 0, st>>>(L);
  GCR_HIP(hipGetLastError());
  return GCR_OK;
}

// ---------------------------------------------------------------------------
// Layering in LDS.  One workgroup per instance keeps the byte counters of
// unplaced ghosts read, each ghost's level and a Kahn queue in LDS (the
// queue in HBM when only the rest fits), and the instance's reverse edges
// too when they fit: level k is the queue segment
// its predecessor level released, so a level costs one pass over its own
// ghosts' reverse edges and one barrier.
//
// If the queue runs dry with ghosts left, those read a cycle directly or
// through others.  The ghosts that no unplaced ghost reads are trimmed
// away, repeatedly, leaving the cycles (and any ghost between two); their
// strongly connected groups (transitive closure, as in k_levels) become
// coupled units.  The unplaced ghosts and units are then placed in
// dependency order, each at 1 + the highest level it reads (the level of
// Sec. 3.2: the longest dependency path, units as single nodes).
//
// The canonical order (level, linear index) comes from a stable counting
// sort: per-wave level counts over contiguous ranges of the linear order,
// level offsets from their totals, a scan over the waves per level, and each
// ghost's rank among its wave's ghosts of the same level by ballots.  An
// instance that does not fit, is deeper than kFastLevels or whose units
// exceed the solver's limits is left to k_levels, launched right after,
// which skips the instances finished here (InstInfo::layered).
constexpr int kFastLevels = 256;
constexpr int kFastWaves = 16;     // 1024 threads
constexpr uint16_t kTrimmed = 0xffff;

// Appends v to list[base + ...] (length counter *size) for the lanes with p
// set, one atomic per wave; entries at or beyond cap are dropped (a node
// enters a queue once, so it never holds more than the instance's ghosts;
// the check keeps LDS writes in bounds regardless).
__device__ __forceinline__ void wave_push16(bool p, int v, uint16_t* list, int base,
                                            int* size, int cap) {
  const unsigned long long m = __ballot(p);
  if (m == 0ull) return;
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll((long long)m) - 1;
  int at = 0;
  if (lane == leader) at = atomicAdd(size, __popcll(m));
  at = __shfl(at, leader);
  const int idx = base + at + __popcll(m & ((1ull << lane) - 1ull));
  if (p && idx < cap) list[idx] = (uint16_t)v;
}

// The canonical order (level, linear index) of an instance's n ghosts, and
// its results: a stable counting sort by one workgroup of BS threads, wave w <
// NW taking linear positions [w R, (w + 1) R).  At most BS and 2^BITS levels;
// tab: NW x nlev counts; level_of(g): the level of ghost g.  Every thread calls
// it, after a barrier behind the last write of a level.
template <int BS, int NW, int BITS, class F>
__device__ __forceinline__ void canonical_order(const LevelsArgs& L, int ii, int64_t lo, int n,
                                                int nlev, int units, int maxunit, int32_t* tab,
                                                int* s_off, int* s_tot, int64_t* sh, F level_of) {
  const int tid = threadIdx.x;
  const int R = ((((n + NW - 1) / NW) + 63) / 64) * 64;
  const int wv = tid >> 6, lane = tid & 63;
  for (int t = tid; t < NW * nlev; t += BS) tab[t] = 0;
  __syncthreads();
  const int r0 = wv * R, r1 = wv < NW ? min(n, r0 + R) : r0;
  for (int g = r0 + lane; g < r1; g += 64) atomicAdd(&tab[wv * nlev + level_of(g) - 1], 1);
  __syncthreads();
  for (int l = tid; l < nlev; l += BS) {
    int t = 0;
    for (int w = 0; w < NW; ++w) t += tab[w * nlev + l];
    s_tot[l] = t;
  }
  __syncthreads();
  {
    const int v = tid < nlev ? s_tot[tid] : 0;
    int64_t tot;
    const int64_t pre = block_excl_scan<BS>(v, &tot, sh);
    if (tid < nlev) s_off[tid] = (int)pre;
    if (tid == 0) s_off[nlev] = (int)tot;
  }
  __syncthreads();
  for (int l = tid; l < nlev; l += BS) {
    int run = s_off[l];
    for (int w = 0; w < NW; ++w) {
      const int t = tab[w * nlev + l];
      tab[w * nlev + l] = run;
      run += t;
    }
  }
  __syncthreads();
  int32_t* __restrict__ lev = L.lev + lo;
  int32_t* __restrict__ perm = L.perm + lo;
  for (int c = r0; c < r1; c += 64) {
    const int g = c + lane;
    const bool valid = g < r1;
    const int l = valid ? level_of(g) - 1 : -1;
    // the lanes of this lane's level: those that agree with it on every bit
    // of the level index, one ballot a bit
    unsigned long long mk = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < BITS; ++bit) {
      const bool on = (l >> bit) & 1;
      const unsigned long long bb = __ballot(valid && on);
      mk &= on ? bb : ~bb;
    }
    const int at = valid ? tab[wv * nlev + l] : 0;
    __builtin_amdgcn_wave_barrier();
    if (valid && lane == __ffsll((long long)mk) - 1) tab[wv * nlev + l] = at + __popcll(mk);
    __builtin_amdgcn_wave_barrier();
    if (valid) {
      lev[g] = l + 1;
      perm[g] = at + __popcll(mk & ((1ull << lane) - 1ull));
    }
  }
  int32_t* lev_off = L.lev_off + (int64_t)ii * (kMaxLevels + 1);
  for (int l = tid; l <= nlev; l += BS) lev_off[l] = s_off[l];
  if (tid < 64) {
    int maxw = 0;
    for (int l = tid; l < nlev; l += 64) maxw = max(maxw, s_tot[l]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) maxw = max(maxw, __shfl_xor(maxw, o));
    if (tid == 0) {
      L.info[ii].nlev = nlev;
      L.info[ii].maxwidth = maxw;
      L.info[ii].nunits = units;
      L.info[ii].maxunit = maxunit;
      L.info[ii].layered = 1;
    }
  }
}

// ---------------------------------------------------------------------------
// Layering by pulling, one workgroup per instance of at most kPullMax ghosts.
// A thread holds its ghosts' dependencies in registers and every ghost's
// level lies in LDS; a ghost whose dependencies all have a level takes 1 +
// the highest.  No order between the waves is needed for that (a level is
// the longest dependency path whenever it is found), so the waves only meet
// every kPullRounds rounds to see whether anything moved: no reverse edges,
// no counters, no queue.  Bound by the chain of LDS reads along the longest
// path, about two per level.
//
// When nothing moves with ghosts left, every one of those reads another that
// has no level.  Following each ghost's first such dependency (pointer
// doubling, as many steps as ghosts left) ends on a cycle; a ghost found
// there gathers the ghosts without level it reads, transitively, up to
// kMaxUnit of them.  If the set is closed and strongly connected it is a
// coupled unit that waits for nothing, and takes 1 + the highest level its
// members read outside it (Sec. 3.2's level with the unit as one node);
// pulling then goes on behind it.  One such unit always exists; if none of
// at most kMaxUnit ghosts does, the instance is left to the other layerings.
// (In 3D beyond 8,192 interface cells a thread holds sixteen ghosts: 128
// registers, 18 spilled; a 128^3 body of 8,684 with 16 units takes 157 us so,
// 210 by the push form.)
// Slots come in no particular order: a unit is solved by itself, and what it
// is called by is its smallest ghost.  The 64-star batch: 50 us
// against 129 for the push form with its reverse edges (which took another
// 24 us to build).
//
// Up to kFastLevels levels are ranked by every wave, more by four, whose rank
// table has room for kMaxLevels there.  A build of 258 levels and 2,864 ghosts
// (a circle on 4096 x 64 cells) takes 222 us so; with the push form behind this
// one 1,065, by the push form alone 930.
constexpr int kPullMax = 16384;
constexpr int kPullRounds = 8;   // (4: 37 us on the 2731^2 airfoil, 8: 34, the stars alike, 32: worse there)
constexpr int kPullCand = 256;   // cycle ghosts looked at per stall
constexpr int kPullWS = 3 * kMaxUnit;   // 2-byte members, 1-byte rows of their reads

__device__ __forceinline__ int lds_get(const uint16_t* p) {
  return (int)__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_put(uint16_t* p, int v) {
  __hip_atomic_store(p, (uint16_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// LDS bytes of an instance of n ghosts: levels (one more entry, always
// placed, stands for "no ghost"), the rank table, the cycle search's
// pointers and marks
__host__ __device__ __forceinline__ int64_t pull_lds(int64_t n, int waves) {
  const int64_t tab = 4 * (int64_t)waves * kFastLevels;
  return ((2 * (n + 1) + 15) & ~int64_t(15)) + (tab > 8192 ? tab : 8192) +
         ((2 * n + 15) & ~int64_t(15)) + ((n + 15) & ~int64_t(15));
}

template <int BS>
struct PullShared {
  int off[BS + 2];   // (a level a thread)
  int tot[BS + 1];
  int64_t sh[17];
  int moved[3];
  int left, cand, units, cyclic, maxunit, maxlev, ok;
};

// NP dependencies per ghost at most (np in this instance), J ghosts per
// thread (strided by BS)
template <int BS, int NP, int J>
__device__ __forceinline__ void pull_instance(const LevelsArgs& L, int ii, int64_t lo, int n,
                                              int np, uint32_t* s_dyn, PullShared<BS>& S) {
  const int tid = threadIdx.x;
  const int64_t cap = L.cap;
  const int32_t* __restrict__ deps = L.deps;
  int32_t* __restrict__ blk_idx = L.blk_idx;
  int32_t* unit_mem = L.unit_mem + (int64_t)ii * kMaxUnits * kMaxUnit;
  int32_t* unit_cnt = L.unit_cnt + (int64_t)ii * kMaxUnits;
  int32_t* unit_lev = L.unit_lev + (int64_t)ii * kMaxUnits;
  auto al = [](int64_t b) { return (b + 15) & ~int64_t(15); };
  char* base = reinterpret_cast<char*>(s_dyn);
  uint16_t* lvl = reinterpret_cast<uint16_t*>(base);   // level + 1; 0: none yet
  int64_t o = al(2 * (int64_t)(n + 1));
  int32_t* tab = reinterpret_cast<int32_t*>(base + o);
  // the cycle search's candidates, before the rank table is needed
  uint16_t* cand = reinterpret_cast<uint16_t*>(base + o);
  char* work = base + o + 2 * kPullCand;
  static_assert(2 * kPullCand + kPullCand * kPullWS <= 8192, "pull_lds holds the search");
  constexpr int64_t kTabB = 4 * (int64_t)(BS / 64) * kFastLevels;
  o += kTabB > 8192 ? kTabB : 8192;
  uint16_t* nxt = reinterpret_cast<uint16_t*>(base + o);
  o += al(2 * (int64_t)n);
  uint8_t* mark = reinterpret_cast<uint8_t*>(base + o);
  // dependency q of ghost g as a local id, -1 if it reads no ghost there
  auto gdep = [&](int g, int q) -> int {
    const int32_t d = deps[(int64_t)q * cap + lo + g];
    return d < 0 ? -1 : (int)(d - lo);
  };

  constexpr int W = (NP + 1) / 2;
  uint32_t dp[J][W];
  uint32_t pend = 0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int g = tid + BS * j;
    int d[2 * W];
#pragma unroll
    for (int q = 0; q < 2 * W; ++q) d[q] = q < np && g < n ? gdep(g, q) : -1;
#pragma unroll
    for (int w = 0; w < W; ++w)
      dp[j][w] = (uint32_t)(d[2 * w] < 0 ? n : d[2 * w]) |
                 (uint32_t)(d[2 * w + 1] < 0 ? n : d[2 * w + 1]) << 16;
    if (g < n) {
      pend |= 1u << j;
      lvl[g] = 0;
      blk_idx[lo + g] = -1;
    }
    // bounds the loads in flight, and so the registers that hold them
    if ((j + 1) * W % 8 == 0) asm volatile("" ::: "memory");
  }
  if (tid == 0) {
    lvl[n] = 1;   // level 0: "no ghost" holds nothing up
    S.units = 0;
    S.cyclic = 0;
    S.maxunit = 0;
    S.maxlev = 0;
    S.left = 0;
    S.moved[0] = S.moved[1] = S.moved[2] = 0;
  }
  __syncthreads();
  int top = 0;     // highest level + 1 this thread gave
  int round = 0;
  for (;;) {
    bool moved;
    do {
      moved = false;
      ++round;
#pragma unroll 1
      for (int r = 0; r < kPullRounds && pend; ++r) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
          if (!((pend >> j) & 1u)) continue;
          int lo_ = 0xffff, hi_ = 0;
#pragma unroll
          for (int w = 0; w < W; ++w) {
            // (opaque: unpacked outside the loop, the pairs would take twice
            // their registers)
            uint32_t d = dp[j][w];
            asm volatile("" : "+v"(d));
            const int a = lds_get(lvl + (d & 0xffffu));
            const int b = 2 * w + 1 < NP ? lds_get(lvl + (d >> 16)) : 1;
            lo_ = min(lo_, min(a, b));
            hi_ = max(hi_, max(a, b));
          }
          if (lo_ == 0) continue;
          lds_put(lvl + tid + BS * j, hi_ + 1);
          top = max(top, hi_ + 1);
          pend &= ~(1u << j);
          moved = true;
        }
      }
      // one barrier a turn: three flags in rotation, the next turn's cleared
      // here (it was last read before the previous barrier)
      if (moved) S.moved[round % 3] = 1;
      if (tid == 0) S.moved[(round + 1) % 3] = 0;
      __syncthreads();
    } while (S.moved[round % 3]);
    if (pend) atomicAdd(&S.left, __popc(pend));
    __syncthreads();
    const int m = S.left;
    __syncthreads();
    if (m == 0) break;

    // ---- a stall: the units at the head of what is left
    if (tid == 0) {
      S.left = 0;
      S.cand = 0;
      S.ok = 0;
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (!((pend >> j) & 1u)) continue;
      int f = n;
#pragma unroll
      for (int q = NP - 1; q >= 0; --q) {
        uint32_t pair = dp[j][q / 2];
        asm volatile("" : "+v"(pair));
        const int d = (int)(q & 1 ? pair >> 16 : pair & 0xffffu);
        if (lds_get(lvl + d) == 0) f = d;
      }
      nxt[tid + BS * j] = (uint16_t)f;
      mark[tid + BS * j] = 0;
    }
    __syncthreads();
    for (int step = 1; step < 2 * m; step <<= 1) {   // (in place: a pointer only runs ahead)
#pragma unroll
      for (int j = 0; j < J; ++j)
        if ((pend >> j) & 1u) lds_put(nxt + tid + BS * j, lds_get(nxt + lds_get(nxt + tid + BS * j)));
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
      if ((pend >> j) & 1u) mark[nxt[tid + BS * j]] = 1;   // every writer stores 1
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (((pend >> j) & 1u) && mark[tid + BS * j]) {
        const int at = atomicAdd(&S.cand, 1);
        if (at < kPullCand) cand[at] = (uint16_t)(tid + BS * j);
      }
    __syncthreads();
    const int nc = min(S.cand, kPullCand);
    // one candidate a thread
    uint16_t* mem = reinterpret_cast<uint16_t*>(work + tid * kPullWS);
    uint8_t* row = reinterpret_cast<uint8_t*>(mem + kMaxUnit);
    int k = 0, ext = 0;
    if (tid < nc) {
      const int c = cand[tid];
      mem[0] = (uint16_t)c;
      row[0] = 0;
      k = 1;
      for (int i = 0; i < k && k > 0; ++i)
        for (int q = 0; q < np; ++q) {
          const int d = gdep(mem[i], q);
          if (d < 0) continue;
          if (lvl[d] != 0) {
            ext = max(ext, (int)lvl[d]);
            continue;
          }
          int t = 0;
          while (t < k && mem[t] != d) ++t;
          if (t == k) {
            if (k == kMaxUnit) {   // too large, or more than the head unit
              k = 0;
              break;
            }
            mem[k] = (uint16_t)d;
            row[k] = 0;
            ++k;
          }
          row[i] |= (uint8_t)(1u << t);
        }
      // closed: strongly connected if every member reaches the candidate,
      // and taken by the smallest candidate among the members
      for (int v = 0; v < k; ++v)
        for (int u = 0; u < k; ++u)
          if ((row[u] >> v) & 1u) row[u] |= row[v];
      bool take = k > 0;
      for (int u = 0; u < k; ++u) take = take && (row[u] & 1u) && !(mark[mem[u]] && mem[u] < c);
      if (!take) k = 0;
      if (k > 0) {
        for (int u = 1; u < k; ++u)   // members ascending
          for (int t = u; t > 0 && mem[t - 1] > mem[t]; --t) {
            const uint16_t x = mem[t];
            mem[t] = mem[t - 1];
            mem[t - 1] = x;
          }
        const int slot = atomicAdd(&S.units, 1);
        if (slot < kMaxUnits) {
          for (int u = 0; u < k; ++u) {
            unit_mem[slot * kMaxUnit + u] = (int32_t)(lo + mem[u]);
            blk_idx[lo + mem[u]] = slot;
          }
          unit_cnt[slot] = k;
          unit_lev[slot] = max(ext, 1);   // (levels in LDS are one higher)
        }
        atomicMax(&S.maxunit, k);
        atomicAdd(&S.cyclic, k);
        S.ok = 1;
      }
    }
    __syncthreads();
    // (more ghosts in cycles than the push form resolves: refused there)
    if (!S.ok || S.units > kMaxUnits || S.cyclic > kMaxResidual) {   // uniform
      for (int g = tid; g < n; g += BS) L.perm[lo + g] = -1;
      return;
    }
    for (int u = 0; u < k; ++u) lds_put(lvl + mem[u], max(ext, 1) + 1);
    if (k > 0) top = max(top, max(ext, 1) + 1);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (((pend >> j) & 1u) && lds_get(lvl + tid + BS * j) != 0) pend &= ~(1u << j);
  }
  if (top) atomicMax(&S.maxlev, top - 1);
  __syncthreads();
  const int nlev = S.maxlev, nu = S.units;
  if (nlev > BS) {   // uniform
    for (int g = tid; g < n; g += BS) L.perm[lo + g] = -1;
    return;
  }
  auto level_of = [&](int g) { return (int)lvl[g] - 1; };
  static_assert((kTabB > 8192 ? kTabB : 8192) >= 16 * BS, "four waves rank a level a thread");
  if (BS <= kFastLevels || nlev <= kFastLevels)
    canonical_order<BS, BS / 64, 8>(L, ii, lo, n, nlev, nu, S.maxunit, tab, S.off, S.tot, S.sh,
                                    level_of);
  else
    canonical_order<BS, 4, 10>(L, ii, lo, n, nlev, nu, S.maxunit, tab, S.off, S.tot, S.sh,
                               level_of);
}

template <int BS, int NP, int J>
__global__ __launch_bounds__(BS) void k_levels_pull(LevelsArgs L, int lds_bytes) {
  extern __shared__ uint32_t s_dyn[];
  __shared__ PullShared<BS> S;
  const int ii = blockIdx.x;
  const int64_t lo = L.g_off[ii];
  const int n = (int)(L.g_off[ii + 1] - lo);
  if (n > BS * J || pull_lds(n, BS / 64) > lds_bytes) return;
  pull_instance<BS, NP, J>(L, ii, lo, n, min(NP, (1 << L.insts[ii].g.dim) - 1), s_dyn, S);
}

__global__ __launch_bounds__(1024) void k_levels_fast(LevelsArgs L, int lds_bytes) {
  extern __shared__ uint32_t s_dyn[];
  __shared__ int s_off[kFastLevels + 2];
  __shared__ int s_tot[kFastLevels + 1];
  __shared__ int s_cnt[3];
  __shared__ int64_t sh[17];
  __shared__ int s_flag, s_units, s_maxunit, s_maxlev, s_placed, s_bad;
  const int ii = blockIdx.x;
  if (L.info[ii].layered) return;   // (a second layering: it left this one out)
  const int tid = threadIdx.x;
  const int64_t lo = L.g_off[ii];
  const int n = (int)(L.g_off[ii + 1] - lo);
  if (n > 65535) return;   // 16-bit ids in the queue
  const int np = (1 << L.insts[ii].g.dim) - 1;
  const int64_t cap = L.cap;
  const int32_t* __restrict__ deps = L.deps;
  const int32_t* __restrict__ roff = L.roff + lo;
  const int32_t* __restrict__ radj = L.radj;
  const uint8_t* __restrict__ dcnt = L.dcnt + lo;
  int32_t* __restrict__ blk_idx = L.blk_idx;      // global linear ids
  int32_t* unit_mem = L.unit_mem + (int64_t)ii * kMaxUnits * kMaxUnit;
  int32_t* unit_cnt = L.unit_cnt + (int64_t)ii * kMaxUnits;
  int32_t* unit_lev = L.unit_lev + (int64_t)ii * kMaxUnits;
  const int64_t e0 = roff[0];
  const int E = (int)(roff[n] - e0);
  auto al = [](int64_t b) { return (b + 15) & ~int64_t(15); };
  char* base = reinterpret_cast<char*>(s_dyn);
  int64_t o = 0;
  uint32_t* cnt = reinterpret_cast<uint32_t*>(base + o);
  o += al(4 * (int64_t)((n + 3) >> 2));
  uint16_t* lvl = reinterpret_cast<uint16_t*>(base + o);
  o += al(2 * (int64_t)n);
  // the release queue: in LDS when it fits beside the rank table, else in the
  // instance's slice of listA (HBM, 2 bytes a ghost of its 4), which leaves
  // 3 bytes a ghost in LDS
  constexpr int64_t kTab = 4 * (int64_t)kFastWaves * kFastLevels;
  const bool qlds = o + al(2 * (int64_t)n) + kTab <= lds_bytes;
  uint16_t* que = qlds ? reinterpret_cast<uint16_t*>(base + o)
                       : reinterpret_cast<uint16_t*>(L.listA + lo);
  if (qlds) o += al(2 * (int64_t)n);
  // [kFastWaves][kFastLevels] rank counts; before that the cycle search's
  // residual list, representatives and unit slots (3 x kMaxResidual)
  int32_t* tab = reinterpret_cast<int32_t*>(base + o);
  o += kTab;
  if (o > lds_bytes) return;   // every thread leaves alike
  // reverse edges, then (used only after a stall) the forward dependencies
  // as local ids and each ghost's unit slot, each where LDS is left
  int32_t* eoff = reinterpret_cast<int32_t*>(base + o);
  const int64_t o_adj = o + al(4 * ((int64_t)n + 1));
  uint16_t* eadj = reinterpret_cast<uint16_t*>(base + o_adj);
  const int64_t o_eend = o_adj + al(2 * (int64_t)E);
  const bool elds = o_eend <= lds_bytes;
  const int64_t o_dep = elds ? o_eend : o;
  uint16_t* fdep = reinterpret_cast<uint16_t*>(base + o_dep);
  const int64_t o_slot = o_dep + al(2 * (int64_t)np * n);
  uint16_t* uslot = reinterpret_cast<uint16_t*>(base + o_slot);
  const bool dlds = o_slot + al(2 * (int64_t)n) <= lds_bytes;
  __shared__ uint16_t s_uhead[kMaxUnits];   // head (smallest member) of each unit
  __shared__ uint8_t s_usize[kMaxUnits];
  auto edge_range = [&](int g, int& ea, int& eb) {
    ea = elds ? eoff[g] : (int)(roff[g] - e0);
    eb = elds ? eoff[g + 1] : (int)(roff[g + 1] - e0);
  };
  auto dependant = [&](int e) { return elds ? (int)eadj[e] : (int)(radj[e0 + e] - lo); };
  // dependency q of ghost g as a local id, -1 if it reads no ghost there
  auto dep = [&](int g, int q) -> int {
    if (dlds) {
      const int v = fdep[q * n + g];
      return v == 0xffff ? -1 : v;
    }
    const int32_t d = deps[(int64_t)q * cap + lo + g];
    return d < 0 ? -1 : (int)(d - lo);
  };
  auto slot_of = [&](int g) -> int {
    if (dlds) {
      const int v = uslot[g];
      return v == 0xffff ? -1 : v;
    }
    return blk_idx[lo + g];
  };

  const int C = (n + 3) >> 2;
  for (int w = tid; w < C; w += 1024) {
    uint32_t v = 0;
    for (int q = 0; q < 4; ++q)
      if (4 * w + q < n) v |= (uint32_t)dcnt[4 * w + q] << (8 * q);
    cnt[w] = v;
  }
  for (int g = tid; g < n; g += 1024) {
    lvl[g] = 0;
    blk_idx[lo + g] = -1;
  }
  if (elds) {
    for (int g = tid; g <= n; g += 1024) eoff[g] = (int)(roff[g] - e0);
    for (int e = tid; e < E; e += 1024) eadj[e] = (uint16_t)(radj[e0 + e] - lo);
  }
  if (tid < 3) s_cnt[tid] = 0;
  if (tid == 0) {
    s_units = 0;
    s_maxunit = 0;
    s_bad = 0;
  }
  __syncthreads();
  // level 1: ghosts that read no ghost
  for (int g = tid; g < n; g += 1024) {
    const bool p = dcnt[g] == 0;
    if (p) lvl[g] = 1;
    wave_push16(p, g, que, 0, &s_cnt[0], n);
  }
  __syncthreads();
  int a = 0, b = s_cnt[0], k = 0;
  // iteration k: level k (queue[a, b)) releases level k + 1 into queue[b,
  // ...), its length accumulating in s_cnt[k % 3].  The counter of the next
  // iteration, s_cnt[(k + 1) % 3], was last read after the barrier that
  // ended iteration k - 2, which every thread has passed since, so thread 0
  // clears it now.
  while (a < b) {
    ++k;
    if (k > kFastLevels) return;   // uniform: every thread counts the same levels
    if (tid == 0) s_cnt[(k + 1) % 3] = 0;
    int* const tail = &s_cnt[k % 3];
    for (int i = a + tid; i < b; i += 1024) {
      const int g = que[i];
      int ea, eb;
      edge_range(g, ea, eb);
      for (int e = ea; e < eb; ++e) {
        const int q = dependant(e);
        const bool rel = cnt_dec(cnt, q) == 1u;
        if (rel) lvl[q] = (uint16_t)(k + 1);
        wave_push16(rel, q, que, b, tail, n);
      }
    }
    __syncthreads();
    a = b;
    b += *tail;
    if (b > n) return;   // cannot happen (each ghost released once)
  }
  if (tid == 0) {
    s_maxlev = k;
    s_placed = b;
  }

  if (b < n && n - b <= L.wave_res) {   // (wave_res <= 64)
    // ---- at most 64 ghosts left (they read a cycle): one wave finds the
    // cycles and places them, with no workgroup barrier.  Lane u holds
    // residual ghost res[u] and the set A of residual ghosts it reads; the
    // closure R = A+ comes from Warshall's pass over its lanes, the group of
    // a ghost on a cycle (u in R[u]) is R[u] & {v : u in R[v]}, whose
    // smallest member is its representative, and the groups' slots follow
    // their representatives' order.  Then every residual ghost or group is
    // placed, in dependency order, at 1 + the highest level it reads outside
    // its group.  The result is the one of the general path below, which
    // trims ghosts off the cycles first: a ghost on a cycle is never trimmed,
    // and the levels are the same longest-path levels.
    if (tid < 64) {
      const int lane = tid;
      int32_t* res = tab;          // [64] residual ghosts, ascending
      int32_t* s_c = tab + 128;    // [64] the placement order
      int m = 0;
      for (int g0 = 0; g0 < n; g0 += 64) {
        const int g = g0 + lane;
        const bool left = g < n && lvl[g] == 0;
        const unsigned long long bm = __ballot(left);
        if (left) res[m + __popcll(bm & ((1ull << lane) - 1ull))] = g;
        m += __popcll(bm);
      }
      __builtin_amdgcn_wave_barrier();
      // dependency q of ghost g as a local id, -1 if it reads no ghost there
      auto gdep = [&](int g, int q) -> int {
        const int32_t d = deps[(int64_t)q * cap + lo + g];
        return d < 0 ? -1 : (int)(d - lo);
      };
      // the residual ghosts each lane reads (A) and the highest level among
      // the ghosts it reads that the layering placed (ext), read once
      const int g = lane < m ? res[lane] : -1;
      unsigned long long A = 0ull;
      int ext = 0;
      if (lane < m)
        for (int q = 0; q < np; ++q) {
          const int d = gdep(g, q);
          if (d < 0) continue;
          if (lvl[d] != 0) {
            ext = max(ext, (int)lvl[d]);
            continue;
          }
          const int v = (int)find_sorted(res, 0, m, d);
          if (v >= 0) A |= 1ull << v;
        }
      // closure R = A+ by Warshall's pass: after step v, R[u] holds every
      // ghost u reaches through intermediates among the first v + 1; row v
      // is read from its lane with readlane (v is uniform), no LDS
      unsigned long long R = A;
      const int mu = __builtin_amdgcn_readfirstlane(m);   // (the same in every lane)
      for (int v = 0; v < mu; ++v) {
        const uint32_t rlo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)R, v);
        const uint32_t rhi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(R >> 32), v);
        if ((R >> v) & 1ull) R |= ((unsigned long long)rhi << 32) | rlo;
      }
      unsigned long long T = 0ull;   // {v : lane in R[v]}
      for (int u = 0; u < m; ++u) {
        const unsigned long long col = __ballot(lane < m && ((R >> u) & 1ull));
        if (lane == u) T = col;
      }
      const bool oncyc = lane < m && ((R >> lane) & 1ull);
      const unsigned long long M = oncyc ? (R & T) : (lane < m ? (1ull << lane) : 0ull);
      const int rep = oncyc ? __ffsll((long long)M) - 1 : -1;
      const int size = __popcll(M);
      const unsigned long long reps = __ballot(oncyc && rep == lane);
      const int nunits = __popcll(reps);
      const bool bad = __ballot(oncyc && size > kMaxUnit) != 0ull;
      int slot = -1;
      if (oncyc) slot = __popcll(reps & ((1ull << rep) - 1ull));
      if (!bad && oncyc) {
        unit_mem[slot * kMaxUnit + __popcll(M & ((1ull << lane) - 1ull))] = (int32_t)(lo + g);
        blk_idx[lo + g] = slot;
        if (rep == lane) unit_cnt[slot] = size;
      }
      // placement in dependency order, in one pass in registers.  Ghost u
      // reading ghost w of another group has a larger key 2 |R[u]| + (u not
      // on a cycle) than w: R[u] holds R[w], and u itself (u on a cycle) or
      // w's own group (w on a cycle) or w (neither) besides.  So the order
      // of (key, lane) places every group after all it reads; a group's
      // members share R and sit together.  c: the highest level the lane
      // reads outside its group (ext to start with), final when its group's
      // turn comes; the group's level is 1 + the highest c of its members.
      int Lown = 0;
      if (!bad) {
        const int key = lane < m ? 2 * __popcll(R) + (oncyc ? 0 : 1) : 0x7fffffff;
        int rank = 0;
        for (int v = 0; v < mu; ++v) {
          const int kv = __builtin_amdgcn_readlane(key, v);
          rank += (kv < key || (kv == key && v < lane)) ? 1 : 0;
        }
        if (lane < m) s_c[rank] = lane;
        __builtin_amdgcn_wave_barrier();
        const int ord = lane < m ? s_c[lane] : 0;
        const unsigned long long outside = A & ~M;
        int c = ext;
        for (int pos = 0; pos < mu; ++pos) {
          const int v = __builtin_amdgcn_readlane(ord, pos);
          if (__builtin_amdgcn_readlane(Lown, v) != 0) continue;   // placed with its group
          const unsigned long long Mv =
              ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(M >> 32), v) << 32) |
              (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)M, v);
          int mx = 0;
          for (unsigned long long w = Mv; w; w &= w - 1ull)
            mx = max(mx, __builtin_amdgcn_readlane(c, __ffsll((long long)w) - 1));
          if ((Mv >> lane) & 1ull) Lown = mx + 1;
          if (outside & Mv) c = max(c, mx + 1);
        }
      }
      if (bad) {
        if (lane == 0) s_bad = 1;
      } else {
        const int L = lane < m ? Lown : 0;
        if (lane < m && L > 0) lvl[g] = (uint16_t)L;
        if (oncyc && rep == lane) unit_lev[slot] = L;
        int mxl = L, mxs = oncyc ? size : 0, done = lane < m && L > 0 ? 1 : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          mxl = max(mxl, __shfl_xor(mxl, o));
          mxs = max(mxs, __shfl_xor(mxs, o));
          done += __shfl_xor(done, o);
        }
        if (lane == 0) {
          s_units = nunits;
          s_maxunit = mxs;
          s_maxlev = max(s_maxlev, mxl);
          s_placed += done;
        }
      }
    }
    __syncthreads();
    if (s_bad) return;
  } else if (b < n) {
    // ---- the ghosts left read a cycle.  Trim those that no unplaced ghost
    // reads (counters: unplaced readers), repeatedly.
    if (dlds) {
      for (int t = tid; t < np * n; t += 1024) {
        const int q = t / n, g = t - q * n;
        const int32_t d = deps[(int64_t)q * cap + lo + g];
        fdep[t] = d < 0 ? (uint16_t)0xffff : (uint16_t)(d - lo);
      }
      for (int g = tid; g < n; g += 1024) uslot[g] = 0xffff;
    }
    for (int w = tid; w < C; w += 1024) cnt[w] = 0;
    __syncthreads();
    for (int g = tid; g < n; g += 1024) {
      if (lvl[g] != 0) continue;
      int ea, eb;
      edge_range(g, ea, eb);
      uint32_t c = 0;
      for (int e = ea; e < eb; ++e) c += lvl[dependant(e)] == 0 ? 1u : 0u;
      if (c) cnt_add(cnt, g, c);
    }
    if (tid < 3) s_cnt[tid] = 0;
    __syncthreads();
    for (int g = tid; g < n; g += 1024) {
      const bool p = lvl[g] == 0 && cnt_get(cnt, g) == 0;
      if (p) lvl[g] = kTrimmed;
      wave_push16(p, g, que, b, &s_cnt[0], n);
    }
    __syncthreads();
    {
      int ta = b, tb = b + s_cnt[0], r = 0;
      while (ta < tb) {
        ++r;
        if (tid == 0) s_cnt[(r + 1) % 3] = 0;
        int* const tail = &s_cnt[r % 3];
        for (int i = ta + tid; i < tb; i += 1024) {
          const int u = que[i];
          for (int q = 0; q < np; ++q) {
            const int dl = dep(u, q);
            bool rel = false;
            if (dl >= 0 && lvl[dl] == 0 && cnt_dec(cnt, dl) == 1u) {
              rel = true;
              lvl[dl] = kTrimmed;
            }
            wave_push16(rel, dl, que, tb, tail, n);
          }
        }
        __syncthreads();
        ta = tb;
        tb += *tail;
        if (tb > n) return;
      }
    }
    // ---- strongly connected groups of the untrimmed ghosts (ascending)
    int32_t* res = tab;
    int32_t* rep = tab + kMaxResidual;
    int32_t* slot = tab + 2 * kMaxResidual;
    int m = 0;
    for (int b0 = 0; b0 < n; b0 += 1024) {
      const int g = b0 + tid;
      const bool left = g < n && lvl[g] == 0;
      int64_t tot;
      const int64_t pre = block_excl_scan<1024>(left ? 1 : 0, &tot, sh);
      if (left && m + pre < kMaxResidual) res[m + pre] = g;
      m += (int)tot;
    }
    if (m == 0 || m > kMaxResidual) return;
    uint32_t* reach = L.reach + (int64_t)ii * kMaxResidual * (kMaxResidual / 32);
    const int RW = (m + 31) / 32;
    for (int t = tid; t < m * RW; t += 1024) reach[t] = 0;
    __threadfence_block();
    __syncthreads();
    for (int u = tid; u < m; u += 1024)
      for (int q = 0; q < np; ++q) {
        const int d = dep(res[u], q);
        if (d < 0 || lvl[d] != 0) continue;
        const int v = (int)find_sorted(res, 0, m, d);
        if (v >= 0) reach[u * RW + (v >> 5)] |= 1u << (v & 31);
      }
    __threadfence_block();
    __syncthreads();
    do {
      if (tid == 0) s_flag = 0;
      __syncthreads();
      int changed = 0;
      for (int u = tid; u < m; u += 1024)
        for (int q = 0; q < np; ++q) {
          const int d = dep(res[u], q);
          if (d < 0 || lvl[d] != 0) continue;
          const int v = (int)find_sorted(res, 0, m, d);
          if (v < 0) continue;
          for (int w = 0; w < RW; ++w) {
            const uint32_t ow = reach[u * RW + w], nw = ow | reach[v * RW + w];
            if (nw != ow) {
              reach[u * RW + w] = nw;
              changed = 1;
            }
          }
        }
      if (changed) s_flag = 1;
      __threadfence_block();
      __syncthreads();
    } while (s_flag);
    // representative: smallest member of the group; -1 off cycles
    for (int u = tid; u < m; u += 1024) {
      int rp = -1;
      if ((reach[u * RW + (u >> 5)] >> (u & 31)) & 1u)
        for (int v = 0; v < m; ++v)
          if (((reach[u * RW + (v >> 5)] >> (v & 31)) & 1u) &&
              ((reach[v * RW + (u >> 5)] >> (u & 31)) & 1u)) {
            rp = v;
            break;
          }
      rep[u] = rp;
    }
    __syncthreads();
    {
      int off = 0;
      for (int b0 = 0; b0 < m; b0 += 1024) {
        const int u = b0 + tid;
        const bool isrep = u < m && rep[u] == u;
        int64_t tot;
        const int64_t pre = block_excl_scan<1024>(isrep ? 1 : 0, &tot, sh);
        if (isrep) slot[u] = off + (int)pre;
        off += (int)tot;
      }
      if (tid == 0) s_units = off;
    }
    __syncthreads();
    if (s_units > kMaxUnits) return;
    for (int u = tid; u < m; u += 1024) {
      const int rp = rep[u];
      if (rp < 0) continue;
      int rank = 0, size = 0;
      for (int v = 0; v < m; ++v)
        if (rep[v] == rp) {
          if (v < u) ++rank;
          ++size;
        }
      if (size > kMaxUnit) {   // larger than the LDS solve's workspace
        s_bad = 1;
        continue;
      }
      const int sl = slot[rp];
      unit_mem[sl * kMaxUnit + rank] = (int32_t)(lo + res[u]);
      blk_idx[lo + res[u]] = sl;
      if (dlds) uslot[res[u]] = (uint16_t)sl;
      if (u == rp) {
        unit_cnt[sl] = size;
        s_uhead[sl] = (uint16_t)res[u];
        s_usize[sl] = (uint8_t)size;
        atomicMax(&s_maxunit, size);
      }
    }
    for (int g = tid; g < n; g += 1024)
      if (lvl[g] == kTrimmed) lvl[g] = 0;
    __threadfence_block();
    __syncthreads();
    if (s_bad) return;

    // ---- the unplaced ghosts and units in dependency order, each at 1 +
    // the highest level it reads (internal edges of a unit excluded)
    auto head_of = [&](int g) {
      const int u = slot_of(g);
      return u >= 0 ? (int)s_uhead[u] : g;
    };
    auto place = [&](int t) {   // level of node t, given to its members
      const int u = slot_of(t);
      const int sz = u >= 0 ? (int)s_usize[u] : 1;
      int mx = 0;
      for (int j = 0; j < sz; ++j) {
        const int gm = u >= 0 ? (int)(unit_mem[u * kMaxUnit + j] - lo) : t;
        for (int q = 0; q < np; ++q) {
          const int d = dep(gm, q);
          if (d < 0 || (u >= 0 && slot_of(d) == u)) continue;
          mx = max(mx, (int)lvl[d]);
        }
      }
      for (int j = 0; j < sz; ++j) {
        const int gm = u >= 0 ? (int)(unit_mem[u * kMaxUnit + j] - lo) : t;
        lvl[gm] = (uint16_t)(mx + 1);
      }
      if (u >= 0) unit_lev[u] = mx + 1;
      atomicAdd(&s_placed, sz);
      atomicMax(&s_maxlev, mx + 1);
    };
    for (int w = tid; w < C; w += 1024) cnt[w] = 0;
    __syncthreads();
    for (int g = tid; g < n; g += 1024) {
      if (lvl[g] != 0) continue;
      const int u = slot_of(g);
      uint32_t c = 0;
      for (int q = 0; q < np; ++q) {
        const int d = dep(g, q);
        if (d < 0 || lvl[d] != 0 || (u >= 0 && slot_of(d) == u)) continue;
        ++c;
      }
      if (c) cnt_add(cnt, head_of(g), c);
    }
    if (tid < 3) s_cnt[tid] = 0;
    __syncthreads();
    for (int g = tid; g < n; g += 1024) {
      bool p = false;
      if (lvl[g] == 0 && head_of(g) == g && cnt_get(cnt, g) == 0) p = true;
      if (p) place(g);
      wave_push16(p, g, que, b, &s_cnt[0], n);
    }
    __threadfence_block();
    __syncthreads();
    int ra = b, rb = b + s_cnt[0], r = 0;
    while (ra < rb) {
      ++r;
      if (tid == 0) s_cnt[(r + 1) % 3] = 0;
      int* const tail = &s_cnt[r % 3];
      for (int i = ra + tid; i < rb; i += 1024) {
        const int t = que[i];
        const int u = slot_of(t);
        const int sz = u >= 0 ? (int)s_usize[u] : 1;
        for (int j = 0; j < sz; ++j) {
          const int gm = u >= 0 ? (int)(unit_mem[u * kMaxUnit + j] - lo) : t;
          int ea, eb;
          edge_range(gm, ea, eb);
          for (int e = ea; e < eb; ++e) {
            const int q = dependant(e);
            bool rel = false;
            int tq = 0;
            if (lvl[q] == 0) {   // members of t's own unit are placed already
              tq = head_of(q);
              if (cnt_dec(cnt, tq) == 1u) {
                rel = true;
                place(tq);
              }
            }
            wave_push16(rel, tq, que, rb, tail, n);
          }
        }
      }
      __threadfence_block();
      __syncthreads();
      ra = rb;
      rb += *tail;
      if (rb > n) return;
    }
  }
  __syncthreads();
  if (s_placed != n || s_maxlev > kFastLevels) return;   // k_levels does it
  canonical_order<1024, kFastWaves, 8>(L, ii, lo, n, s_maxlev, s_units, s_maxunit, tab, s_off, s_tot, sh,
                        [&](int g) { return (int)lvl[g]; });
}

constexpr int kRelU = 4;   // ghosts per thread whose releases are issued together
constexpr int kRelE = 4;   // their edges loaded up front (the rest, if any, one by one)

// InLds: byte counters and level bitmap in LDS; CurLds: the current level's
// list too (it is written and read back within each level)
template <bool InLds, bool CurLds>
__global__ __launch_bounds__(1024) void k_levels(LevelsArgs L) {
  extern __shared__ uint32_t s_dyn[];
  const int ii = blockIdx.x;
  if (L.info[ii].layered) return;   // the LDS layering finished it
  const int tid = threadIdx.x;
  const int np = (1 << L.insts[ii].g.dim) - 1;
  const int64_t lo = L.g_off[ii];
  const int n = (int)(L.g_off[ii + 1] - lo);
  const int W = (n + 31) >> 5;   // bitmap words
  const int C = (n + 3) >> 2;    // counter words
  const int64_t cap = L.cap;
  const int32_t* __restrict__ deps = L.deps;
  int32_t* __restrict__ lev = L.lev;
  int32_t* __restrict__ blk_idx = L.blk_idx;
  int32_t* __restrict__ perm = L.perm;
  const uint8_t* __restrict__ dcnt = L.dcnt + lo;
  const int32_t* __restrict__ roff = L.roff + lo;   // global ids in radj
  const int32_t* __restrict__ radj = L.radj;
  int32_t* lev_off = L.lev_off + (int64_t)ii * (kMaxLevels + 1);
  int32_t* unit_mem = L.unit_mem + (int64_t)ii * kMaxUnits * kMaxUnit;
  int32_t* unit_cnt = L.unit_cnt + (int64_t)ii * kMaxUnits;
  int32_t* unit_lev = L.unit_lev + (int64_t)ii * kMaxUnits;
  uint32_t* reach = L.reach + (int64_t)ii * kMaxResidual * (kMaxResidual / 32);
  // the level list: its first cur_cap entries in LDS after the counters
  // and bitmap (the rest, if a level is wider, in HBM)
  int32_t* gcur = L.listA + lo;
  int32_t* lcur = CurLds ? reinterpret_cast<int32_t*>(s_dyn + C + W) : nullptr;
  const int ccap = CurLds ? L.cur_cap : 0;
  // instance ii owns words [(lo >> 2) + ii, + C) and [(lo >> 5) + ii, + W):
  // the next instance starts at ((lo + n) >> 2) + ii + 1 >= that end
  uint32_t* cnt = InLds ? s_dyn : L.cnt + (lo >> 2) + ii;
  uint32_t* bits = InLds ? s_dyn + C : L.bits + (lo >> 5) + ii;

  __shared__ int64_t sh[17];
  __shared__ int s_flag, s_units, s_maxunit;
  __shared__ int32_t res[kMaxResidual];
  __shared__ int32_t rep[kMaxResidual];
  __shared__ int32_t slot[kMaxResidual];

  for (int g = tid; g < n; g += 1024) blk_idx[lo + g] = -1;
  if (tid == 0) {
    lev_off[0] = 0;
    s_units = 0;
    s_maxunit = 0;
  }
  __syncthreads();

  bool units = false;
  int k = 0, placed = 0, maxwidth = 0;
  uint32_t err = 0;
  for (;;) {
    // ---- counters of unplaced ghosts read (per ghost, or per unit on its
    // first member), internal edges of a unit excluded
    for (int g = tid; g < n; g += 1024) {
      lev[lo + g] = 0;
      perm[lo + g] = -1;
    }
    if (!units) {
      // four counters per word, and level 1 = ghosts that read no ghost
      for (int w = tid; w < C; w += 1024) {
        uint32_t v = 0;
        for (int q = 0; q < 4; ++q)
          if (4 * w + q < n) v |= (uint32_t)dcnt[4 * w + q] << (8 * q);
        cnt[w] = v;
      }
      // level-1 bitmap: each wave reads 64 consecutive counts (one byte per
      // lane) and writes the two words of their ballot
      for (int g0 = tid & ~63; g0 < n; g0 += 1024) {
        const int g = g0 + (tid & 63);
        const unsigned long long m = __ballot(g < n && dcnt[g] == 0);
        if ((tid & 63) == 0) {
          bits[g0 >> 5] = (uint32_t)m;
          if ((g0 >> 5) + 1 < W) bits[(g0 >> 5) + 1] = (uint32_t)(m >> 32);
        }
      }
      __syncthreads();
    } else {
      for (int w = tid; w < C; w += 1024) cnt[w] = 0;
      for (int w = tid; w < W; w += 1024) bits[w] = 0;
      __syncthreads();
      for (int g = tid; g < n; g += 1024) {
        const int u = blk_idx[lo + g];
        const int tgt = u >= 0 ? (int)(unit_mem[u * kMaxUnit] - lo) : g;
        uint32_t c = 0;
        for (int m = 0; m < np; ++m) {
          const int32_t d = deps[(int64_t)m * cap + lo + g];
          if (d >= 0 && !(u >= 0 && blk_idx[d] == u)) ++c;
        }
        if (c) cnt_add(cnt, tgt, c);
      }
      __syncthreads();
      // level 1: nodes that read no unplaced ghost
      for (int g = tid; g < n; g += 1024) {
        const int u = blk_idx[lo + g];
        if (u >= 0 && unit_mem[u * kMaxUnit] - lo != g) continue;
        if (cnt_get(cnt, g) != 0) continue;
        if (u >= 0) {
          unit_lev[u] = 1;
          for (int q = 0; q < unit_cnt[u]; ++q) {
            const int v = (int)(unit_mem[u * kMaxUnit + q] - lo);
            atomicOr(&bits[v >> 5], 1u << (v & 31));
          }
        } else {
          atomicOr(&bits[g >> 5], 1u << (g & 31));
        }
      }
      __syncthreads();
    }

    k = 0;
    placed = 0;
    maxwidth = 0;
    for (;;) {
      // ---- emit the next level from the bitmap, in linear-index order
      int newly = 0;
      for (int base = 0; base < W; base += 1024) {
        const int w = base + tid;
        uint32_t word = w < W ? bits[w] : 0u;
        int64_t tot;
        const int64_t pre = block_excl_scan<1024>(__popc(word), &tot, sh);
        if (word) {
          bits[w] = 0u;
          int pos = newly + (int)pre;
          while (word) {
            const int b = __ffs(word) - 1;
            word &= word - 1;
            const int g = w * 32 + b;
            if (pos < ccap) lcur[pos] = g;
            else gcur[pos] = g;
            perm[lo + g] = placed + pos;
            lev[lo + g] = k + 1;
            ++pos;
          }
        }
        newly += (int)tot;
      }
      if (newly == 0) break;
      ++k;
      if (k > kMaxLevels) {
        err |= kErrUnsupported;
        break;
      }
      placed += newly;
      maxwidth = max(maxwidth, newly);
      if (tid == 0) lev_off[k] = placed;
      __syncthreads();
      // ---- dependants of level k: the last edge into a node releases it.
      // A thread takes kRelU ghosts of the level at a time and issues their
      // loads together (list entry, edge range, first kRelE edges), so the
      // dependent global round trips are paid once per group, not per ghost;
      // the order of releases does not matter (a counter reaching zero sets
      // a bit of the next level's bitmap)
      auto release = [&](int rg, int ug) {
        const int r = (int)(rg - lo);
        const int ur = units ? blk_idx[lo + r] : -1;
        if (ur >= 0 && ur == ug) return;
        const int tgt = ur >= 0 ? (int)(unit_mem[ur * kMaxUnit] - lo) : r;
        if (cnt_dec(cnt, tgt) != 1u) return;
        if (ur >= 0) {
          unit_lev[ur] = k + 1;
          for (int q = 0; q < unit_cnt[ur]; ++q) {
            const int v = (int)(unit_mem[ur * kMaxUnit + q] - lo);
            atomicOr(&bits[v >> 5], 1u << (v & 31));
          }
        } else {
          atomicOr(&bits[r >> 5], 1u << (r & 31));
        }
      };
      for (int i0 = tid; i0 < newly; i0 += 1024 * kRelU) {
        int gg[kRelU], ea[kRelU], eb[kRelU], rr[kRelU][kRelE];
#pragma unroll
        for (int u = 0; u < kRelU; ++u) {
          const int i = i0 + u * 1024;
          gg[u] = i >= newly ? -1 : i < ccap ? lcur[i] : gcur[i];
        }
#pragma unroll
        for (int u = 0; u < kRelU; ++u) {
          ea[u] = gg[u] >= 0 ? roff[gg[u]] : 0;
          eb[u] = gg[u] >= 0 ? roff[gg[u] + 1] : 0;
        }
#pragma unroll
        for (int u = 0; u < kRelU; ++u)
#pragma unroll
          for (int q = 0; q < kRelE; ++q) rr[u][q] = ea[u] + q < eb[u] ? radj[ea[u] + q] : -1;
#pragma unroll
        for (int u = 0; u < kRelU; ++u) {
          if (gg[u] < 0) continue;
          const int ug = units ? blk_idx[lo + gg[u]] : -1;
#pragma unroll
          for (int q = 0; q < kRelE; ++q)
            if (rr[u][q] >= 0) release(rr[u][q], ug);
          for (int e = ea[u] + kRelE; e < eb[u]; ++e) release(radj[e], ug);
        }
      }
      __syncthreads();
    }
    if (err || placed == n) break;
    if (units) {
      err |= kErrCycle;
      break;
    }

    // ---- the unplaced ghosts (ascending) hold cycles
    int m = 0;
    for (int base = 0; base < n; base += 1024) {
      const int g = base + tid;
      const bool left = g < n && lev[lo + g] == 0;
      int64_t tot;
      const int64_t pre = block_excl_scan<1024>(left ? 1 : 0, &tot, sh);
      if (left && m + pre < kMaxResidual) res[m + pre] = g;
      m += (int)tot;
    }
    if (m > kMaxResidual) {   // workspace capacity, not a property of the graph
      err |= kErrUnsupported;
      break;
    }
    const int RW = (m + 31) / 32;
    for (int t = tid; t < m * RW; t += 1024) reach[t] = 0;
    __syncthreads();
    for (int u = tid; u < m; u += 1024) {
      for (int q = 0; q < np; ++q) {
        const int32_t d = deps[(int64_t)q * cap + lo + res[u]];
        if (d >= 0 && lev[d] == 0) {
          const int v = (int)find_sorted(res, 0, m, (int)(d - lo));
          if (v >= 0) reach[u * RW + (v >> 5)] |= 1u << (v & 31);
        }
      }
    }
    __threadfence_block();
    __syncthreads();
    do {
      if (tid == 0) s_flag = 0;
      __syncthreads();
      int changed = 0;
      for (int u = tid; u < m; u += 1024) {
        for (int q = 0; q < np; ++q) {
          const int32_t d = deps[(int64_t)q * cap + lo + res[u]];
          if (d < 0 || lev[d] != 0) continue;
          const int v = (int)find_sorted(res, 0, m, (int)(d - lo));
          if (v < 0) continue;
          for (int w = 0; w < RW; ++w) {
            const uint32_t o = reach[u * RW + w], nw = o | reach[v * RW + w];
            if (nw != o) {
              reach[u * RW + w] = nw;
              changed = 1;
            }
          }
        }
      }
      if (changed) s_flag = 1;
      __threadfence_block();
      __syncthreads();
    } while (s_flag);
    // representative = smallest member of the group; -1 off cycles
    for (int u = tid; u < m; u += 1024) {
      int rp = -1;
      if ((reach[u * RW + (u >> 5)] >> (u & 31)) & 1u) {
        for (int v = 0; v < m; ++v)
          if (((reach[u * RW + (v >> 5)] >> (v & 31)) & 1u) &&
              ((reach[v * RW + (u >> 5)] >> (u & 31)) & 1u)) {
            rp = v;
            break;
          }
      }
      rep[u] = rp;
    }
    __syncthreads();
    {
      int off = 0;
      for (int base = 0; base < m; base += 1024) {
        const int u = base + tid;
        const bool isrep = u < m && rep[u] == u;
        int64_t tot;
        const int64_t pre = block_excl_scan<1024>(isrep ? 1 : 0, &tot, sh);
        if (isrep) slot[u] = off + (int)pre;
        off += (int)tot;
      }
      if (tid == 0) s_units = off;
    }
    __syncthreads();
    if (s_units > kMaxUnits) {
      err |= kErrUnsupported;
      break;
    }
    for (int u = tid; u < m; u += 1024) {
      const int rp = rep[u];
      if (rp < 0) continue;
      int rank = 0, size = 0;
      for (int v = 0; v < m; ++v)
        if (rep[v] == rp) {
          if (v < u) ++rank;
          ++size;
        }
      if (size > kMaxUnit) {   // larger than the LDS solve's workspace
        atomicOr(&L.info[ii].err, kErrUnsupported);
        continue;
      }
      const int sl = slot[rp];
      unit_mem[sl * kMaxUnit + rank] = (int32_t)(lo + res[u]);
      blk_idx[lo + res[u]] = sl;
      if (u == rp) {
        unit_cnt[sl] = size;
        atomicMax(&s_maxunit, size);
      }
    }
    __syncthreads();
    if (L.info[ii].err & kErrUnsupported) break;
    units = true;   // restart the layering with the units as nodes
  }
  if (tid == 0) {
    if (err) atomicOr(&L.info[ii].err, err);
    L.info[ii].nlev = k;
    L.info[ii].maxwidth = maxwidth;
    L.info[ii].nunits = units ? s_units : 0;
    L.info[ii].maxunit = s_maxunit;
  }
}

bool levels_pull(int64_t max_n) { return max_n <= kPullMax && wave_residual() == kWaveResidual; }

template <int BS, int NP, int J>
static gcr_status launch_pull(const LevelsArgs& L, int ninst, int64_t n, hipStream_t st) {
  static std::mutex mu;
  static bool ready = false;
  const int bytes = (int)pull_lds(n, BS / 64);
  if (bytes > 65536) {
    std::lock_guard<std::mutex> lk(mu);
    if (!ready)
      GCR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_levels_pull<BS, NP, J>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)pull_lds(BS * J, BS / 64)));
    ready = true;
  }
  k_levels_pull<BS, NP, J><<<ninst, BS, bytes, st>>>(L, bytes);
  GCR_HIP(hipGetLastError());
  return GCR_OK;
}

// Small instances take a workgroup of four waves: its barriers are cheaper
// than sixteen waves' (128^2 circle, 99 ghosts: 8.2 us a launch against
// 9.7 for the push form).  Larger ones: as few ghosts a thread as the largest
// instance allows.
gcr_status launch_levels_pull(const LevelsArgs& L, int ninst, int64_t max_n, bool all_2d,
                              hipStream_t st) {
  const int64_t n = std::max<int64_t>(max_n, 1);
  if (all_2d) {
    if (n <= 1024) return launch_pull<256, 3, 4>(L, ninst, n, st);
    if (n <= 4096) return launch_pull<1024, 3, 4>(L, ninst, n, st);
    if (n <= 8192) return launch_pull<1024, 3, 8>(L, ninst, n, st);
    return launch_pull<1024, 3, 16>(L, ninst, n, st);
  }
  if (n <= 1024) return launch_pull<256, 7, 4>(L, ninst, n, st);
  if (n <= 4096) return launch_pull<1024, 7, 4>(L, ninst, n, st);
  if (n <= 8192) return launch_pull<1024, 7, 8>(L, ninst, n, st);
  return launch_pull<1024, 7, 16>(L, ninst, n, st);
}

// Counters and bitmap in LDS when the largest instance fits, else in HBM.
gcr_status launch_levels(const LevelsArgs& L, int ninst, int64_t max_n, hipStream_t st) {
  // device limits, taken once; the LDS attribute only grows, under the lock,
  // so builds on several host threads never launch beyond it
  static std::mutex mu;
  static int lds_max = -1;
  std::unique_lock<std::mutex> lk(mu);
  if (lds_max < 0) {
    int dev = 0, a = 0, b = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&a, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
      a = 0;
    if (hipDeviceGetAttribute(&b, hipDeviceAttributeSharedMemPerBlockOptin, dev) != hipSuccess)
      b = 0;
    (void)hipGetLastError();
    hipFuncAttributes fa{};
    int stat = 8192;
    if (hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(&k_levels<true, true>)) ==
        hipSuccess)
      stat = (int)fa.sharedSizeBytes;
    (void)hipGetLastError();
    lds_max = std::max(0, std::max(a, b) - stat - 256);
  }
  const int lds_avail = lds_max;
  lk.unlock();
  const int64_t nn = std::max<int64_t>(max_n, 1);
  const int64_t bytes = 4 * (((nn + 3) >> 2) + ((nn + 31) >> 5));
  LevelsArgs F = L;   // the one-workgroup layering
  {
    // the LDS layering first; k_levels below skips what it finished
    static int fast_lds = -1;
    lk.lock();
    if (fast_lds < 0) {
      int dev = 0, a = 0, b = 0;
      (void)hipGetDevice(&dev);
      if (hipDeviceGetAttribute(&a, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        a = 0;
      if (hipDeviceGetAttribute(&b, hipDeviceAttributeSharedMemPerBlockOptin, dev) != hipSuccess)
        b = 0;
      hipFuncAttributes fa{};
      int stat = 4096;
      if (hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(&k_levels_fast)) == hipSuccess)
        stat = (int)fa.sharedSizeBytes;
      (void)hipGetLastError();
      int v = std::max(0, std::max(a, b) - stat - 256) & ~255;
      if (v > 0 && hipFuncSetAttribute(reinterpret_cast<const void*>(&k_levels_fast),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, v) != hipSuccess) {
        (void)hipGetLastError();
        v = 0;
      }
      fast_lds = v;
    }
    const int fl = fast_lds;
    lk.unlock();
    if (fl > 0) k_levels_fast<<<ninst, 1024, (size_t)fl, st>>>(L, fl);
  }
  // what LDS is left holds the level list (worth it from a few thousand)
  const int64_t cur_cap =
      bytes <= lds_avail ? std::min<int64_t>(nn, (lds_avail - bytes) / 4) : 0;
  const int64_t bytes_cur = bytes + 4 * cur_cap;
  F.cur_cap = (int)cur_cap;
  if (cur_cap >= 2048) {
    static int64_t attr = 0;
    lk.lock();
    if (bytes_cur > attr) {
      GCR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_levels<true, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes_cur));
      attr = bytes_cur;
    }
    lk.unlock();
    k_levels<true, true><<<ninst, 1024, (size_t)bytes_cur, st>>>(F);
  } else if (bytes <= lds_avail) {
    static int64_t attr = 0;
    lk.lock();
    if (bytes > attr) {
      GCR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_levels<true, false>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
      attr = bytes;
    }
    lk.unlock();
    k_levels<true, false><<<ninst, 1024, (size_t)bytes, st>>>(F);
  } else {
    k_levels<false, false><<<ninst, 1024, 0, st>>>(F);
  }
  GCR_HIP(hipGetLastError());
  return GCR_OK;
}

}  // namespace gcr
