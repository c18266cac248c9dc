// adjoint.hip -- adjoints of the fill, the surface evaluation and the forces.
//
// The fill is affine: phi_G = ws b_G + sum_k w_k phi_{P_k}.  Its adjoint runs
// the levels in reverse, each ghost waiting for its readers' adjoints unless a
// schedule is forced.  Every value is produced by exactly one thread and
// every sum is taken in a fixed order, so results are bitwise reproducible.
// Both adjoints pull through the transposed stencil ("support"), built on
// the first adjoint call of a plan and kept with it: every cell that some
// ghost's stencil box touches gets a slot holding its readers (ghost,
// corner), sorted by (canonical ghost position, corner).  Then
//   * a ghost pulls w * lambda from the ghosts that read it (higher levels);
//   * a non-ghost cell sums all its readers once, in its own slot;
//   * a coupled unit solves its transposed system;
//   * the surface adjoint groups caller points by anchor ghost, forms
//     per-corner seeds in ascending point order, and each slot sums the seeds
//     of the anchors whose box holds it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "gcr_apply.hpp"
#include "gcr_fill.hpp"
#include "gcr_impl.hpp"

namespace gcr {

// Transposed stencil.  Entry = (reader << 4) | (corner << 1) | fill, with
// fill = 1 when the fill reads that corner (corner > 0, not skipped);
// corner 0 (the ghost's own cell) and skipped corners belong to the box the
// surface evaluation uses.
struct SupView {
  const int32_t* off;    // [bound + 1] slot -> first entry
  const int32_t* ent;    // [bound]
  const int32_t* cell;   // [bound] slot -> cell
  const int32_t* ghost;  // [bound] slot -> canonical ghost position or -1
  const int32_t* gslot;  // [ng] ghost -> slot of its own cell
  const int32_t* nslot;  // device count of slots
  int64_t bound;         // ng << dim
};

constexpr uint32_t kSupEmpty = 0xffffffffu;

__device__ __forceinline__ uint32_t sup_hash(uint32_t c) {
  uint32_t h = c * 2654435761u;
  return h ^ (h >> 15);
}

struct SupBuild {
  PlanD P;
  uint32_t* key;
  int32_t* val;
  uint32_t hmask;
  int32_t* nslot;
  int32_t* cnt;
  int32_t* off;
  int32_t* fillc;
  int32_t* ent;
  int32_t* cell;
  int32_t* ghost;
  int32_t* gslot;
  int64_t bound;
};

__device__ __forceinline__ int sup_find(const SupBuild& B, uint32_t q) {
  uint32_t h = sup_hash(q) & B.hmask;
  for (;;) {
    const uint32_t k = B.key[h];
    if (k == q) return B.val[h];
    if (k == kSupEmpty) return -1;
    h = (h + 1) & B.hmask;
  }
}

// corner m of ghost p, or -1 off the grid
template <int D>
__device__ __forceinline__ int sup_corner(const PlanD& P, int p, int m, uint32_t& code) {
  code = P.code[p];
  const int c = P.cell[p];
  int i, j, k;
  unlinear(P.g, c, i, j, k);
  if (!corner_in_grid(P.g, code, i, j, k, m)) return -1;
  return c + corner_offset(P.g, code, m);
}

__global__ void k_sup_clear(SupBuild B) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t <= (int64_t)B.hmask) B.key[t] = kSupEmpty;
  if (t < B.bound) {
    B.cnt[t] = 0;
    B.fillc[t] = 0;
    B.ghost[t] = -1;
  }
  if (t == 0) B.nslot[0] = 0;
}

template <int D>
__global__ __launch_bounds__(256) void k_sup_insert(SupBuild B) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= B.bound) return;
  const int p = (int)(t >> D), m = (int)(t & ((1 << D) - 1));
  uint32_t code;
  const int q = sup_corner<D>(B.P, p, m, code);
  if (q < 0) return;
  // the table holds at most `bound` keys in >= 2 * bound entries: a free
  // entry is always reached
  uint32_t h = sup_hash((uint32_t)q) & B.hmask;
  for (;;) {
    const uint32_t prev = atomicCAS(&B.key[h], kSupEmpty, (uint32_t)q);
    if (prev == kSupEmpty) {
      B.val[h] = atomicAdd(B.nslot, 1);
      return;
    }
    if (prev == (uint32_t)q) return;
    h = (h + 1) & B.hmask;
  }
}

template <int D>
__global__ __launch_bounds__(256) void k_sup_count(SupBuild B) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= B.bound) return;
  const int p = (int)(t >> D), m = (int)(t & ((1 << D) - 1));
  uint32_t code;
  const int q = sup_corner<D>(B.P, p, m, code);
  if (q < 0) return;
  const int s = sup_find(B, (uint32_t)q);
  if (s < 0) return;
  atomicAdd(&B.cnt[s], 1);
  B.cell[s] = q;
  if (m == 0) {
    B.ghost[s] = p;
    B.gslot[p] = s;
  }
}

template <int D>
__global__ __launch_bounds__(256) void k_sup_fill(SupBuild B) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= B.bound) return;
  const int p = (int)(t >> D), m = (int)(t & ((1 << D) - 1));
  uint32_t code;
  const int q = sup_corner<D>(B.P, p, m, code);
  if (q < 0) return;
  const int s = sup_find(B, (uint32_t)q);
  if (s < 0) return;
  const int fill = (m != 0 && !(m & code_skip(code))) ? 1 : 0;
  B.ent[B.off[s] + atomicAdd(&B.fillc[s], 1)] = (p << 4) | (m << 1) | fill;
}

// each slot's readers in ascending (ghost, corner) order
__global__ __launch_bounds__(256) void k_sup_sort(SupBuild B) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= B.bound || s >= B.nslot[0]) return;
  const int b = B.off[s], e = B.off[s + 1];
  for (int i = b + 1; i < e; ++i) {
    const int v = B.ent[i];
    int j = i - 1;
    while (j >= b && B.ent[j] > v) {
      B.ent[j + 1] = B.ent[j];
      --j;
    }
    B.ent[j + 1] = v;
  }
}

__global__ __launch_bounds__(1024) void k_sadj_scan(const int32_t* __restrict__ cnt, int n,
                                                    int32_t* __restrict__ off);

static inline unsigned nblk(int64_t n, int bs) { return (unsigned)std::max<int64_t>(1, (n + bs - 1) / bs); }

// Builds the transposed stencil of plan p on `st` (once; later calls reuse it).
static gcr_status plan_support(gcr_plan* p, hipStream_t st, SupView* out) {
  const int D = p->dim;
  const int64_t bound = p->ng << D;
  uint32_t H = 1;
  while ((int64_t)H < 2 * bound) H <<= 1;
  const size_t n32 = 2 * (size_t)H + 6 * (size_t)bound + 2 + (size_t)p->ng + 1;
  char* base = (char*)p->sup;
  if (!base) {
    base = (char*)pool_alloc(sizeof(int32_t) * n32);
    if (!base) return GCR_E_NOMEM;
    SupBuild B;
    std::memset(&B, 0, sizeof(B));
    B.P = plan_view(p);
    B.key = (uint32_t*)base;
    B.val = (int32_t*)(B.key + H);
    B.cnt = B.val + H;
    B.off = B.cnt + bound + 1;
    B.fillc = B.off + bound + 1;
    B.ent = B.fillc + bound;
    B.cell = B.ent + bound;
    B.ghost = B.cell + bound;
    B.gslot = B.ghost + bound;
    B.nslot = B.gslot + p->ng;
    B.hmask = H - 1;
    B.bound = bound;
    const int64_t nt = std::max<int64_t>((int64_t)H, bound);
    k_sup_clear<<<nblk(nt, 256), 256, 0, st>>>(B);
    if (D == 2) {
      k_sup_insert<2><<<nblk(bound, 256), 256, 0, st>>>(B);
      k_sup_count<2><<<nblk(bound, 256), 256, 0, st>>>(B);
    } else {
      k_sup_insert<3><<<nblk(bound, 256), 256, 0, st>>>(B);
      k_sup_count<3><<<nblk(bound, 256), 256, 0, st>>>(B);
    }
    k_sadj_scan<<<1, 1024, 0, st>>>(B.cnt, (int)bound, B.off);
    if (D == 2) k_sup_fill<2><<<nblk(bound, 256), 256, 0, st>>>(B);
    else k_sup_fill<3><<<nblk(bound, 256), 256, 0, st>>>(B);
    k_sup_sort<<<nblk(bound, 256), 256, 0, st>>>(B);
    GCR_HIP(hipGetLastError());
    p->sup = base;
    p->sup_bound = bound;
    p->sup_hmask = H - 1;
  }
  const uint32_t* key = (const uint32_t*)base;
  const int32_t* val = (const int32_t*)(key + (p->sup_hmask + 1));
  const int32_t* cnt = val + (p->sup_hmask + 1);
  out->off = cnt + bound + 1;
  const int32_t* fillc = out->off + bound + 1;
  out->ent = fillc + bound;
  out->cell = out->ent + bound;
  out->ghost = out->cell + bound;
  out->gslot = out->ghost + bound;
  out->nslot = out->gslot + p->ng;
  out->bound = bound;
  return GCR_OK;
}

// Fields that a thread takes together; one at a time where a caller passes
// one array for several fields, whose sums then follow each other.
static int field_group(int nf, double* const* lam) {
  for (int f = 0; f < nf; ++f)
    for (int g = 0; g < f; ++g)
      if (lam[f] == lam[g]) return 1;
  return std::min(nf, 4);
}

struct AdjArgs {
  PlanD P;
  int nf;
  int kind[kMaxFields];
  const uint8_t* bt[kMaxFields];
  double* lam[kMaxFields];     // dense, in/out
  double* lam_bc[kMaxFields];  // [ng]
  double* Lam;                 // [nf][ng] adjoint of each filled ghost value
  const double* w[2];          // the plan's cached weights per kind, [2^D][ng]
  SupView S;
};

template <int D>
__device__ __forceinline__ void weights_of(const PlanD& P, int g, int bc, double w[8]) {
  double dl[3], nn[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    dl[a] = a < D ? P.dl[a][g] : 0.0;
    nn[a] = a < D ? P.nn[a][g] : 0.0;
  }
  double X[3];
  stencil_span(P.g, P.code[g], P.cell[g], X);
  ghost_weights<D>(dl, nn, X, bc, w);
}

__device__ __forceinline__ int field_bc(const AdjArgs& A, int f, int g) {
  return A.kind[f] == 2 ? (int)A.bt[f][g] : A.kind[f];
}

// the weight of corner m in reader r's relation for field f
__device__ __forceinline__ double reader_weight(const AdjArgs& A, int f, int r, int m) {
  return (field_bc(A, f, r) == 0 ? A.w[0] : A.w[1])[(int64_t)m * A.P.ng + r];
}

// acc + w[corner] * Lam of each fill reader of slot s in field f, in entry
// order; readers inside unit `skip_unit` (>= 0) are left out.  With
// `left` given, each reader's value is waited for: false once *left polls
// have passed.
__device__ __forceinline__ bool pull_readers(const AdjArgs& A, int s, int skip_unit, int f,
                                             double& acc, int* left = nullptr) {
  const PlanD& P = A.P;
  const int b = A.S.off[s], e = A.S.off[s + 1];
  const double* const L = A.Lam + (int64_t)f * P.ng;
  for (int t = b; t < e; ++t) {
    const int en = A.S.ent[t];
    if (!(en & 1)) continue;
    const int r = en >> 4, m = (en >> 1) & 7;
    if (skip_unit >= 0 && P.blk[r] == skip_unit) continue;
    double v;
    if (left) {
      unsigned long long x;
      while ((x = poll_value(L + r)) == kFillOpen)
        if ((*left)-- <= 0) return false;
      v = __longlong_as_double((long long)x);
    } else {
      v = L[r];
    }
    acc += reader_weight(A, f, r, m) * v;
  }
  return true;
}

// Adjoint of coupled unit u in field f: (I - W_int)^T mu = lam + external
// pulls, solved in an LDS workspace (one unit per thread); false where a wait
// gave up.
template <int D>
__device__ __forceinline__ bool adj_unit(const AdjArgs& A, int u, int f, UnitWS& ws,
                                         int* left = nullptr) {
  const PlanD& P = A.P;
  const int k = P.unit_cnt[u];
  for (int i = 0; i < k; ++i) {
    ws.mem[i] = P.unit_mem[u * kMaxUnit + i];
    ws.cel[i] = P.cell[ws.mem[i]];
  }
  // transposed matrix directly: M[t][i] = delta - w(i reads t)
  for (int i = 0; i < k * k; ++i) ws.M[i] = 0.0;
  for (int i = 0; i < k; ++i) {
    ws.M[i * k + i] = 1.0;
    double acc = 0.0;
    if (!pull_readers(A, A.S.gslot[ws.mem[i]], u, f, acc, left)) return false;
    ws.rhs[i] = A.lam[f][ws.cel[i]] + acc;
  }
  for (int i = 0; i < k; ++i) {
    double w[8];
    weights_of<D>(P, ws.mem[i], field_bc(A, f, ws.mem[i]), w);
    const uint32_t code = P.code[ws.mem[i]];
    for (int c = 1; c < (1 << D); ++c) {
      if (c & code_skip(code)) continue;
      const int q = ws.cel[i] + corner_offset(P.g, code, c);
      for (int t = 0; t < k; ++t)
        if (ws.cel[t] == q) ws.M[t * k + i] -= w[c];
    }
  }
  ws_solve(ws, k);
  for (int i = 0; i < k; ++i) post_value(A.Lam + (int64_t)f * P.ng + ws.mem[i], ws.rhs[i]);
  return true;
}

template <int D>
__device__ __forceinline__ void adj_units_of_level(const AdjArgs& A, int level, UnitWS* ws,
                                                   int tid, int nthreads) {
  for (int s = tid; s < A.P.nunits; s += nthreads)
    if (A.P.unit_lev[s] == level)
      for (int f = 0; f < A.nf; ++f) adj_unit<D>(A, s, f, ws[tid]);
}

__device__ __forceinline__ void adj_ghost(const AdjArgs& A, int p, int f) {
  const PlanD& P = A.P;
  if (P.blk[p] >= 0) return;   // coupled units: adj_units_of_level
  double acc = A.lam[f][P.cell[p]];
  pull_readers(A, A.S.gslot[p], -1, f, acc);
  A.Lam[(int64_t)f * P.ng + p] = fill_result(acc);
}

__global__ __launch_bounds__(256) void k_adj_range(AdjArgs A, int lo, int hi) {
  const int p = lo + blockIdx.x * blockDim.x + threadIdx.x;
  if (p < hi) adj_ghost(A, p, blockIdx.y);
}

// The whole sweep by one workgroup; with `fault` given, only where it is set.
template <int D>
__global__ __launch_bounds__(256) void k_adj_wg(AdjArgs A, const int32_t* __restrict__ lev_off,
                                                int nlev, const int32_t* __restrict__ fault) {
  __shared__ UnitWS ws[64];
  if (fault && fault[0] == 0) return;   // uniform
  for (int l = nlev - 1; l >= 0; --l) {
    const int lo = lev_off[l], n = (lev_off[l + 1] - lo) * A.nf;
    for (int e = (int)threadIdx.x; e < n; e += blockDim.x) adj_ghost(A, lo + e / A.nf, e % A.nf);
    __syncthreads();
    if (A.P.nunits) {
      if (threadIdx.x < 64) adj_units_of_level<D>(A, l + 1, ws, threadIdx.x, 64);
      __syncthreads();
    }
  }
}

template <int D>
__global__ __launch_bounds__(64) void k_adj_units(AdjArgs A, int level) {
  __shared__ UnitWS ws[64];
  adj_units_of_level<D>(A, level, ws, threadIdx.x, 64);
}

// --------------------------------------------------------------------------
// The sweep by waiting, as the fill's (k_fill_flow): k_adj_open marks every
// ghost's adjoint open, then one thread per ghost and field, the last level
// first, polls the adjoints of the ghosts that read it and stores its own.
// Readers lie in later levels, so workgroups wait for earlier ones; their
// entries and weights are gathered eight at a time before the first poll, and
// summed in entry order.  A coupled unit is one thread's, four to a workgroup,
// and those workgroups lead the grid: they wait for later ones, but fill a
// corner of the chip at most.  Waits are bounded as the fill's are; a thread
// that passes the bound computes what it waits for (adj_help), or, in a plan
// with coupled units, sets the plan's fault word (k_adj_open clears it), for
// k_adj_wg to sweep this call again.
// Bound by the chain of levels.  160^3 spherical-harmonic body, four fields,
// ten levels: 20 us for the two launches against 90 for ten.
// --------------------------------------------------------------------------
constexpr int kAdjUnitsPerBlock = 4;

__global__ __launch_bounds__(256) void k_adj_open(double* __restrict__ Lam, int64_t n,
                                                  int32_t* __restrict__ fault) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0) fault[0] = 0;
  if (i < n) Lam[i] = __longlong_as_double((long long)kFillOpen);
}

// The adjoint of ghost p in field f, posted, without waiting (as fill_help:
// down to a reader that is open, until one has all of its own).  Plans without
// coupled units.
__device__ __forceinline__ void adj_help(const AdjArgs& A, int p, int f) {
  const PlanD& P = A.P;
  double* const L = A.Lam + (int64_t)f * P.ng;
  for (int cur = p;;) {
    const int s = A.S.gslot[cur], e = A.S.off[s + 1];
    double acc = A.lam[f][P.cell[cur]];
    int open = -1;
    for (int t = A.S.off[s]; t < e && open < 0; ++t) {
      const int en = A.S.ent[t], r = en >> 4;
      if (!(en & 1)) continue;
      const unsigned long long x = poll_value(L + r);
      if (x == kFillOpen) open = r;
      else acc += reader_weight(A, f, r, (en >> 1) & 7) * __longlong_as_double((long long)x);
    }
    if (open >= 0) {
      cur = open;
      continue;
    }
    post_value(L + cur, acc);
    if (cur == p) return;
    cur = p;
  }
}

template <int D>
__global__ __launch_bounds__(256) void k_adj_flow(AdjArgs A, int unit_blocks, int polls) {
  __shared__ UnitWS ws[kAdjUnitsPerBlock];
  const PlanD& P = A.P;
  const int f = blockIdx.y;
  if ((int)blockIdx.x < unit_blocks) {
    const int wave = threadIdx.x >> 6, u = blockIdx.x * kAdjUnitsPerBlock + wave;
    int left = polls;
    if ((threadIdx.x & 63) == 0 && u < P.nunits && !adj_unit<D>(A, u, f, ws[wave], &left))
      atomicOr(P.fill_fault, 1);
    return;
  }
  // (past the first ghost: that one again)
  const int p = max(P.ng - 1 - (int)((blockIdx.x - unit_blocks) * 256 + threadIdx.x), 0);
  double* const L = A.Lam + (int64_t)f * P.ng;
  const int s = A.S.gslot[p];
  bool done = P.blk[p] >= 0;
  double acc = A.lam[f][P.cell[p]];
  int t = A.S.off[s];
  const int e = A.S.off[s + 1];
  double w[8], val[8];
  int r[8];
  uint32_t use = 0, open = 0;
  bool fetch = true;
  for (int left = polls;; --left) {
    if (!done) {
      if (fetch) {
        use = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int en = t + j < e ? A.S.ent[t + j] : 0;
          r[j] = en >> 4;
          use |= (uint32_t)(en & 1) << j;
          // (an entry that is not read: any weight of ghost r)
          w[j] = reader_weight(A, f, r[j], (en >> 1) & ((1 << D) - 1));
        }
        open = use;
        fetch = false;
      }
      unsigned long long x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = (open >> j) & 1u ? poll_value(L + r[j]) : kFillOpen;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (x[j] != kFillOpen) {
          val[j] = __longlong_as_double((long long)x[j]);
          open &= ~(1u << j);
        }
      if (!open) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if ((use >> j) & 1u) acc += w[j] * val[j];
        t += 8;
        fetch = true;
        if (t >= e) {
          post_value(L + p, acc);
          done = true;
        }
      }
    }
    if (__ballot(!done) == 0ull) return;
    if (left <= 0) {
      if (!done && P.nunits == 0) adj_help(A, p, f);
      else if (!done) atomicOr(P.fill_fault, 1);
      return;
    }
  }
}

template <int D>
static void adj_flow(const AdjArgs& A, const int32_t* d_lev_off, int nlev, hipStream_t st) {
  const int64_t n = (int64_t)A.nf * A.P.ng;
  const int ub = (A.P.nunits + kAdjUnitsPerBlock - 1) / kAdjUnitsPerBlock;
  k_adj_open<<<nblk(n, 256), 256, 0, st>>>(A.Lam, n, A.P.fill_fault);
  k_adj_flow<D><<<dim3((unsigned)ub + nblk(A.P.ng, 256), (unsigned)A.nf), 256, 0, st>>>(
      A, ub, fill_polls());
  if (ub) k_adj_wg<D><<<1, 256, 0, st>>>(A, d_lev_off, nlev, A.P.fill_fault);
}

// Per slot: a ghost's own cell gives its boundary-data sensitivity and is
// zeroed (the fill overwrites it); a non-ghost cell sums its readers once.
// Eight entries are read at a time and NF fields together (field_group); bound
// by the scattered cells it reads and writes (160^3, four fields, 25,000
// slots: 18 us, 100,000 cells of distinct lines).
template <int D, int NF>
__global__ __launch_bounds__(256) void k_adj_support(AdjArgs A) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= A.S.bound || s >= A.S.nslot[0]) return;
  const PlanD& P = A.P;
  const int q = A.S.cell[s];
  const int p = A.S.ghost[s];
  if (p >= 0) {
    for (int f0 = 0; f0 < A.nf; f0 += NF) {
      double v[NF];
#pragma unroll
      for (int g = 0; g < NF; ++g) {
        const int f = min(f0 + g, A.nf - 1);
        v[g] = reader_weight(A, f, p, 0) * A.Lam[(int64_t)f * P.ng + p];
      }
#pragma unroll
      for (int g = 0; g < NF; ++g)
        if (f0 + g < A.nf) {
          A.lam_bc[f0 + g][p] = v[g];
          A.lam[f0 + g][q] = 0.0;
        }
    }
    return;
  }
  const int b = A.S.off[s], e = A.S.off[s + 1];
  for (int f0 = 0; f0 < A.nf; f0 += NF) {
    double acc[NF], was[NF];
#pragma unroll
    for (int g = 0; g < NF; ++g) {
      acc[g] = 0.0;
      was[g] = A.lam[min(f0 + g, A.nf - 1)][q];
    }
    bool any = false;
    for (int t = b; t < e; t += 8) {
      int r[8], m[8];
      uint32_t use = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int en = t + j < e ? A.S.ent[t + j] : 0;
        r[j] = en >> 4;
        m[j] = (en >> 1) & ((1 << D) - 1);
        use |= (uint32_t)(en & 1) << j;
      }
      any |= use != 0;
#pragma unroll
      for (int g = 0; g < NF; ++g) {
        const int f = min(f0 + g, A.nf - 1);
        double w[8], v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          w[j] = reader_weight(A, f, r[j], m[j]);
          v[j] = A.Lam[(int64_t)f * P.ng + r[j]];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if ((use >> j) & 1u) acc[g] += w[j] * v[j];
      }
    }
    if (!any) return;
#pragma unroll
    for (int g = 0; g < NF; ++g)
      if (f0 + g < A.nf) A.lam[f0 + g][q] = was[g] + acc[g];
  }
}

template <int D>
static void adj_support(const AdjArgs& A, hipStream_t st) {
  const unsigned nb = nblk(A.S.bound, 256);
  const int n = field_group(A.nf, A.lam);
  if (n == 1) k_adj_support<D, 1><<<nb, 256, 0, st>>>(A);
  else if (n == 2) k_adj_support<D, 2><<<nb, 256, 0, st>>>(A);
  else if (n == 3) k_adj_support<D, 3><<<nb, 256, 0, st>>>(A);
  else k_adj_support<D, 4><<<nb, 256, 0, st>>>(A);
}

// --------------------------------------------------------------------------
// surface adjoint
// --------------------------------------------------------------------------

struct SurfAdjArgs {
  PlanD P;
  int nf;
  int64_t nq;
  const double* xq;
  const double* gval;    // [nf][nq] or null
  const double* ggrad;   // [nf][dim][nq] or null
  double* lam[kMaxFields];
  const double *nrm, *wq, *gF;   // the force's instead of gval, ggrad, or null
  double mu;
  int32_t* anchor;       // [nq]
  int32_t* rank;         // [nq] place of the point among its anchor's
  int32_t* cnt;          // [ng + 1] points per anchor; [ng]: places given out
  int32_t* off;          // [ng] first place of an anchor's points
  int32_t* bucket;       // [nq]
  int32_t* sorted;       // [nf][nq] the points of anchors with many, ascending
  double* seed;          // [nf][8][ng]
  SupView Sp;
};

__global__ void k_zero_i32(int32_t* __restrict__ a, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0;
}

template <int D>
__global__ __launch_bounds__(256) void k_sadj_anchor(SurfAdjArgs S) {
  constexpr int NL = anchor_lanes<D>();
  const int sub = (int)threadIdx.x % NL;
  const int64_t q = (int64_t)blockIdx.x * (256 / NL) + threadIdx.x / NL;
  const bool active = q < S.nq;
  double x[3] = {0.0, 0.0, 0.0};
  if (active)
#pragma unroll
    for (int a = 0; a < D; ++a) x[a] = S.xq[a * S.nq + q];
  const int g = find_anchor_group<D, NL>(S.P, x, sub, active);
  if (!active || sub != 0) return;
  S.anchor[q] = g;
  if (g >= 0) S.rank[q] = atomicAdd(&S.cnt[g], 1);
}

// Places for each anchor's points.  Which anchor's come first does not matter,
// so a wave takes its ghosts' total from one counter; a scan over all ghosts
// by one workgroup took 9 us at 7,000.
__global__ __launch_bounds__(256) void k_sadj_place(SurfAdjArgs S) {
  const int g = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63;
  const int c = g < S.P.ng ? S.cnt[g] : 0;
  int sum = c;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(sum, d);
    if (lane >= d) sum += o;
  }
  int base = 0;
  if (lane == 63 && sum) base = atomicAdd(&S.cnt[S.P.ng], sum);
  base = __shfl(base, 63);
  if (g < S.P.ng) S.off[g] = base + sum - c;
}

// exclusive scan of n counts (one workgroup)
__global__ __launch_bounds__(1024) void k_sadj_scan(const int32_t* __restrict__ cnt, int n,
                                                    int32_t* __restrict__ off) {
  __shared__ int64_t sh[17];
  block_scan_i32(cnt, n, off, sh);
}

__global__ __launch_bounds__(256) void k_sadj_bucket(SurfAdjArgs S) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= S.nq) return;
  const int g = S.anchor[q];
  if (g >= 0) S.bucket[S.off[g] + S.rank[q]] = (int32_t)q;
}

// Cotangents of field f's value and gradient at point q: the caller's, or
// those of J = gF . F, where per point d J / d p = -w (gF . n) and
// d J / d (d u_i / d x_j) = mu w (gF_i n_j + gF_j n_i); p is field 0.
template <int D, bool FORCE>
__device__ __forceinline__ void cotangents(const SurfAdjArgs& S, int f, int64_t q, double& gv,
                                           double gg[3]) {
  gv = 0.0;
  gg[0] = gg[1] = gg[2] = 0.0;
  if (!FORCE) {
    if (S.gval) gv = S.gval[(int64_t)f * S.nq + q];
    if (S.ggrad)
#pragma unroll
      for (int a = 0; a < D; ++a) gg[a] = S.ggrad[((int64_t)f * D + a) * S.nq + q];
    return;
  }
  double n[3], g[3];
#pragma unroll
  for (int a = 0; a < D; ++a) {
    n[a] = S.nrm[a * S.nq + q];
    g[a] = S.gF[a];
  }
  const double w = S.wq[q];
  if (f == 0) {
    double gn = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) gn += g[a] * n[a];
    gv = -w * gn;
    return;
  }
  double gi = g[0], ni = n[0];
#pragma unroll
  for (int a = 1; a < D; ++a)
    if (f == 1 + a) {
      gi = g[a];
      ni = n[a];
    }
#pragma unroll
  for (int j = 0; j < D; ++j) gg[j] = S.mu * w * (gi * n[j] + g[j] * ni);
}

// per anchor and field, over its points in ascending index: the seeds
// seed[f][corner][g] = sum_q coef(corner, x_q) . (gval, ggrad).  The next
// index is searched among an anchor's few points; nothing is moved, so the
// fields' threads share the bucket.  Beyond kSeedFew the search would take
// longer than the sum (it grows with the square: 2,048 points at one anchor
// 280 ms), so there the wave first ranks the points, 64 lanes at a time, into
// the field's own list: 1.7 ms.
constexpr int kSeedFew = 32;

template <int D, bool FORCE>
__global__ __launch_bounds__(256) void k_sadj_seed(SurfAdjArgs S) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x, f = blockIdx.y, lane = threadIdx.x & 63;
  const PlanD& P = S.P;
  const int n = g < P.ng ? S.cnt[g] : 0, off = n ? S.off[g] : 0;
  int32_t* const sorted = S.sorted + (int64_t)f * S.nq;
  for (unsigned long long many = __ballot(n > kSeedFew); many; many &= many - 1ull) {   // uniform
    const int src = __ffsll((long long)many) - 1;
    const int m = __builtin_amdgcn_readlane(n, src), o = __builtin_amdgcn_readlane(off, src);
    const int32_t* const from = S.bucket + o;
    constexpr int kOwn = 4;
    for (int t0 = 0; t0 < m; t0 += 64 * kOwn) {
      int v[kOwn], rank[kOwn];
#pragma unroll
      for (int u = 0; u < kOwn; ++u) {
        const int t = t0 + 64 * u + lane;
        v[u] = t < m ? from[t] : 0;
        rank[u] = 0;
      }
      for (int j = 0; j < m; j += 64) {
        const int e = j + lane < m ? from[j + lane] : 0x7fffffff;   // (below no index)
#pragma unroll
        for (int k = 0; k < 64; ++k) {
          const int x = __builtin_amdgcn_readlane(e, k);
#pragma unroll
          for (int u = 0; u < kOwn; ++u) rank[u] += x < v[u] ? 1 : 0;
        }
      }
#pragma unroll
      for (int u = 0; u < kOwn; ++u)
        if (t0 + 64 * u + lane < m) sorted[o + rank[u]] = v[u];
    }
  }
  __threadfence_block();   // the lists, before their anchors' lanes read them
  if (n == 0) return;
  const int32_t* const bucket = (n > kSeedFew ? sorted : S.bucket) + off;
  const uint32_t code = P.code[g];
  int i, j, k;
  unlinear(P.g, P.cell[g], i, j, k);
  const int ijk[3] = {i, j, k};
  double X[3];
  stencil_span(P.g, code, P.cell[g], X);
  double acc[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) acc[m] = 0.0;
  int32_t last = -1;
  for (int t = 0; t < n; ++t) {
    int32_t q = 0x7fffffff;
    if (n > kSeedFew) q = bucket[t];
    else
      for (int u = 0; u < n; ++u) {
        const int32_t c = bucket[u];
        if (c > last && c < q) q = c;
      }
    last = q;
    double rel[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < D; ++a) rel[a] = S.xq[a * S.nq + q] - centre(P.g, a, ijk[a]);
    double gv, gg[3];
    cotangents<D, FORCE>(S, f, q, gv, gg);
#pragma unroll
    for (int m = 0; m < (1 << D); ++m) {
      double cv, cg[3];
      box_coeffs<D>(rel, X, m, cv, cg);
      double s = cv * gv;
#pragma unroll
      for (int a = 0; a < D; ++a) s += cg[a] * gg[a];
      acc[m] += s;
    }
  }
#pragma unroll
  for (int m = 0; m < (1 << D); ++m) S.seed[((int64_t)f * 8 + m) * P.ng + g] = acc[m];
}

// each slot: the seeds of every anchor whose box holds its cell, in entry
// order (ghosts that anchor no point have no seeds).  Bound by the chain
// entry -> count -> seed: eight entries at a time, NF fields together
// (field_group).  160^3, four fields, 2,048 points: 9.4 us, entry by entry 17.
template <int NF>
__global__ __launch_bounds__(256) void k_sadj_pull(SurfAdjArgs S) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S.Sp.bound || s >= S.Sp.nslot[0]) return;
  const int64_t ng = S.P.ng;
  const int b = S.Sp.off[s], e = S.Sp.off[s + 1];
  const int q = S.Sp.cell[s];
  for (int f0 = 0; f0 < S.nf; f0 += NF) {
    double acc[NF], was[NF];
#pragma unroll
    for (int g = 0; g < NF; ++g) {
      acc[g] = 0.0;
      was[g] = S.lam[min(f0 + g, S.nf - 1)][q];
    }
    bool any = false;
    for (int t = b; t < e; t += 8) {
      int r[8], m[8], c[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int en = t + j < e ? S.Sp.ent[t + j] : -1;
        r[j] = max(en >> 4, 0);
        m[j] = (en >> 1) & 7;
        c[j] = en < 0 ? -1 : 0;
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) c[j] = c[j] < 0 ? 0 : S.cnt[r[j]];
#pragma unroll
      for (int g = 0; g < NF; ++g) {
        const int f = min(f0 + g, S.nf - 1);
        double v[8];   // (of no meaning where an anchor has no points)
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = S.seed[((int64_t)f * 8 + m[j]) * ng + r[j]];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (c[j] != 0) {
            any = true;
            acc[g] += v[j];
          }
      }
    }
    if (!any) return;
#pragma unroll
    for (int g = 0; g < NF; ++g)
      if (f0 + g < S.nf) S.lam[f0 + g][q] = was[g] + acc[g];
  }
}

// S: fields, points and cotangents set
static gcr_status surface_adjoint_impl(gcr_plan* p, SurfAdjArgs S, double* const* lam,
                                       hipStream_t st) {
  const int64_t ng = p->ng, nq = S.nq;
  if (nq == 0 || ng == 0) return GCR_OK;
  S.P = plan_view(p);
  for (int f = 0; f < S.nf; ++f) S.lam[f] = lam[f];
  {
    const gcr_status ss = plan_support(p, st, &S.Sp);
    if (ss != GCR_OK) return ss;
  }
  int32_t* ib = (int32_t*)plan_scratch(p, 1, sizeof(int32_t) * ((3 + S.nf) * nq + 2 * (ng + 1)));
  S.seed = (double*)plan_scratch(p, 2, sizeof(double) * (size_t)S.nf * 8 * ng);
  if (!ib || !S.seed) return GCR_E_NOMEM;
  S.anchor = ib;
  S.rank = S.anchor + nq;
  S.bucket = S.rank + nq;
  S.cnt = S.bucket + nq;
  S.off = S.cnt + (ng + 1);
  S.sorted = S.off + (ng + 1);
  k_zero_i32<<<nblk(ng + 1, 256), 256, 0, st>>>(S.cnt, ng + 1);
  const int D = p->dim;
  const unsigned nba = (unsigned)force_blocks(D, nq);
  if (D == 2) k_sadj_anchor<2><<<nba, 256, 0, st>>>(S);
  else k_sadj_anchor<3><<<nba, 256, 0, st>>>(S);
  k_sadj_place<<<nblk(ng, 256), 256, 0, st>>>(S);
  k_sadj_bucket<<<nblk(nq, 256), 256, 0, st>>>(S);
  const dim3 gs(nblk(ng, 256), (unsigned)S.nf);
  if (D == 2) {
    if (S.gF) k_sadj_seed<2, true><<<gs, 256, 0, st>>>(S);
    else k_sadj_seed<2, false><<<gs, 256, 0, st>>>(S);
  } else {
    if (S.gF) k_sadj_seed<3, true><<<gs, 256, 0, st>>>(S);
    else k_sadj_seed<3, false><<<gs, 256, 0, st>>>(S);
  }
  const unsigned nbp = nblk(S.Sp.bound, 256);
  const int n = field_group(S.nf, S.lam);
  if (n == 1) k_sadj_pull<1><<<nbp, 256, 0, st>>>(S);
  else if (n == 2) k_sadj_pull<2><<<nbp, 256, 0, st>>>(S);
  else if (n == 3) k_sadj_pull<3><<<nbp, 256, 0, st>>>(S);
  else k_sadj_pull<4><<<nbp, 256, 0, st>>>(S);
  GCR_HIP(hipGetLastError());
  return GCR_OK;
}

static bool nonnull(int n, const void* const* a) {
  if (!a || n < 1 || n > kMaxFields) return false;
  for (int i = 0; i < n; ++i)
    if (!a[i]) return false;
  return true;
}

}  // namespace gcr

using namespace gcr;

extern "C" {

gcr_status gcr_surface_adjoint(const gcr_plan* plan, int64_t nq, const double* xq, int32_t nf,
                               const double* gval, const double* ggrad, double* const* lam,
                               void* stream) {
  if (!plan_ok(plan) || nq < 0 || (nq > 0 && !xq) || !nonnull(nf, (const void* const*)lam))
    return GCR_E_ARG;
  if (nq >= (int64_t(1) << 31)) return GCR_E_UNSUPPORTED;
  SurfAdjArgs S;
  std::memset(&S, 0, sizeof(S));
  S.nf = nf;
  S.nq = nq;
  S.xq = xq;
  S.gval = gval;
  S.ggrad = ggrad;
  return surface_adjoint_impl(const_cast<gcr_plan*>(plan), S, lam, (hipStream_t)stream);
}

gcr_status gcr_forces_adjoint(const gcr_plan* plan, int64_t nq, const double* xq,
                              const double* nrm, const double* wq, double mu, const double* gF,
                              double* lam_p, double* const* lam_u, void* stream) {
  if (!plan_ok(plan) || nq < 0 || !gF || !lam_p || !lam_u) return GCR_E_ARG;
  if (nq > 0 && (!xq || !nrm || !wq)) return GCR_E_ARG;
  const int d = plan->dim;
  for (int a = 0; a < d; ++a)
    if (!lam_u[a]) return GCR_E_ARG;
  if (nq == 0) return GCR_OK;
  if (nq >= (int64_t(1) << 31)) return GCR_E_UNSUPPORTED;
  gcr_plan* p = const_cast<gcr_plan*>(plan);
  SurfAdjArgs S;
  std::memset(&S, 0, sizeof(S));
  S.nf = 1 + d;
  S.nq = nq;
  S.xq = xq;
  S.nrm = nrm;
  S.wq = wq;
  S.gF = gF;
  S.mu = mu;
  double* lam[4] = {lam_p, lam_u[0], lam_u[1], d == 3 ? lam_u[2] : nullptr};
  return surface_adjoint_impl(p, S, lam, (hipStream_t)stream);
}

gcr_status gcr_fill_adjoint(const gcr_plan* plan, int32_t nf, double* const* lam,
                            const int32_t* bc_kind, const uint8_t* const* bc_type,
                            double* const* lam_bc, void* stream) {
  gcr::touch_thread_storage();   // (autograd calls this from a thread of its own)
  if (!plan_ok(plan) || !nonnull(nf, (const void* const*)lam) || !bc_kind ||
      !nonnull(nf, (const void* const*)lam_bc))
    return GCR_E_ARG;
  gcr_plan* p = const_cast<gcr_plan*>(plan);
  AdjArgs A;
  std::memset(&A, 0, sizeof(A));
  A.P = plan_view(p);
  A.nf = nf;
  for (int f = 0; f < nf; ++f) {
    if (bc_kind[f] < 0 || bc_kind[f] > 2) return GCR_E_ARG;
    if (bc_kind[f] == GCR_MIXED && (!bc_type || !bc_type[f])) return GCR_E_ARG;
    A.kind[f] = bc_kind[f];
    A.bt[f] = bc_kind[f] == GCR_MIXED ? bc_type[f] : nullptr;
    A.lam[f] = lam[f];
    A.lam_bc[f] = lam_bc[f];
  }
  const int64_t ng = p->ng;
  if (ng == 0) return GCR_OK;
  A.Lam = (double*)plan_scratch(p, 4, sizeof(double) * (size_t)nf * ng);
  if (!A.Lam) return GCR_E_NOMEM;
  hipStream_t st = (hipStream_t)stream;
  {
    const gcr_status ws = plan_weights(p, nf, A.kind, A.w, st);
    if (ws != GCR_OK) return ws;
  }
  {
    const gcr_status ss = plan_support(p, st, &A.S);
    if (ss != GCR_OK) return ss;
  }
  // As the fill: by waiting, or a forced schedule's one workgroup or launch
  // per level.  Up to two ghosts' fields to each lane one workgroup costs less
  // than the launch that opens the waits: 28 to 480 ghosts in at most 12
  // levels, one field, 10.8 to 24.0 us against 13.7 to 25.6.  It is the slower
  // one from 600 on (201 ghosts, four fields: 26.6 us against 25.7), in more
  // levels (267 ghosts in 17: 28.0 us against 25.0) and with a coupled unit,
  // which holds its lanes up (216 ghosts: 30.4 us against 25.0).
  const bool small = p->ng * nf <= 512 && p->nlev <= 12 && p->unit_lev_host.empty();
  if (p->schedule == kSchedAuto && !small) {
    if (p->dim == 2) adj_flow<2>(A, p->d_lev_off, p->nlev, st);
    else adj_flow<3>(A, p->d_lev_off, p->nlev, st);
  } else if (p->schedule == kSchedAuto || p->schedule == kSchedWorkgroup) {
    if (p->dim == 2) k_adj_wg<2><<<1, 256, 0, st>>>(A, p->d_lev_off, p->nlev, nullptr);
    else k_adj_wg<3><<<1, 256, 0, st>>>(A, p->d_lev_off, p->nlev, nullptr);
  } else {
    for (int l = p->nlev - 1; l >= 0; --l) {
      const int lo = p->lev_off[l], hi = p->lev_off[l + 1];
      k_adj_range<<<dim3(nblk(hi - lo, 256), (unsigned)nf), 256, 0, st>>>(A, lo, hi);
      for (int32_t ul : p->unit_lev_host)
        if (ul == l + 1) {
          if (p->dim == 2) k_adj_units<2><<<1, 64, 0, st>>>(A, l + 1);
          else k_adj_units<3><<<1, 64, 0, st>>>(A, l + 1);
          break;
        }
    }
  }
  if (p->dim == 2) adj_support<2>(A, st);
  else adj_support<3>(A, st);
  GCR_HIP(hipGetLastError());
  return GCR_OK;
}

}  // extern "C"
