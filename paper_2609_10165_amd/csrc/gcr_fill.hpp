// gcr_fill.hpp -- per-ghost fill of the level-by-level reconstruction
// (relations of Sec. 4.1 / 5.1 in tensor-product form), shared by the
// single-plan and batched kernels.  Ghosts that belong to a coupled unit are
// skipped by the per-ghost path and solved together afterwards, one unit per
// thread, in an LDS workspace.
#pragma once

#include "gcr_apply.hpp"

namespace gcr {

// One field of coupled unit u: (I - W_int) phi = W_ext phi_ext + ws b.  Apart:
// as stencil_span's.
template <int D, bool Apart = false>
__device__ __forceinline__ void fill_unit_field(const PlanD& P, int u, double* F,
                                                const double* b, const uint8_t* bt, int kind,
                                                UnitWS& ws) {
  const int k = P.unit_cnt[u];
  for (int i = 0; i < k; ++i) {
    ws.mem[i] = P.unit_mem[u * kMaxUnit + i];
    ws.cel[i] = P.cell[ws.mem[i]];
  }
  for (int i = 0; i < k; ++i) {
    const int p = ws.mem[i];
    const uint32_t code = P.code[p];
    const uint32_t skip = code_skip(code);
    double dl[3], nn[3], w[8];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      dl[a] = a < D ? P.dl[a][p] : 0.0;
      nn[a] = a < D ? P.nn[a][p] : 0.0;
    }
    const int bc = kind == 2 ? (int)bt[p] : kind;
    double X[3];
    stencil_span<Apart>(P.g, code, ws.cel[i], X);
    ghost_weights<D>(dl, nn, X, bc, w);
    for (int t = 0; t < k; ++t) ws.M[i * k + t] = (t == i) ? 1.0 : 0.0;
    double r = w[0] * b[p];
#pragma unroll
    for (int c = 1; c < (1 << D); ++c) {
      if (c & skip) continue;
      const int q = ws.cel[i] + corner_offset(P.g, code, c);
      int t = -1;
      for (int s = 0; s < k; ++s)
        if (ws.cel[s] == q) t = s;
      if (t >= 0) ws.M[i * k + t] -= w[c];
      else r += w[c] * F[q];
    }
    ws.rhs[i] = r;
  }
  ws_solve(ws, k);
  for (int i = 0; i < k; ++i) F[ws.cel[i]] = ws.rhs[i];
}

// Loads are ordered so that each ghost costs two dependent round trips:
// first its metadata, boundary data and cached weights (none depends on
// another load), then its stencil corners; all stores come last.  A ghost of
// level k reads only fluid cells and ghosts of lower levels, never a slot
// that this launch writes, so this order is exact.  (The compiler cannot
// prove that on its own, since field and weight arrays could alias.)
// Ghosts of coupled units compute but do not store (their unit solve does).
constexpr int kFieldGroup = 4;

// Fields f0 .. f0 + kFieldGroup - 1 of ghost p (metadata already loaded).
template <int D>
__device__ __forceinline__ void fill_group(const FillArgs& A, int p, int f0, bool live, int c,
                                           uint32_t code) {
  const PlanD& P = A.P;
  const int ng = P.ng;
  const double* const W0 = A.w[0];
  const double* const W1 = A.w[1];
  int bc[kFieldGroup];
  double bv[kFieldGroup];
  // slots past nf load field nf - 1 again (never stored): no branches here
#pragma unroll
  for (int j = 0; j < kFieldGroup; ++j) {
    const int f = min(f0 + j, A.nf - 1);
    bc[j] = (int)A.bt[f][(int64_t)p * A.bts[f]];
    bv[j] = A.b[f][p];
  }
  // both kinds' arrays are always allocated (a kind no field uses holds
  // unused values), so the loads need not wait for the kinds
  double wD[8], wN[8];
#pragma unroll
  for (int k = 0; k < (1 << D); ++k) {
    wD[k] = W0[(int64_t)k * ng + p];
    wN[k] = W1[(int64_t)k * ng + p];
  }
  const uint32_t skip = code_skip(code);
  double val[kFieldGroup][8];
  // x-adjacent corners (multiplier 1 along x, x not skipped): one 16-byte
  // load per pair, as in fill_single
  const bool pair = !(skip & 1u) && code_r(code, 0) == 1;
  const int lo = code_e(code, 0) < 0 ? -1 : 0;
#pragma unroll
  for (int j = 0; j < kFieldGroup; ++j) {
    const double* F = A.f[min(f0 + j, A.nf - 1)];
    if (pair) {
#pragma unroll
      for (int k = 0; k < (1 << D); k += 2) {
        if (k & skip) {
          val[j][k] = val[j][k + 1] = 0.0;
          continue;
        }
        double two[2];
        __builtin_memcpy(two, F + c + corner_offset(P.g, code, k) + lo, 16);
        val[j][k] = lo ? two[1] : two[0];
        val[j][k + 1] = lo ? two[0] : two[1];
      }
    } else {
#pragma unroll
      for (int k = 1; k < (1 << D); ++k)
        val[j][k] = (k & skip) ? 0.0 : F[c + corner_offset(P.g, code, k)];
    }
  }
  double v[kFieldGroup];
#pragma unroll
  for (int j = 0; j < kFieldGroup; ++j) {
    const bool dir = bc[j] == 0;
    double sum = (dir ? wD[0] : wN[0]) * bv[j];
#pragma unroll
    for (int k = 1; k < (1 << D); ++k)
      if (!(k & skip)) sum += (dir ? wD[k] : wN[k]) * val[j][k];
    v[j] = sum;
  }
  if (live)
#pragma unroll
    for (int j = 0; j < kFieldGroup; ++j)
      if (f0 + j < A.nf) A.f[f0 + j][c] = v[j];
}

template <int D>
__device__ __forceinline__ void fill_ghost(const FillArgs& A, int p) {
  const PlanD& P = A.P;
  const bool live = P.blk[p] < 0;
  const int c = P.cell[p];
  const uint32_t code = P.code[p];
  // straight-line groups (kMaxFields = 2 * kFieldGroup), so the first
  // group's independent loads issue together with the metadata loads
  fill_group<D>(A, p, 0, live, c, code);
  if (A.nf > kFieldGroup) fill_group<D>(A, p, kFieldGroup, live, c, code);
}

// Units of level `level` (1-based), every field; threads tid < nthreads each
// take units round-robin, with ws[tid] as workspace.
template <int D>
__device__ __forceinline__ void fill_units_of_level(const FillArgs& A, int level, UnitWS* ws,
                                                    int tid, int nthreads) {
  const PlanD& P = A.P;
  for (int s = tid; s < P.nunits; s += nthreads) {
    if (P.unit_lev[s] != level) continue;
    for (int f = 0; f < A.nf; ++f) fill_unit_field<D>(P, s, A.f[f], A.b[f], A.bt[f], A.kind[f], ws[tid]);
  }
}

// A value not known yet, in a field's ghost slot (k_fill_flow): a NaN no
// arithmetic produces; a result that equals it (an input's NaN passed
// through) is stored as another NaN.
constexpr unsigned long long kFillOpen = 0x7ff85eed0f11e57aull;

__device__ __forceinline__ double fill_result(double v) {
  return __double_as_longlong(v) == (long long)kFillOpen ? __longlong_as_double(0x7ff8000000000000LL)
                                                         : v;
}

// One field of one ghost (the batched kernel's inner step).  Waited: in a launch
// whose values others then wait for.
template <int D, bool Waited = false>
__device__ __forceinline__ void fill_single(const PlanD& P, int p, double* F, const double* b,
                                            const uint8_t* bt, int kind) {
  const int blk = P.blk[p];
  const int c = P.cell[p];
  const uint32_t code = P.code[p];
  double dl[3], nn[3], w[8], val[8];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    dl[a] = a < D ? P.dl[a][p] : 0.0;
    nn[a] = a < D ? P.nn[a][p] : 0.0;
  }
  const int bc = kind == 2 ? (int)bt[p] : kind;
  const double bv = b[p];
  if (blk >= 0) return;
  const uint32_t skip = code_skip(code);
  if (!(skip & 1u) && code_r(code, 0) == 1) {
    // corners k and k + 1 differ by one cell along x: one 16-byte load per
    // pair (corner 0's partner is the ghost's own slot, read and unused)
    const int lo = code_e(code, 0) < 0 ? -1 : 0;
#pragma unroll
    for (int k = 0; k < (1 << D); k += 2) {
      if (k & skip) {
        val[k] = val[k + 1] = 0.0;
        continue;
      }
      double two[2];
      __builtin_memcpy(two, F + c + corner_offset(P.g, code, k) + lo, 16);
      val[k] = lo ? two[1] : two[0];
      val[k + 1] = lo ? two[0] : two[1];
    }
  } else {
#pragma unroll
    for (int k = 1; k < (1 << D); ++k)
      val[k] = (k & skip) ? 0.0 : F[c + corner_offset(P.g, code, k)];
  }
  double X[3];
  stencil_span(P.g, code, c, X);
  ghost_weights<D>(dl, nn, X, bc, w);
  double v = w[0] * bv;
#pragma unroll
  for (int k = 1; k < (1 << D); ++k)
    if (!(k & skip)) v += w[k] * val[k];
  F[c] = Waited ? fill_result(v) : v;
}

// a value that another workgroup may be about to post, and its posting
__device__ __forceinline__ unsigned long long poll_value(const double* p) {
  return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void post_value(double* p, double v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p),
                     (unsigned long long)__double_as_longlong(fill_result(v)), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// The value of ghost p of a field that others may still be filling, posted,
// without waiting: as long as one of its corners is open, the thread goes down
// to that ghost, and from there on, until one has all its corners; it posts
// that one's value (the same, whoever computes it) and starts again from p.
// Corners lie in lower levels and each round leaves one ghost fewer open, so
// this ends whatever other workgroups do.
template <int D>
__device__ __forceinline__ void fill_help(const PlanD& P, int p, double* F,
                                          const double* __restrict__ b,
                                          const uint8_t* __restrict__ bt, int kind) {
  for (int cur = p;;) {
    const int c = P.cell[cur];
    const uint32_t code = P.code[cur], skip = code_skip(code), ghosts = code_ghosts(code);
    double val[8];
    int open = -1;
#pragma unroll
    for (int k = 1; k < (1 << D); ++k) {
      if (k & skip) continue;
      const int q = c + corner_offset(P.g, code, k);
      const unsigned long long x = poll_value(F + q);
      if (((ghosts >> k) & 1u) && x == kFillOpen) open = q;
      val[k] = __longlong_as_double((long long)x);
    }
    if (open >= 0) {
      cur = ghost_at(P, open);
      continue;
    }
    double dl[3], nn[3], w[8], X[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      dl[a] = a < D ? P.dl[a][cur] : 0.0;
      nn[a] = a < D ? P.nn[a][cur] : 0.0;
    }
    stencil_span(P.g, code, c, X);
    ghost_weights<D>(dl, nn, X, kind == 2 ? (int)bt[cur] : kind, w);
    double v = w[0] * b[cur];
#pragma unroll
    for (int k = 1; k < (1 << D); ++k)
      if (!(k & skip)) v += w[k] * val[k];
    post_value(F + c, v);
    if (cur == p) return;
    cur = p;
  }
}

// Ghost p of a level above the first, whose wave's lanes each hold such a
// ghost: its fluid corners and weights are gathered, the slots of its ghost
// corners (the code's mask) polled until each holds a value, its own stored.
// After `polls` the lanes still waiting compute what they wait for.
template <int D>
__device__ __forceinline__ void fill_wait(const PlanD& P, int p, double* F,
                                          const double* __restrict__ b,
                                          const uint8_t* __restrict__ bt, int kind, int polls) {
  const int c = P.cell[p];
  const uint32_t code = P.code[p];
  double dl[3], nn[3], w[8], val[8];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    dl[a] = a < D ? P.dl[a][p] : 0.0;
    nn[a] = a < D ? P.nn[a][p] : 0.0;
  }
  const int bc = kind == 2 ? (int)bt[p] : kind;
  const double bv = b[p];
  const uint32_t skip = code_skip(code);
  uint32_t open = code_ghosts(code);
#pragma unroll
  for (int k = 1; k < (1 << D); ++k)
    val[k] = (k & skip) || ((open >> k) & 1u) ? 0.0 : F[c + corner_offset(P.g, code, k)];
  double X[3];
  stencil_span(P.g, code, c, X);
  ghost_weights<D>(dl, nn, X, bc, w);
  bool done = false;
  for (int left = polls;; --left) {
    if (!done) {
      unsigned long long x[8];
#pragma unroll
      for (int k = 1; k < (1 << D); ++k)
        x[k] = (open >> k) & 1u ? poll_value(F + c + corner_offset(P.g, code, k)) : kFillOpen;
#pragma unroll
      for (int k = 1; k < (1 << D); ++k)
        if (x[k] != kFillOpen) {
          val[k] = __longlong_as_double((long long)x[k]);
          open &= ~(1u << k);
        }
      if (!open) {
        double v = w[0] * bv;
#pragma unroll
        for (int k = 1; k < (1 << D); ++k)
          if (!(k & skip)) v += w[k] * val[k];
        post_value(F + c, v);
        done = true;
      }
    }
    if (__ballot(!done) == 0ull) return;
    if (left <= 0) {
      if (!done) fill_help<D>(P, p, F, b, bt, kind);
      return;
    }
  }
}

// --------------------------------------------------------------------------
// The fill of one field of a 2D plan by one workgroup, in LDS.
//
// A prologue takes every ghost at once into a record of kRecWords doubles:
// the term of its boundary value and, per stencil corner, a factor and the
// LDS place of the value it goes with: for a corner that is a ghost the
// weight and that ghost's record, else the product of weight and fluid value
// and a constant 1, for a skipped corner -0 (which a sum passes over, -0
// included) and the 1.  So a ghost is r0 + r1 g1 + r2 g2 + r3 g3, added in
// corner order as fill_single adds it, with the same bits; the first word
// becomes its value.  Level 1 is computed there.
//
// The other levels are swept by one wave.  A 2D level holds a few dozen
// ghosts, which one wave covers; within it LDS accesses are in order, so a
// level needs no barrier and no wait but for its own corners, and the next
// level's records are read meanwhile.  (A barrier of all waves a level took
// 0.40 us, every ghost polling its corners 0.33 us, with sixteen waves
// sharing the LDS; this one 0.21 us.)  Coupled units are solved from the
// members' records by eight lanes, as fill_unit_field solves them.
//
// Bound by that chain along the levels after one gather of every ghost's
// stencil by one compute unit (4.8 us below).  4096^2 airfoil, 2,083 ghosts,
// three fields: 21.6 us where its place in the cell gives 67 levels, 29.1 where
// it gives 111, against 121 and more for a level at a time from HBM; 128^2
// circle, 106 ghosts: 6 against 11.
// --------------------------------------------------------------------------
constexpr int kRecWords = 5;
constexpr int kRecUnitWS = 8;    // unit workspaces
constexpr uint64_t kRecMember = 1ull << 63;

// A load through a global-address-space pointer (the plan's and the
// field's arrays are device memory): a flat load would also count against
// the LDS wait counter that every LDS access of the sweep waits on.
template <class T>
__device__ __forceinline__ T gload(const T* p) {
  return *(const __attribute__((address_space(1))) T*)p;
}
__device__ __forceinline__ void gstore(double* p, double v) {
  *(__attribute__((address_space(1))) double*)p = v;
}

// LDS bytes for ng ghosts (nunits of 0: no unit workspaces): the constant
// 1, the records and 64 more that are read but not used, the workspaces
__host__ __device__ __forceinline__ size_t fill_lds_bytes(int ng, int nunits) {
  return sizeof(double) * (1 + (size_t)kRecWords * (ng + 64)) +
         (nunits ? kRecUnitWS * sizeof(UnitWS) : 0);
}
// (places in LDS are 16-bit counts of doubles)
__host__ __device__ __forceinline__ bool fill_lds_ok(const PlanD& P) {
  return P.g.dim == 2 && P.cgi && 1 + (int64_t)kRecWords * P.ng < 65536;
}

// Coupled unit u: (I - W_int) phi = W_ext phi_ext + w0 b, assembled from the
// members' records in fill_unit_field's order.
__device__ __forceinline__ void unit_lds2(const PlanD& P, int u, double* lds, UnitWS& ws) {
  double* rec = lds + 1;
  const int k = P.unit_cnt[u];
  for (int i = 0; i < k; ++i) ws.mem[i] = P.unit_mem[u * kMaxUnit + i];
  for (int i = 0; i < k; ++i) {
    const double* r = rec + (int64_t)kRecWords * ws.mem[i];
    const uint64_t pk = (uint64_t)__double_as_longlong(r[4]);
    for (int t = 0; t < k; ++t) ws.M[i * k + t] = (t == i) ? 1.0 : 0.0;
    double rr = r[0];
    for (int c = 1; c < 4; ++c) {
      const int at = (int)((pk >> (16 * (c - 1))) & 0xffffu);
      int t = -1;
      for (int s = 0; s < k; ++s)
        if (1 + kRecWords * ws.mem[s] == at) t = s;
      if (t >= 0) ws.M[i * k + t] -= r[c];
      else rr += r[c] * lds[at];
    }
    ws.rhs[i] = rr;
  }
  ws_solve(ws, k);
  for (int i = 0; i < k; ++i) rec[(int64_t)kRecWords * ws.mem[i]] = ws.rhs[i];
}

// By a whole workgroup (any multiple of 64 threads); lds: fill_lds_bytes of
// it.  Ends with a barrier behind every store.
__device__ __forceinline__ void fill_lds2(const PlanD& P, const int32_t* __restrict__ lev_off,
                                          int nl, double* __restrict__ F,
                                          const double* __restrict__ b,
                                          const uint8_t* __restrict__ bt, int kind,
                                          double* __restrict__ lds) {
  const int T = blockDim.x, tid = threadIdx.x, ng = P.ng;
  double* rec = lds + 1;
  const int n1 = gload(lev_off + 1);
  if (tid == 0) lds[0] = 1.0;
  if (tid < 64) {   // the records past the last: they name the constant only
    double* q = rec + (int64_t)kRecWords * (ng + tid);
#pragma unroll
    for (int k = 0; k < kRecWords; ++k) q[k] = 0.0;
  }
  // two ghosts of a thread at a time, each array of both read together, then
  // their corners; a position past the end reads the last ghost's
  constexpr int kB = 2;
#pragma unroll 1
  for (int p0 = tid; p0 < ng; p0 += kB * T) {
    int c[kB], blk[kB], gi[kB][3], bc[kB];
    uint32_t code[kB];
    double dl[kB][2], nn[kB][2], r[kB][4];
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const int p = min(p0 + i * T, ng - 1);
      c[i] = gload(P.cell + p);
      code[i] = gload(P.code + p);
      blk[i] = gload(P.blk + p);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        dl[i][a] = gload(P.dl[a] + p);
        nn[i][a] = gload(P.nn[a] + p);
      }
      bc[i] = kind == 2 ? (int)gload(bt + p) : kind;
      r[i][0] = gload(b + p);
#pragma unroll
      for (int k = 0; k < 3; ++k) gi[i][k] = gload(P.cgi + (int64_t)k * P.cgi_stride + p);
    }
#pragma unroll
    for (int i = 0; i < kB; ++i)
#pragma unroll
      for (int k = 1; k < 4; ++k)
        r[i][k] = gload(F + c[i] + (gi[i][k - 1] == -1 ? corner_offset(P.g, code[i], k) : 0));
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const int p = p0 + i * T;
      if (p >= ng) continue;
      double d3[3] = {dl[i][0], dl[i][1], 0.0}, n3[3] = {nn[i][0], nn[i][1], 0.0}, X[3], w[8];
      stencil_span(P.g, code[i], c[i], X);
      ghost_weights<2>(d3, n3, X, bc[i], w);
      double v = w[0] * r[i][0];
      uint64_t pk = blk[i] >= 0 ? kRecMember : 0ull;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int g = gi[i][k];
        r[i][k + 1] = g >= 0 ? w[k + 1] : g == -1 ? w[k + 1] * r[i][k + 1] : -0.0;
        pk |= (uint64_t)(g >= 0 ? 1 + kRecWords * g : 0) << (16 * k);
      }
      double* q = rec + (int64_t)kRecWords * p;
      if (p < n1 && blk[i] < 0) {   // reads no ghost
        v = v + r[i][1];
        v = v + r[i][2];
        v = v + r[i][3];
      }
      q[0] = v;
#pragma unroll
      for (int k = 1; k < 4; ++k) q[k] = r[i][k];
      q[4] = __longlong_as_double((long long)pk);
    }
  }
  __syncthreads();
  if (tid < 64) {
    const int lane = tid, nunits = P.nunits;
    UnitWS* ws = reinterpret_cast<UnitWS*>(rec + (int64_t)kRecWords * (ng + 64));
    // lowest level of a unit this lane has to solve
    int unext = 0x7fffffff;
    if (lane < kRecUnitWS)
      for (int s = lane; s < nunits; s += kRecUnitWS) unext = min(unext, gload(P.unit_lev + s));
    // level offsets 64 at a time, lane j holding lev_off[base + j]
    int vlev = lane <= nl ? gload(lev_off + lane) : 0;
    double* const mine = rec + (int64_t)kRecWords * lane;
    // one level [lo, hi): w holds the wave's first records of it, wn receives
    // the next level's (from hi on), read behind this level's corners
    auto level = [&](int l, int lo, int hi, const double (&w)[kRecWords], double (&wn)[kRecWords]) {
      for (int p = lo + 64; p < hi; p += 64) {   // a wide level's other records
        double* r = mine + (int64_t)kRecWords * p;
        if (p + lane >= hi) continue;
        const uint64_t pk = (uint64_t)__double_as_longlong(r[4]);
        double v = r[0];
#pragma unroll
        for (int k = 0; k < 3; ++k) v = v + r[k + 1] * lds[(pk >> (16 * k)) & 0xffffu];
        if (!(pk & kRecMember)) r[0] = v;
      }
      const uint64_t pk = (uint64_t)__double_as_longlong(w[4]);
      double g[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) g[k] = lds[(pk >> (16 * k)) & 0xffffu];
#pragma unroll
      for (int k = 0; k < kRecWords; ++k) wn[k] = mine[(int64_t)kRecWords * hi + k];
      double v = w[0];
#pragma unroll
      for (int k = 0; k < 3; ++k) v = v + w[k + 1] * g[k];
      // (members of a unit: with their unit, below)
      if (lo + lane < hi && !(pk & kRecMember)) mine[(int64_t)kRecWords * lo] = v;
      if (nunits && __ballot(unext == l + 1) != 0ull) {
        // lane s < kRecUnitWS takes units s, s + kRecUnitWS, ...; unext is
        // the lowest level among those not solved yet
        if (unext == l + 1) {
          unext = 0x7fffffff;
          for (int s = lane; s < nunits; s += kRecUnitWS) {
            const int ul = gload(P.unit_lev + s);
            if (ul == l + 1) unit_lds2(P, s, lds, ws[lane]);
            else if (ul > l + 1) unext = min(unext, ul);
          }
        }
      }
    };
    auto bound = [&](int l) {   // lev_off[l], l <= nl, called for l = 2, 3, ...
      if ((l & 63) == 0) vlev = l + lane <= nl ? gload(lev_off + l + lane) : 0;
      return __builtin_amdgcn_readlane(vlev, l & 63);
    };
    double wa[kRecWords], wb[kRecWords];
#pragma unroll
    for (int k = 0; k < kRecWords; ++k) wa[k] = 0.0;
    // level 1 is done but for its units
    level(0, n1, n1, wa, wb);
    int lo = n1;
    for (int l = 1; l < nl; l += 2) {
      int hi = bound(l + 1);
      level(l, lo, hi, wb, wa);
      lo = hi;
      if (l + 1 >= nl) break;
      hi = bound(l + 2);
      level(l + 1, lo, hi, wa, wb);
      lo = hi;
    }
  }
  __syncthreads();
  for (int p = tid; p < ng; p += T) gstore(F + gload(P.cell + p), rec[(int64_t)kRecWords * p]);
  __syncthreads();
}

}  // namespace gcr
